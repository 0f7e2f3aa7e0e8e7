// The reverse walk of the backward pass (bf16 storage): one workgroup owns a run of consecutive chunks of a sequence,
// or a span of a packed batch's chunks, and walks it from the last chunk to the first with the state gradient in fp32
// MFMA accumulators.  The formulas are those at the top of bwd_grad.hip; with the state gradient carried as
//     E_n = D'_n + Q~_n^T dO_n ,   D'_n = (g_n / G_m,n) dS_{n+1} ,   dS_n = G_m,n E_n .
//
// Layout.  A wave owns the 32 x 32 tile (row tile rt, channel tile at) of everything that is [token][channel], and a
// lane the 16 tokens of one channel that the accumulator of a 32 x 32 product gives it: tokens 32 rt + 8 c + 4 g + j,
// channel 32 at + lane % 32 (c, j = 0..3, g = lane / 32).  The gate products are formed in that layout: four
// tokens in a row in a lane, eight such groups to a tile, whose totals the two half waves exchange.  The mid-chunk reference is
// the boundary of the two row tiles, so a wave finds every factor of its tile by itself, without a word from another one; and the
// products X, Y1, Ks leave their MFMAs in the very registers the element-wise end wants them in.  (The walk this replaced
// kept a channel pair of eight consecutive tokens in a lane: block totals through LDS, 96 KB of fp32 staging written and read
// per chunk, seven barriers instead of three.)
// Rows arrive as 16-byte vectors; those of f and q go through the wave's own corner of the operand tiles and
// come back from it by transpose reads.  Q~ and K~ are kept transposed, [channel][token], which is how a lane writes
// four tokens at once.  dq, df, dv leave from the accumulators: neighbouring lanes trade halves, so that each holds a pair of channels.
// Chunks are addressed through buffer descriptors that cover exactly their tokens: rows that stand for no token read as
// zero (their gates are set to one) and are not stored, in ragged chunks and in fine ones (ChunkRows), without a branch.
// Where a chunk's rows lie too far apart for a descriptor (walk_rows.hpp), kernels of their own (FAR) take 64-bit row addresses.
//
// What bounds it, per chunk of 128 x 128 and compute unit (15.6 kcycles with everything in the caches, 6.6 us): 8.0 kcycles of vector
// instructions, 6.8 of LDS, 3.2 of MFMA (SQ counters), of which the matrix stage and the element-wise stages overlap little; over
// buffers that leave the caches, memory as much: 720 MB at 4.3 to 4.8 TB/s.  us, the walk it replaced -> this one, six sets of buffers in
// turn (the benchmark's two: 156 to 160): training pair's backward
// of 8 x 16 heads of 128, 2048 tokens 190 -> 173, gate formed in the walk, token-major 213 -> 197; 2 x 16 heads, 16384 tokens, fp32 gates 449 -> 404;
// 16 x 16 heads, 512 tokens 87 -> 74; 8 x 32 heads of 64, 2000 tokens, gate formed 179 -> 173, 16 x 32, 512 tokens 66 -> 60;
// 8 x 16 heads of 64 x 128, 1024 tokens 91 -> 70, of 128 x 64 73 -> 67.
#include "bwd_common.hpp"
#include "walk_rows.hpp"

namespace hgrn2 {

// Workgroups of eight waves, one on a compute unit; heads of 64 x 64: four waves, two on a compute unit.
constexpr int walk_waves(int dk, int dv) { return dk == 64 && dv == 64 ? 4 : 8; }

template <int DK, int DV> struct WalkLds {
    static constexpr int C = kChunk;
    // Pitches in elements.  In banks of four bytes they are 36 (rows of 64 elements), 76 (128) and 44 (64 + 24): rows that a
    // 16-byte or an 8-byte access touches at once lie four banks apart, and 36 and 76 also keep apart the four rows of
    // 8 banks of a transpose read (44 does not: rows 0 and 3 overlap; 68 would put them on top of each other).
    static constexpr int PT = C + 8;        // Q~, K~ [DK][PT]
    static constexpr int PV = DV + 24;      // dO [C][PV], D' [DK][PV]   (columns in the order of the state fragments)
    static constexpr int PVR = DV + 8;      // V [C][PVR]                (the same order)
    static constexpr int PC = C + 8;        // P^T, dP^T [C][PC]
    static constexpr size_t qt = 0;
    static constexpr size_t kt = qt + (size_t)DK * PT * 2;
    static constexpr size_t vm = kt + (size_t)DK * PT * 2;
    static constexpr size_t dom = vm + (size_t)C * PVR * 2;
    static constexpr size_t dsm = dom + (size_t)C * PV * 2;
    static constexpr size_t pt = dsm + (size_t)DK * PV * 2;
    static constexpr size_t dpt = pt + (size_t)C * PC * 2;
    static constexpr size_t tot = dpt + (size_t)C * PC * 2;             // [2][2][DK] fp32: gate products of the row tiles (light walk: two sets)
    static constexpr size_t ex = tot + (size_t)4 * DK * 4;              // [2][DK] fp32: the tiles' sums of e' and of K~ Ks
    static constexpr size_t stash = ex + (size_t)2 * DK * 4;            // [2][NT] 16 bytes: sa, sz of every lane (gates formed in the walk)
    static constexpr size_t total = stash + (size_t)walk_waves(DK, DV) * 64 * 32;
    static_assert(total * (8 / walk_waves(DK, DV)) <= 160 * 1024, "LDS budget of the workgroups of a compute unit");
    // the light walk alone (bwd_ends_kernel): one set of tiles, two workgroups on a compute unit
    static constexpr size_t lq = 0;
    static constexpr size_t ld = lq + (size_t)DK * PT * 2;
    static constexpr size_t lt = ld + (size_t)C * PV * 2;
    static constexpr size_t light_total = lt + (size_t)4 * DK * 4;
};

typedef Mma<__bf16> WM;
typedef WM::frag wfrag;

// ---- rows of a chunk through buffer descriptors -----------------------------------------------------------------
typedef __amdgpu_buffer_rsrc_t WalkRsrc;
// Stores of the gradients: non-temporal (nt), at system scope (sc1).  A store covers half lines, of which the wave of the next channel tile
// writes the other half; with nt alone many left the caches one by one (16 x 16 heads, 2048 tokens: 490 MB written instead of 403), ordinary
// stores push what is read twice out of them (512 tokens, one set of buffers: 77 us instead of 64).
constexpr int kWalkStream = 2 | 16;

// The tokens of chunk rows cr of a tensor whose sequence starts at element `off`: row r, column c of the chunk lies at
// byte walk_row_offset(r, lo, ld, c, es) with lo the first row that stands for a token.  (FAR: `bytes` is the number of rows.)
struct ChunkSpan { uint32_t lo, hi, bytes; };
template <bool FAR>
__device__ __forceinline__ ChunkSpan chunk_span(const void* tensor, size_t off, const ChunkRows& cr, int ld, int width, int es)
{
    const uintptr_t base = reinterpret_cast<uintptr_t>(tensor) + (off + (size_t)cr.first * (size_t)ld) * es;
    const int rows = max(cr.end - cr.first, 0);
    return ChunkSpan{(uint32_t)base, (uint32_t)(base >> 32), FAR ? (uint32_t)rows : walk_chunk_bytes(rows, ld, width, es)};
}
__device__ __forceinline__ WalkRsrc span_rsrc(const ChunkSpan& s)
{
    // (all of it is the same for the whole wave; said again here, since where scalar registers run out the compiler otherwise
    // keeps descriptors in vector registers and loops over the lanes at every access)
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.lo), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.hi);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uintptr_t)lo | ((uintptr_t)hi << 32)), 0,
                                             __builtin_amdgcn_readfirstlane((int)s.bytes), 0x00020000);
}
__device__ __forceinline__ WalkRsrc chunk_rsrc(const void* tensor, size_t off, const ChunkRows& cr, int ld, int width, int es)
{
    return span_rsrc(chunk_span<false>(tensor, off, cr, ld, width, es));
}
// (FAR) 16 or 4 bytes at row `row`, counted from the span's first one, and column `col`; zero where no token is
template <typename V>
__device__ __forceinline__ V far_load(const ChunkSpan& s, int row, int ld, int col, int es)
{
    const uintptr_t base = (uintptr_t)s.lo | ((uintptr_t)s.hi << 32);
    V x = {};
    if ((uint32_t)row < s.bytes) x = *reinterpret_cast<const V*>(base + ((size_t)row * (size_t)ld + (size_t)col) * es);
    return x;
}
__device__ __forceinline__ u32x4 rsrc_load16(WalkRsrc r, unsigned off)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// The raw rows of a chunk that a thread holds while they are in flight.
template <bool GATE_BF16> struct RawGate;
template <> struct RawGate<true> { u32x4 v[2]; };
template <> struct RawGate<false> { float v[16]; };

struct WalkWave {         // which tiles a wave owns
    int w, at, rt;
    bool has_a;
};
template <int NAT, int NW> __device__ __forceinline__ WalkWave walk_wave(int w)
{
    WalkWave ww;
    ww.w = w;
    ww.at = w % NAT;
    ww.has_a = 2 * NAT == NW || w < 2 * NAT;
    ww.rt = ww.has_a ? w / NAT : 0;
    return ww;
}

// f and q of the wave's tile: bf16 rows as four 16-byte pieces each, lane l the piece l % 4 of rows l / 4 and l / 4 + 16; fp32 gates
// as the lane will use them, a row of 32 channels per half wave and load.
template <int DK, bool GATE_BF16, bool FAR>
__device__ __forceinline__ void load_gate_query(const BwdGradParams& p, RawGate<GATE_BF16>& rf, u32x4 (&rq)[2], const ChunkAt& c,
                                                const WalkWave& ww, int lane)
{
    const ChunkRows cr = chunk_rows(p.lay.sub, c.n, c.sv.N);
    const int ld = (int)p.lay.sn_k, lo = cr.first - cr.tok0;
    if constexpr (FAR) {
        const ChunkSpan f = chunk_span<true>(p.f, c.sv.off_k, cr, ld, DK, GATE_BF16 ? 2 : 4), q = chunk_span<true>(p.q, c.sv.off_k, cr, ld, DK, 2);
        const int row = 32 * ww.rt + (lane >> 2) - lo, col = 32 * ww.at + 8 * (lane & 3);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            rq[i] = far_load<u32x4>(q, row + 16 * i, ld, col, 2);
            if constexpr (GATE_BF16) rf.v[i] = far_load<u32x4>(f, row + 16 * i, ld, col, 2);
        }
        if constexpr (!GATE_BF16) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                rf.v[i] = far_load<float>(f, 32 * ww.rt + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3) - lo, ld, 32 * ww.at + (lane & 31), 4);
        }
        return;
    }
    const WalkRsrc f = chunk_rsrc(p.f, c.sv.off_k, cr, ld, DK, GATE_BF16 ? 2 : 4), q = chunk_rsrc(p.q, c.sv.off_k, cr, ld, DK, 2);
    const unsigned at = walk_row_offset(32 * ww.rt + (lane >> 2), lo, ld, 32 * ww.at + 8 * (lane & 3), 2), step = (unsigned)(32 * ld);
    rq[0] = rsrc_load16(q, at);
    rq[1] = rsrc_load16(q, at + step);
    if constexpr (GATE_BF16) {
        rf.v[0] = rsrc_load16(f, at);
        rf.v[1] = rsrc_load16(f, at + step);
    } else {
        const unsigned a = walk_row_offset(32 * ww.rt + 4 * (lane >> 5), lo, ld, 32 * ww.at + (lane & 31), 4);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            rf.v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(f, a + (unsigned)((8 * (i >> 2) + (i & 3)) * ld * 4), 0, 0));
    }
}

// 16 columns of a row of V or dO per thread
template <int DV, bool FAR>
__device__ __forceinline__ void load_value_rows(const BwdGradParams& p, Raw16<__bf16>& r, const void* tensor, const ChunkAt& c, int tid)
{
    const ChunkRows cr = chunk_rows(p.lay.sub, c.n, c.sv.N);
    const int ld = (int)p.lay.sn_v, row = tid / (DV / 16), grp = tid % (DV / 16);
    if constexpr (FAR) {
        const ChunkSpan s = chunk_span<true>(tensor, c.sv.off_v, cr, ld, DV, 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) r.v[i] = far_load<u32x4>(s, row - (cr.first - cr.tok0), ld, 16 * grp + 8 * i, 2);
        return;
    }
    const WalkRsrc d = chunk_rsrc(tensor, c.sv.off_v, cr, ld, DV, 2);
    const unsigned at = walk_row_offset(row, cr.first - cr.tok0, ld, 16 * grp, 2);
    r.v[0] = rsrc_load16(d, at);
    r.v[1] = rsrc_load16(d, at + 16);
}

// The lane's number, from nothing that would have to be kept in a register (and, being opaque, is not).
__device__ __forceinline__ int lane_id()
{
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// A wave-uniform value that the compiler cannot see through.
__device__ __forceinline__ int opaque_uniform(int x)
{
    int y;
    asm volatile("s_mov_b32 %0, %1" : "=s"(y) : "s"(x));
    return y;
}

// ---- the tile layout ----------------------------------------------------------------------------------------------
// x of lane % 32 and of lane % 32 + 32
__device__ __forceinline__ f32x2 both_halves(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return f32x2{__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// LDS accesses of a wave to its own corner of a tile are in order; this keeps the compiler from moving them.
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The wave's tile of raw bf16 rows -> corner of a [channel][token] tile (as 32 rows of 32 channels) -> 16 values a lane.
template <int PT> __device__ __forceinline__ void put_raw_tile(__bf16* corner, const u32x4 (&raw)[2], int lane)
{
    __bf16* d = corner + (size_t)(lane >> 2) * PT + 8 * (lane & 3);
    *reinterpret_cast<u32x4*>(d) = raw[0];
    *reinterpret_cast<u32x4*>(d + 16 * PT) = raw[1];
}
template <int PT> __device__ __forceinline__ void get_tile(float (&x)[16], const __bf16* corner, int lane)
{
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const int i16 = lane & 15;
    const __bf16* s = corner + (size_t)(4 * (lane >> 5) + (i16 >> 2)) * PT + (lane & 16) + 4 * (i16 & 3);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const bf16x4 t = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(s + 8 * c * PT));
#pragma unroll
        for (int j = 0; j < 4; ++j) x[4 * c + j] = (float)t[j];
    }
}

// Gates of rows that stand for no token are one.
__device__ __forceinline__ void fill_gates(float (&f)[16], const ChunkRows& cr, int rt, int lane)
{
    const int lo = cr.first - cr.tok0, hi = cr.end - cr.tok0;
    if (32 * rt < lo || 32 * rt + 32 > hi) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = 32 * rt + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
            f[i] = (row >= lo && row < hi) ? f[i] : 1.0f;
        }
    }
}

// The gates and the q of the tile as floats.
template <int PT, bool GATE_BF16, bool GATED>
__device__ __forceinline__ void unpack_tile(float (&f)[16], float (&q)[16], const RawGate<GATE_BF16>& rf,
                                            const u32x4 (&rq)[2], __bf16* f_corner, __bf16* q_corner, const ChunkRows& cr,
                                            const WalkWave& ww, int lane, float beta)
{
    put_raw_tile<PT>(q_corner, rq, lane);
    if constexpr (GATE_BF16) put_raw_tile<PT>(f_corner, rf.v, lane);
    wave_order();
    if constexpr (GATE_BF16) get_tile<PT>(f, f_corner, lane);
    else {
#pragma unroll
        for (int i = 0; i < 16; ++i) f[i] = rf.v[i];
    }
    get_tile<PT>(q, q_corner, lane);
    wave_order();
    if constexpr (GATED) {
#pragma unroll
        for (int i = 0; i < 16; ++i) f[i] = lower_bounded_gate(f[i], beta);
    }
    fill_gates(f, cr, ww.rt, lane);
}

// Inside the groups of four tokens: a inclusive products from the group's start, z exclusive ones to its end.
__device__ __forceinline__ void group_products(float (&a)[16], float (&z)[16], const float (&f)[16])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        a[4 * c] = f[4 * c]; z[4 * c + 3] = 1.0f; z[4 * c + 2] = f[4 * c + 3];
        a[4 * c + 1] = a[4 * c] * f[4 * c + 1]; z[4 * c + 1] = z[4 * c + 2] * f[4 * c + 2];
        a[4 * c + 2] = a[4 * c + 1] * f[4 * c + 2]; z[4 * c] = z[4 * c + 1] * f[4 * c + 1];
        a[4 * c + 3] = a[4 * c + 2] * f[4 * c + 3];
    }
}

// 16 values of the tile layout, columns from `col0` on, to the rows of `dst` (lo: first row that stands for a token).
// Neighbouring lanes trade halves of their bf16 pairs: the even lane then has both channels of the first token of
// two, the odd one of the second, and a store covers four rows with 64 bytes each.
template <bool FAR> struct TileStore {
    WalkRsrc dst;
    unsigned at, sel;
    int ld;
    __device__ __forceinline__ TileStore(const ChunkSpan& span, int rt, int col0, int lo, int ld_, int lane)
        : dst(span_rsrc(span)), at(walk_row_offset(32 * rt + 4 * (lane >> 5) + (lane & 1), lo, ld_, col0 + (lane & 30), 2)),
          sel((lane & 1) ? 0x03020706u : 0x05040100u), ld(ld_)
    {
    }
    // tokens 2 i, 2 i + 1 of the lane's 16
    __device__ __forceinline__ void pair(int i, float x0, float x1) const
    {
        bf16x2 h;
        h.x = (__bf16)x0;
        h.y = (__bf16)x1;
        const uint32_t u = __builtin_bit_cast(uint32_t, h);
        const uint32_t n = __builtin_amdgcn_update_dpp(0u, u, 0xB1, 0xf, 0xf, true);      // the neighbour's
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_perm(n, u, sel), dst, at + (unsigned)((8 * (i >> 1) + 2 * (i & 1)) * ld * 2), 0, kWalkStream);
    }
};
template <> struct TileStore<true> {
    ChunkSpan span;
    int row, col, ld;
    unsigned sel;
    __device__ __forceinline__ TileStore(const ChunkSpan& span_, int rt, int col0, int lo, int ld_, int lane)
        : span(span_), row(32 * rt + 4 * (lane >> 5) + (lane & 1) - lo), col(col0 + (lane & 30)), ld(ld_),
          sel((lane & 1) ? 0x03020706u : 0x05040100u)
    {
    }
    __device__ __forceinline__ void pair(int i, float x0, float x1) const
    {
        bf16x2 h;
        h.x = (__bf16)x0;
        h.y = (__bf16)x1;
        const uint32_t u = __builtin_bit_cast(uint32_t, h);
        const uint32_t n = __builtin_amdgcn_update_dpp(0u, u, 0xB1, 0xf, 0xf, true);
        const int r = row + 8 * (i >> 1) + 2 * (i & 1);
        const uintptr_t base = (uintptr_t)span.lo | ((uintptr_t)span.hi << 32);
        if ((uint32_t)r < span.bytes)
            __builtin_nontemporal_store(__builtin_amdgcn_perm(n, u, sel), reinterpret_cast<uint32_t*>(base + ((size_t)r * (size_t)ld + (size_t)col) * 2));
    }
};

// ---- light walk, last chunk to first, over `count` chunks of one sequence from chunk `cur` on -------------------------
// dS_n = Diag(g_n) dS_{n+1} + Q^_n^T dO_n with Q^ = q G, G the gate product from the chunk's start: no quotient.  The two
// halves of a chunk follow one another, dS = T0 (T1 dS + Q1^T dO1) + Q0^T dO0 with G from the start of each half, so that no wave
// waits for another's products.  The true state gradient in the accumulators (tiles as in walk_body).  SETS = 2: the
// tiles of two chunks in LDS (q_set, d_set elements apart), one barrier a chunk; else two.  Returns the chunk before the last one walked, whose f, q and dO rows are
// then loaded.  decay (null: not wanted): receives the product of the gates passed.
template <int DK, int DV, bool GATE_BF16, bool GATED, int NW, int SETS, int TPW>
__device__ __forceinline__ ChunkAt light_walk(const BwdGradParams& p, __bf16* Qs, int q_set, __bf16* dOs, int d_set, float* tot, ChunkAt cur,
                                              int count, f32x16 (&accD)[TPW], float* decay, RawGate<GATE_BF16>& raw_f, u32x4 (&raw_q)[2],
                                              Raw16<__bf16>& raw_d, const WalkWave& ww)
{
    typedef WalkLds<DK, DV> L;
    constexpr int C = kChunk, NAT = DK / 32, NBT = DV / 32, GPR = DV / 16, PT = L::PT, PV = L::PV;
    const int tid = threadIdx.x;
    const bool has_d = (NAT * NBT) % NW == 0 || ww.w < NAT * NBT, vd_act = 64 * NW == C * GPR || tid < C * GPR;
    const float beta = GATED ? p.beta[(size_t)(cur.bh / p.lay.seg % p.H) * DK + 32 * ww.at + (tid & 31)] : 0.0f;
    auto load = [&](const ChunkAt& c, int lane) {
        if (ww.has_a) load_gate_query<DK, GATE_BF16, false>(p, raw_f, raw_q, c, ww, lane);
        if (vd_act) load_value_rows<DV, false>(p, raw_d, p.dO, c, 64 * ww.w + lane);
    };
    load(cur, tid & 63);
    float g_run = 1.0f;
    for (int li = 0; li < count; ++li) {
        const int lane = lane_id(), r32 = lane & 31, g = lane >> 5;
        const int set = SETS == 2 ? (li & 1) : 0;
        __bf16* Q = Qs + set * q_set;
        __bf16* dO = dOs + set * d_set;
        float* T = tot + set * 2 * DK;
        if (vd_act) raw_d.store_swapped(dO + (size_t)((64 * ww.w + lane) / GPR) * PV + 16 * ((64 * ww.w + lane) % GPR));
        const ChunkRows cr = chunk_rows(p.lay.sub, cur.n, cur.sv.N);
        if (ww.has_a) {
            const int ch = 32 * ww.at + r32;
            __bf16* corner = Q + (size_t)(32 * ww.at) * PT + 32 * ww.rt;
            float f[16], q[16], a[16], z[16];
            // (both raw tiles pass through the one corner, one after the other)
            if constexpr (GATE_BF16) {
                put_raw_tile<PT>(corner, raw_f.v, lane);
                wave_order();
                get_tile<PT>(f, corner, lane);
                wave_order();
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) f[i] = raw_f.v[i];
            }
            put_raw_tile<PT>(corner, raw_q, lane);
            wave_order();
            get_tile<PT>(q, corner, lane);
            wave_order();
            if constexpr (GATED) {
#pragma unroll
                for (int i = 0; i < 16; ++i) f[i] = lower_bounded_gate(f[i], beta);
            }
            fill_gates(f, cr, ww.rt, lane);
            group_products(a, z, f);
            float run = 1.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x2 t = both_halves(a[4 * c + 3]);
                const float B = g ? run * t.x : run;
                run *= t.x * t.y;
                bf16x4 x;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = (__bf16)(q[4 * c + j] * (B * a[4 * c + j]));
                *reinterpret_cast<bf16x4*>(corner + (size_t)r32 * PT + 8 * c + 4 * g) = x;
            }
            if (g == 0) T[ww.rt * DK + ch] = run;
        }
        ChunkAt nxt = cur;            // the chunk before, in the same sequence
        nxt.n = cur.n - 1;
        if (nxt.n < 0) nxt.n = 0;     // (the walk's last request may be one too many: it re-reads the first chunk)
        load(nxt, lane);
        __syncthreads();
        if (has_d) {
            const float t0 = T[32 * ww.at + r32], t1 = T[DK + 32 * ww.at + r32];
            g_run *= t0 * t1;
#pragma unroll
            for (int h = 1; h >= 0; --h) {
                const float t = h ? t1 : t0;
#pragma unroll
                for (int j = 0; j < TPW; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) accD[j][v] *= t;
#pragma unroll
                for (int ks = 2 * h; ks < 2 * h + 2; ++ks) {
                    const wfrag qf = WM::load(Q + (size_t)(32 * ww.at + r32) * PT + 16 * ks + 8 * g);
#pragma unroll
                    for (int j = 0; j < TPW; ++j)
                        WM::mma(accD[j], WM::load_kmajor_swapped(dO, PV, 16 * ks, 32 * ((ww.w + NW * j) / NAT), lane), qf);
                }
            }
        }
        cur.n -= 1;
        if (SETS == 1) __syncthreads();
    }
    if (SETS == 2) __syncthreads();
    if (decay && ww.w < NAT && (tid & 63) < 32) decay[32 * ww.at + (tid & 31)] = g_run;
    return cur;
}

// GROUPED: the walk over a span of a packed batch's chunks.  The chunks of one head, sequence after sequence, are
// cut into `spans` equal pieces, each of which may start and end inside a sequence: the state gradient starts from a
// sequence's grad_hT (or zero) at its last chunk and leaves as its grad_h0 after its first, and the rows of the next chunk of the
// walk -- be it of the sequence before -- are always in flight.  A span that ends inside a sequence first takes the light walk
// over the chunks between its end and the sequence's; or, with `span_add`, adds up what bwd_ends_kernel found for the later
// spans of that sequence:
//     dS = Diag(decay_{s+1}) ( ... Diag(decay_last) grad_hT + add_last ... ) + add_{s+1}.
// FAR: rows too far apart for descriptors.  So many heads are never cut (walk_rows.hpp), and no such walk is light.
template <int DK, int DV, bool GATE_BF16, bool GATED, bool GROUPED, bool FAR>
__device__ __forceinline__ void walk_body(const BwdGradParams& p)
{
    typedef __bf16 T;
    typedef WalkLds<DK, DV> L;
    constexpr int C = kChunk, NW = walk_waves(DK, DV), NT = 64 * NW, NAT = DK / 32, NBT = DV / 32, GPR = DV / 16;
    constexpr int PT = L::PT, PV = L::PV, PVR = L::PVR, PC = L::PC;
    constexpr int NDT = NAT * NBT, TPW = (NDT + NW - 1) / NW;      // tiles of the state gradient, and those of a wave
    static_assert(2 * NAT <= NW && 2 * NBT <= NW, "one tile of each kind per wave");

    extern __shared__ __align__(16) char smem[];
    T* QT = reinterpret_cast<T*>(smem + L::qt);
    T* KT = reinterpret_cast<T*>(smem + L::kt);
    T* Vm = reinterpret_cast<T*>(smem + L::vm);
    T* dOm = reinterpret_cast<T*>(smem + L::dom);
    T* dSm = reinterpret_cast<T*>(smem + L::dsm);
    T* Pt = reinterpret_cast<T*>(smem + L::pt);
    T* dPt = reinterpret_cast<T*>(smem + L::dpt);
    float* tot = reinterpret_cast<float*>(smem + L::tot);
    float* ex = reinterpret_cast<float*>(smem + L::ex);
    f32x4* stash = reinterpret_cast<f32x4*>(smem + L::stash);

    if (not_chosen(p.lay)) return;       // (a packed batch whose table chose the other backward pass; a chunk length not called for)
    const int tid = threadIdx.x;
    const int w_ = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WalkWave ww = walk_wave<NAT, NW>(w_);
    const int w = w_, at = ww.at;
    const bool has_a = ww.has_a, has_b = 2 * NBT == NW || w_ < 2 * NBT, has_d = NDT % NW == 0 || w_ < NDT;
    const bool vd_act = NT == C * GPR || tid < C * GPR;

    int g_head = 0;
    auto chunk_en = [&](int e, int n) {        // GROUPED: chunk n of sequence e of the span's head
        ChunkAt c;
        c.bh = e * p.lay.H + g_head;
        c.n = n;
        c.sv = seq_view<false, DK, DV>(p.lay, p.N, p.NC, c.bh);
        return c;
    };
    // the chunk the walk visits after c: the one before it in its sequence, else the last chunk of
    // the nearest earlier sequence that has tokens; after the very last one, c again
    auto walk_next = [&](const ChunkAt& c) {
        if (c.n > 0) { ChunkAt r = c; r.n = c.n - 1; return r; }
        if constexpr (GROUPED)
            for (int e = c.bh / p.lay.H - 1; e >= 0; --e) {
                const int len = table_read(p.lay.vl, p.lay.B + 1 + e);
                if (len > 0) return chunk_en(e, p.lay.chunks_of(len) - 1);
            }
        return c;
    };

    // the workgroup's chunks
    int n_iter, f_bh = 0, f_run = 0, f_first = 0, f_last = 0;
    int span_first = 0, span_end = 0, span_total = 0;    // GROUPED: the span's chunks and the number of all, counted over the head's chunks
    if constexpr (GROUPED) {
        if ((int)blockIdx.x >= p.lay.spans * p.lay.H) return;
        const int grp = (int)blockIdx.x / p.lay.H;
        g_head = (int)blockIdx.x - grp * p.lay.H;
        const int total = table_read(p.lay.vl, 2 * (p.lay.B + 1) + p.lay.B);       // chunks of one head
        span_first = (int)((long long)grp * total / p.lay.spans);
        span_end = (int)((long long)(grp + 1) * total / p.lay.spans);
        span_total = total;
        n_iter = span_end - span_first;
        // a sequence without tokens hands the gradient of its final state on to its initial state
        // (such sequences lie in no span: they are dealt out by their number)
        if (p.dh0)
            for (int e = grp; e < p.lay.B; e += p.lay.spans)
                if (table_read(p.lay.vl, p.lay.B + 1 + e) == 0)
                    for (int i = tid; i < DK * DV; i += NT) {
                        const size_t x = (size_t)(e * p.lay.H + g_head) * DK * DV + i;
                        p.dh0[x] = p.dhT ? p.dhT[x] : 0.0f;
                    }
    } else {
        f_bh = (int)blockIdx.x / p.R;
        f_run = (int)blockIdx.x - f_bh * p.R;
        if (f_bh >= p.BH) return;
        if (p.light) {
            f_first = p.bnd[f_run];
            f_last = p.bnd[f_run + 1] - 1;
        } else {
            f_first = f_run * p.rc;
            f_last = min(p.NC, f_first + p.rc) - 1;
        }
        n_iter = f_last - f_first + 1;
    }

    // Tiles of the state gradient owned by this wave, tile id w + NW j -> (channel tile id % NAT, which is this wave's `at`;
    // dv tile id / NAT), as [dv][channel].  Element (tile j, register v) of a [dk][dv] fp32 state: a wave-uniform address
    // (sequence, dv tile, group of four registers) plus one per-lane 32-bit byte offset plus a small constant.
    f32x16 accD[TPW];
    float gm_prev = 1.0f;                 // first-half gate product of the chunk done before, channel 32 at + lane % 32
    auto st_lane = [&]() { const int l = lane_id(); return (uint32_t)((32 * at + (l & 31)) * DV + 4 * (l >> 5)) * 4u; };
    auto state_cols = [&](const float* base, size_t seq, int j, int c) {
        return reinterpret_cast<const char*>(base) + (seq * DK * DV + (size_t)(32 * ((w + NW * j) / NAT) + 8 * c)) * 4;
    };
    auto set_state = [&](const float* base, size_t seq) {        // (base may be null: zero)
        if (base && has_d) {              // (one branch: a choice per element would wait for every load by itself)
#pragma unroll
            for (int j = 0; j < TPW; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const char* cols = state_cols(base, seq, j, c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) accD[j][4 * c + e] = *reinterpret_cast<const float*>(cols + st_lane() + 4 * e);
                }
        } else {
#pragma unroll
            for (int j = 0; j < TPW; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) accD[j][v] = 0.0f;
        }
    };
    auto leave_state = [&](float* base, size_t seq) {            // dS = G_m E
#pragma unroll
        for (int j = 0; j < TPW; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                char* cols = const_cast<char*>(state_cols(base, seq, j, c));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    accD[j][4 * c + e] *= gm_prev;
                    *reinterpret_cast<float*>(cols + st_lane() + 4 * e) = accD[j][4 * c + e];
                }
            }
    };
    if constexpr (!GROUPED) {
        if (f_run == p.R - 1 || p.light) set_state(p.dhT, (size_t)f_bh);
        else if (f_run == 0) set_state(p.bound0, (size_t)f_bh);
        else set_state(p.run_state, (size_t)f_bh * p.seg_tail + (size_t)f_run * p.s_sub - 1);
    }
    // the run's (span's) partial sums of the gradient w.r.t. beta, added up chunk after chunk in a fixed order: a row for every
    // row tile and half wave, and as many of zeros (row sets are eight rows everywhere)
    float run_b = 0.0f;
    auto store_run_beta = [&]() {
        int slot = f_bh * p.R + f_run;
        if constexpr (GROUPED) {
            // (beta_spans() row sets per head.  More spans than that leave at most one chunk to a span: those with a chunk
            // take the place of its number, those without fill the places behind.)
            const int grp = (int)blockIdx.x / p.lay.H;
            int grp_slot = grp;
            if (p.lay.spans > p.beta_spans) grp_slot = span_end > span_first ? span_first : span_total + grp - span_first;
            if (grp_slot >= p.beta_spans) return;
            slot = g_head * p.beta_spans + grp_slot;
        }
        if (GATED && has_a) {
            float* row = p.beta_partials + ((size_t)slot * kRowBlocks + 4 * ww.rt + 2 * (lane_id() >> 5)) * DK + 32 * at + (lane_id() & 31);
            row[0] = run_b;
            row[DK] = 0.0f;
        }
    };
    if (n_iter <= 0) {                    // a span without chunks
        store_run_beta();
        return;
    }

    RawGate<GATE_BF16> raw_f;
    u32x4 raw_q[2];
    Raw16<T> raw_v, raw_d;
    auto load_rows_of = [&](const ChunkAt& c, bool values_only, const WalkWave& ww, int lane) {
        if (!values_only) {
            if (has_a) load_gate_query<DK, GATE_BF16, FAR>(p, raw_f, raw_q, c, ww, lane);
            if (vd_act) load_value_rows<DV, FAR>(p, raw_d, p.dO, c, 64 * ww.w + lane);
        }
        if (vd_act) load_value_rows<DV, FAR>(p, raw_v, p.v, c, 64 * ww.w + lane);
    };
    ChunkAt cur;
    {
        int n_light = 0;
        if constexpr (GROUPED) {
            // the sequence the span ends in (found by the table kernel): the last one whose chunks
            // start at or before the span's last chunk
            const int* before = p.lay.vl + 2 * (p.lay.B + 1);
            const int lo = min(max(table_read(p.lay.span_seq, (int)blockIdx.x / p.lay.H), 0), p.lay.B - 1);
            const int nc_e = table_read(before, lo + 1) - table_read(before, lo);
            cur = chunk_en(lo, nc_e - 1);                          // that sequence's last chunk
            n_light = table_read(before, lo + 1) - span_end;       // its chunks after the span
            const int seq_end = table_read(before, lo + 1);
            if (n_light > 0) set_state(p.dhT, (size_t)cur.bh);     // (the chunk loop does that itself for a sequence whose last chunk lies in the span)
            if (n_light > 0 && p.span_add && table_read(p.lay.span_walks, 1) != 0) {
                // the spans from the one in which the sequence ends down to the next one, two requested at a time
                const int span = (int)blockIdx.x / p.lay.H;
                int k = span + 1;
                while (k + 1 < p.lay.spans && (int)((long long)(k + 1) * span_total / p.lay.spans) < seq_end) ++k;
                constexpr int AHEAD = 2;
                if (has_d)
                    for (; k > span; k -= AHEAD) {
                        float dm[AHEAD];
                        f32x4 add[AHEAD][TPW][4];
#pragma unroll
                        for (int u = 0; u < AHEAD; ++u) {
                            const int slot = max(k - u, span + 1) * p.lay.H + g_head;
                            dm[u] = p.span_decay[(size_t)slot * DK + 32 * at + (tid & 31)];
#pragma unroll
                            for (int j = 0; j < TPW; ++j)
#pragma unroll
                                for (int c = 0; c < 4; ++c) add[u][j][c] = *reinterpret_cast<const f32x4*>(state_cols(p.span_add, (size_t)slot, j, c) + st_lane());
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < AHEAD; ++u) {
                            if (k - u <= span) break;
#pragma unroll
                            for (int j = 0; j < TPW; ++j)
#pragma unroll
                                for (int v = 0; v < 16; ++v) accD[j][v] = fmaf(dm[u], accD[j][v], add[u][j][v >> 2][v & 3]);
                        }
                    }
                cur.n -= n_light;                                  // the span's last chunk
                n_light = 0;
            }
        } else {
            cur.bh = f_bh;
            cur.sv = seq_view<false, DK, DV>(p.lay, p.N, p.NC, f_bh);
            n_light = p.light ? p.NC - 1 - f_last : 0;
            cur.n = f_last + n_light;
        }
        if constexpr (FAR) n_light = 0;
        else if (n_light > 0) {
            // (second set: the tiles of K~ and D')
            cur = light_walk<DK, DV, GATE_BF16, GATED, NW, 2>(p, QT, DK * PT, dOm, C * PV, tot, cur, n_light, accD, nullptr, raw_f, raw_q, raw_d, ww);
        }
        load_rows_of(cur, n_light > 0, ww, tid & 63);      // (after a light walk: what the full pass needs on top)
    }
    // (outside the loop: a load in it, though taken only with beta, made the compiler wait for every load in flight)
    const float beta_ = GATED ? p.beta[(size_t)(cur.bh % p.H) * DK + 32 * at + (tid & 31)] : 0.0f;
    // The gate gradient of a chunk waits for the sums of the other row tile, that is for the barrier after its contractions: df = u + other r
    // with r = 1 / f is left in this form, and finished in the next chunk's matrix stage, which leaves the vector unit room.
    // (Gate formed from its pre-activation: r and u carry the factor that turns df into dz, and the shares of beta's gradient go along.)
    float df_u[16], df_r[16], beta_u = 0.0f, beta_r = 0.0f;
    ChunkSpan df_dst = {0u, 0u, 0u};
    int df_lo = 0;
    auto finish_df = [&](const WalkWave& ww, int lane, int ld_k) {
        const float other = ex[(1 - ww.rt) * DK + 32 * ww.at + (lane & 31)];
        const TileStore<FAR> out(df_dst, ww.rt, 32 * ww.at, df_lo, ld_k, lane);
#pragma unroll
        for (int i = 0; i < 8; ++i) out.pair(i, fmaf(other, df_r[2 * i], df_u[2 * i]), fmaf(other, df_r[2 * i + 1], df_u[2 * i + 1]));
        if constexpr (GATED) run_b += fmaf(other, beta_r, beta_u);
    };
    float below_floor = 1.0f;             // smallest product a reciprocal was taken of (reported once, at the end)

    for (int it = 0; it < n_iter; ++it) {
        // indices from values the compiler cannot see through: it would keep dozens of loop-invariant addresses
        // in registers across the loop, and spill (and a reload waits for every load in flight)
        const int lane = lane_id(), r32 = lane & 31, g = lane >> 5;
        float beta = beta_;
        if constexpr (GATED) asm volatile("" : "+v"(beta));
        const WalkWave ww = walk_wave<NAT, NW>(opaque_uniform(w_));
        const int w = ww.w, at = ww.at, rt = ww.rt, ch = 32 * at + r32, ld_k = opaque_uniform((int)p.lay.sn_k), ld_v = (int)p.lay.sn_v;
        const int rt_b = has_b ? w / NBT : 0, bt = w % NBT;            // (row tile, column tile) of dv
        const ChunkRows cr = chunk_rows(p.lay.sub, cur.n, cur.sv.N);
        const int lo = cr.first - cr.tok0;
        T* q_corner = QT + (size_t)(32 * at) * PT + 32 * rt;
        T* k_corner = KT + (size_t)(32 * at) * PT + 32 * rt;

        wfrag sS[2 * NBT];                // G_m S_n of channel tile `at`, operand fragments (contraction over dv)
        if (has_a) {
            const T* s = static_cast<const T*>(p.ws_s) + (cur.sv.chunk0 + (size_t)cur.n) * DK * DV + state_frag_offset(at, 0, NBT, 0, lane);
#pragma unroll
            for (int kk = 0; kk < 2 * NBT; ++kk) sS[kk] = *reinterpret_cast<const wfrag*>(s + 512 * kk);
        }
        // ---------------- operand tiles ----------------
        // With m = product of the gates between the mid-chunk reference and the row:
        //   rows after the reference:  Q~ = q m,   K~ = k / m        rows before it:  Q~ = q / m, K~ = k m
        // m = B a (after) or B z (before) with B the product of the groups between the reference and the row's, and
        // 1/m = z / (B t) or a / (B t) with t the group's total: one reciprocal per group, with a floor under it so that it
        // stays finite outside the supported gate range.  So Q~/q = sa a and K~/k = sz z; sa, sz are kept for the end.
        if (vd_act) {
            const int t = 64 * w + lane;
            raw_v.store_swapped(Vm + (size_t)(t / GPR) * PVR + 16 * (t % GPR));
            raw_d.store_swapped(dOm + (size_t)(t / GPR) * PV + 16 * (t % GPR));
        }
        float f[16], sa[4], sz[4];
        if (has_a) {
            float q[16], a[16], z[16], t_lo[4], t_hi[4];
            unpack_tile<PT, GATE_BF16, GATED>(f, q, raw_f, raw_q, k_corner, q_corner, cr, ww, lane, beta);
            group_products(a, z, f);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x2 t = both_halves(a[4 * c + 3]);
                t_lo[c] = t.x; t_hi[c] = t.y;
            }
            float run = 1.0f;
            if (rt) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float B = g ? run * t_lo[c] : run, m = B * a[4 * c + 3];
                    run *= t_lo[c] * t_hi[c];
                    below_floor = fminf(below_floor, m);
                    sa[c] = B; sz[c] = fast_rcp(fmaxf(m, kTinyProduct));
                }
            } else {
#pragma unroll
                for (int c = 3; c >= 0; --c) {
                    const float B = g ? run : run * t_hi[c], m = B * a[4 * c + 3];
                    run *= t_lo[c] * t_hi[c];
                    below_floor = fminf(below_floor, m);
                    sz[c] = B; sa[c] = fast_rcp(fmaxf(m, kTinyProduct));
                }
            }
            if (g == 0) tot[rt * DK + ch] = run;
            if constexpr (GATED) {        // (sixteen registers of gates formed leave no room for these until the end)
                stash[64 * w + lane] = f32x4{sa[0], sa[1], sa[2], sa[3]};
                stash[NT + 64 * w + lane] = f32x4{sz[0], sz[1], sz[2], sz[3]};
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                bf16x4 qb, kb;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = 4 * c + j;
                    qb[j] = (T)(q[i] * (sa[c] * a[i]));
                    kb[j] = (T)((1.0f - f[i]) * (sz[c] * z[i]));
                }
                *reinterpret_cast<bf16x4*>(q_corner + (size_t)r32 * PT + 8 * c + 4 * g) = qb;
                *reinterpret_cast<bf16x4*>(k_corner + (size_t)r32 * PT + 8 * c + 4 * g) = kb;
            }
        }
        if constexpr (GROUPED) {
            // the walk enters a sequence at its last chunk: the state gradient starts from its grad_hT
            if (cur.n == cur.sv.NC - 1) {
                gm_prev = 1.0f;
                set_state(p.dhT, (size_t)cur.bh);
            }
        }
        __syncthreads();

        // ---------------- P^T and dP^T; D'_n ----------------
        // next chunk of the walk: its rows are in flight during everything below (the last one re-reads itself)
        ChunkAt nxt = cur;
        auto request_next = [&]() {
            if (it + 1 < n_iter) nxt = walk_next(cur);
            load_rows_of(nxt, false, ww, lane);
        };
        // (the walk over spans has fewer registers to spare: it asks behind the P blocks)
        if constexpr (!GROUPED) request_next();
        // Eight waves: 0..2 take the P blocks (I,J) = (0,0), (1,0), (1,1), 3..5 the same for dP, 6 and 7 zero
        // the never-computed block (rows j >= 32, columns i < 32) so that every later contraction can run
        // over the full chunk without reading stale data.  Four waves: 0..2 take a block of both, 3 zeroes both.
        auto p_block = [&](bool is_dp, int b) {
            const int I = (b == 0) ? 0 : 1, J = (b == 2) ? 1 : 0;
            f32x16 acc0, acc1;
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc0[v] = 0.0f; acc1[v] = 0.0f; }
            if (is_dp) {
#pragma unroll
                for (int ks = 0; ks < DV / 16; ks += 2) {
                    WM::mma(acc0, WM::load(dOm + (32 * I + r32) * PV + 16 * ks + 8 * g), WM::load(Vm + (32 * J + r32) * PVR + 16 * ks + 8 * g));
                    WM::mma(acc1, WM::load(dOm + (32 * I + r32) * PV + 16 * (ks + 1) + 8 * g), WM::load(Vm + (32 * J + r32) * PVR + 16 * (ks + 1) + 8 * g));
                }
            } else {
#pragma unroll
                for (int ks = 0; ks < DK / 16; ks += 2) {
                    WM::mma(acc0, WM::load_kmajor(QT, PT, 16 * ks, 32 * I, lane), WM::load_kmajor(KT, PT, 16 * ks, 32 * J, lane));
                    WM::mma(acc1, WM::load_kmajor(QT, PT, 16 * (ks + 1), 32 * I, lane), WM::load_kmajor(KT, PT, 16 * (ks + 1), 32 * J, lane));
                }
            }
            // acc[row i][col j]; keep j <= i; stored transposed: dst[j][i .. i+3]
            T* dst = is_dp ? dPt : Pt;
            const int j_glob = 32 * J + r32;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i0 = 32 * I + 8 * c + 4 * g;
                bf16x4 pk;
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) pk[ii] = (T)((j_glob <= i0 + ii) ? acc0[4 * c + ii] + acc1[4 * c + ii] : 0.0f);
                *reinterpret_cast<bf16x4*>(dst + (size_t)j_glob * PC + i0) = pk;
            }
        };
        auto zero_block = [&](T* dst) {      // rows 32..63, columns 0..31: 32 x 32 values, 16 per lane
            const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int k = 0; k < 2; ++k) *reinterpret_cast<u32x4*>(dst + (size_t)(32 + (lane >> 1)) * PC + 16 * (lane & 1) + 8 * k) = zero;
        };
        if constexpr (NW == 4) {
            if (w < 3) { p_block(false, w); p_block(true, w); }
            else { zero_block(Pt); zero_block(dPt); }
        } else {
            if (w < 6) p_block(w >= 3, w >= 3 ? w - 3 : w);
            else zero_block((w == 6) ? Pt : dPt);
        }
        if (has_d) {
            const float gm = tot[ch], c = tot[DK + ch] * gm_prev;
            gm_prev = gm;
#pragma unroll
            for (int j = 0; j < TPW; ++j) {
                const int btj = (w + NW * j) / NAT;
#pragma unroll
                for (int v = 0; v < 16; ++v) accD[j][v] *= c;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = accD[j][8 * half + e];
                    *reinterpret_cast<wfrag*>(dSm + (size_t)ch * PV + 32 * btj + 16 * half + 8 * g) = WM::pack(x);
                }
            }
        }
        if constexpr (GROUPED) request_next();
        if (has_a && it > 0) finish_df(ww, lane, ld_k);
        __syncthreads();

        // ---------------- contractions ----------------
        // dv tile (rt_b, bt): P^T dO over the chunk and K~ D' over the channels
        auto dv_tile = [&]() {
            f32x16 aV;
#pragma unroll
            for (int v = 0; v < 16; ++v) aV[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < C / 16; ++ks)
                WM::mma(aV, WM::load(Pt + (32 * rt_b + r32) * PC + 16 * ks + 8 * g), WM::load_kmajor_swapped(dOm, PV, 16 * ks, 32 * bt, lane));
#pragma unroll
            for (int ks = 0; ks < DK / 16; ++ks)
                WM::mma(aV, WM::load_kmajor(KT, PT, 16 * ks, 32 * rt_b, lane), WM::load_kmajor_swapped(dSm, PV, 16 * ks, 32 * bt, lane));
            const TileStore<FAR> out(chunk_span<FAR>(p.dv, cur.sv.off_v, cr, ld_v, DV, 2), rt_b, 32 * bt, lo, ld_v, lane);
#pragma unroll
            for (int i = 0; i < 8; ++i) out.pair(i, aV[2 * i], aV[2 * i + 1]);
        };
        if (has_b) dv_tile();
        // tile (rt, at):   X = dP K~ + dO (G_m S_n)^T,   Y1 = dP^T Q~,   Ks = V D'^T,   R = rowsum(D' * (G_m S_n))
        f32x16 aX, aY, aKs;
        float R = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) { aX[v] = 0.0f; aY[v] = 0.0f; aKs[v] = 0.0f; }
#pragma unroll
        for (int ks = 0; ks < C / 16; ++ks) {
            const wfrag qf = WM::load(QT + (size_t)ch * PT + 16 * ks + 8 * g);
            if (has_a) {
                WM::mma(aX, WM::load_kmajor(dPt, PC, 16 * ks, 32 * rt, lane), WM::load(KT + (size_t)ch * PT + 16 * ks + 8 * g));
                WM::mma(aY, WM::load(dPt + (32 * rt + r32) * PC + 16 * ks + 8 * g), qf);
            }
            // E_n = D'_n + Q~^T dO: rows = dv (true column order), columns = channels
            if (has_d) {
#pragma unroll
                for (int j = 0; j < TPW; ++j) WM::mma(accD[j], WM::load_kmajor_swapped(dOm, PV, 16 * ks, 32 * ((w + NW * j) / NAT), lane), qf);
            }
        }
        if (has_a) {
#pragma unroll
            for (int kk = 0; kk < 2 * NBT; ++kk) {
                const wfrag d = WM::load(dSm + (size_t)ch * PV + 16 * kk + 8 * g);
                WM::mma(aKs, WM::load(Vm + (32 * rt + r32) * PVR + 16 * kk + 8 * g), d);
                WM::mma(aX, WM::load(dOm + (32 * rt + r32) * PV + 16 * kk + 8 * g), sS[kk]);
                // (R: each row tile takes half of the columns)
                if ((kk >= NBT) == (rt != 0))
#pragma unroll
                for (int e = 0; e < 8; e += 2)
                    R = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{d[e], d[e + 1]}, bf16x2{sS[kk][e], sS[kk][e + 1]}, R, false);
            }
        }
        if constexpr (GROUPED) {
            // the walk leaves a sequence after its first chunk: dS_0 = G_m E is its grad_h0 (formed in
            // place: the next chunk of the walk starts from its own sequence's grad_hT)
            if (cur.n == 0 && p.dh0 && has_d) leave_state(p.dh0, (size_t)cur.bh);
        }

        if constexpr (GATED || DK != DV) __builtin_amdgcn_sched_barrier(0);        // (the end's loads moved up here would not fit: spills)
        // ---------------- element-wise end ----------------
        //   dq = sq X,  dk = sk (Y1 + Ks),  e' = bf16(Q~) X - bf16(K~) Y1,  kk = bf16(K~) Ks
        //   dg_s = sum_{i >= s in chunk} e'_i + sum_{j < s in chunk} kk_j + R
        // (bf16(.) are the values the MFMAs consumed, so that the pair terms inside e' cancel to fp32 accuracy)
        if (has_a) {
            float a[16], z[16], gs[16], dk[16], te[4], tk[4];
            const TileStore<FAR> out(chunk_span<FAR>(p.dq, cur.sv.off_k, cr, ld_k, DK, 2), rt, 32 * at, lo, ld_k, lane);
            if constexpr (GATED) {
                const f32x4 xa = stash[64 * w + lane], xz = stash[NT + 64 * w + lane];
#pragma unroll
                for (int c = 0; c < 4; ++c) { sa[c] = xa[c]; sz[c] = xz[c]; }
            }
            group_products(a, z, f);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bf16x4 qb = *reinterpret_cast<const bf16x4*>(q_corner + (size_t)r32 * PT + 8 * c + 4 * g);
                const bf16x4 kb = *reinterpret_cast<const bf16x4*>(k_corner + (size_t)r32 * PT + 8 * c + 4 * g);
                float se = 0.0f, pk = 0.0f;
#pragma unroll
                for (int j = 3; j >= 0; --j) {                     // inclusive suffix inside the group
                    const int i = 4 * c + j;
                    se = fmaf((float)qb[j], aX[i], se);
                    se = fmaf(-(float)kb[j], aY[i], se);
                    gs[i] = se;
                    dk[i] = (sz[c] * z[i]) * (aY[i] + aKs[i]);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {                      // exclusive prefix inside the group
                    const int i = 4 * c + j;
                    gs[i] += pk;
                    pk = fmaf((float)kb[j], aKs[i], pk);
                }
                te[c] = se; tk[c] = pk;
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    const int i = 4 * c + j;
                    out.pair(i / 2, (sa[c] * a[i]) * aX[i], (sa[c] * a[i + 1]) * aX[i + 1]);
                }
            }
            // groups after this one (sum of e'), groups before it (sum of K~ Ks), inside the tile; the tile's totals for the other one
            const f32x2 r2 = both_halves(R);
            float add[4], after = 0.0f, before = 0.0f;
            f32x2 e2[4], k2[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) { e2[c] = both_halves(te[c]); k2[c] = both_halves(tk[c]); }
#pragma unroll
            for (int c = 3; c >= 0; --c) {
                add[c] = after + (g ? 0.0f : e2[c].y);
                after += e2[c].x + e2[c].y;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                add[c] += before + (g ? k2[c].x : 0.0f);
                before += k2[c].x + k2[c].y;
            }
            const float Rs = r2.x + r2.y;
            if (g == 0) ex[rt * DK + ch] = Rs + (rt ? after : before);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                df_r[i] = fast_rcp(f[i] + 1e-30f);
                df_u[i] = fmaf(gs[i] + (add[i >> 2] + Rs), df_r[i], -dk[i]);
            }
            if constexpr (GATED) {
                // gate formed from its pre-activation z (paper Eq. 2): with g = sigmoid(z) = (f - beta)/(1 - beta),
                //   dL/dz = df (1 - beta) g (1 - g) = df (f - beta)(1 - f)/(1 - beta),   dL/dbeta = sum df (1 - g)
                // (rows past the end of the sequence have f = 1 and drop out of the sum by themselves)
                const float inv = fast_rcp(1.0f - beta);
                beta_u = 0.0f; beta_r = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float h = (1.0f - f[i]) * inv, u = df_u[i] * h, r = df_r[i] * h;
                    beta_u += u; beta_r += r;
                    df_u[i] = u * (f[i] - beta);
                    df_r[i] = r * (f[i] - beta);
                }
            }
            df_dst = chunk_span<FAR>(p.df, cur.sv.off_k, cr, ld_k, DK, 2);
            df_lo = lo;
        }
        __syncthreads(); // every wave is done with the tiles
        cur = nxt;
    }
    if (has_a) finish_df(ww, lane_id(), (int)p.lay.sn_k);
    if (p.flag && below_floor < kTinyProduct) *p.flag = 1;
    store_run_beta();
    if constexpr (!GROUPED) {
        // run 0 ends at the start of the sequence: dS_0 = G_m E of its first chunk is grad_h0
        if (f_run == 0 && p.dh0 && has_d) leave_state(p.dh0, (size_t)f_bh);
    }
}

template <int DK, int DV, bool GATE_BF16, bool GATED, bool FAR = false>
__global__ __launch_bounds__(64 * walk_waves(DK, DV), 2) void bwd_walk_kernel(BwdGradParams p)
{
    walk_body<DK, DV, GATE_BF16, GATED, false, FAR>(p);
}

// The walk over spans of a packed batch (a kernel of its own).
template <int DK, int DV, bool GATE_BF16, bool GATED, bool FAR = false>
__global__ __launch_bounds__(64 * walk_waves(DK, DV), 2) void bwd_walk_grouped_kernel(BwdGradParams p)
{
    walk_body<DK, DV, GATE_BF16, GATED, true, FAR>(p);
}

template <int DK, int DV, bool GATED>
static hipError_t launch_walk_one(const SeqDims& d, const BwdGradParams& p, bool grouped, hipStream_t stream)
{
    typedef WalkLds<DK, DV> L;
    const bool bf = d.gate_bf16;
    auto kern = grouped ? (bf ? bwd_walk_grouped_kernel<DK, DV, true, GATED> : bwd_walk_grouped_kernel<DK, DV, false, GATED>)
                        : (bf ? bwd_walk_kernel<DK, DV, true, GATED> : bwd_walk_kernel<DK, DV, false, GATED>);
    if (!walk_rows_near(d.lay.sn_k, d.lay.sn_v, bf ? 2 : 4)) {
        if (grouped ? d.lay.spans != 1 : p.R != 1) return hipErrorInvalidValue;
        kern = grouped ? (bf ? bwd_walk_grouped_kernel<DK, DV, true, GATED, true> : bwd_walk_grouped_kernel<DK, DV, false, GATED, true>)
                       : (bf ? bwd_walk_kernel<DK, DV, true, GATED, true> : bwd_walk_kernel<DK, DV, false, GATED, true>);
    }
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)L::total);
    if (e != hipSuccess) return e;
    const unsigned grid = grouped ? (unsigned)(d.lay.spans * d.lay.H) : (unsigned)(d.BH * p.R);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * walk_waves(DK, DV)), L::total, stream, p);
    return hipGetLastError();
}

template <bool GATED>
static hipError_t launch_walk(const SeqDims& d, const BwdGradParams& p, bool grouped, hipStream_t stream)
{
    if (d.dk == 128 && d.dv == 128) return launch_walk_one<128, 128, GATED>(d, p, grouped, stream);
    if (d.dk == 64 && d.dv == 64) return launch_walk_one<64, 64, GATED>(d, p, grouped, stream);
    if (d.dk == 128 && d.dv == 64) return launch_walk_one<128, 64, GATED>(d, p, grouped, stream);
    if (d.dk == 64 && d.dv == 128) return launch_walk_one<64, 128, GATED>(d, p, grouped, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_bwd_walk(const SeqDims& d, const BwdGradParams& p, bool grouped, hipStream_t stream)
{
    return p.beta ? launch_walk<true>(d, p, grouped, stream) : launch_walk<false>(d, p, grouped, stream);
}

// ---- the light walk alone ---------------------------------------------------------------------------------------------
// What a run of chunks adds to the state gradient from zero, and the product of its
// gates: for every run of segmented sequences, or for every span of a packed batch whose first sequence has
// begun in an earlier span, over that sequence's chunks in the span.
template <int DK, int DV, bool GATE_BF16, bool GATED, bool GROUPED>
__device__ __forceinline__ void ends_body(const BwdGradParams& p)
{
    typedef WalkLds<DK, DV> L;
    constexpr int NW = walk_waves(DK, DV), NAT = DK / 32, NBT = DV / 32, NDT = NAT * NBT, TPW = (NDT + NW - 1) / NW;
    extern __shared__ __align__(16) char smem[];
    if (not_chosen(p.lay)) return;
    const int tid = threadIdx.x, slot = blockIdx.x;
    const WalkWave ww = walk_wave<NAT, NW>(__builtin_amdgcn_readfirstlane(tid >> 6));
    ChunkAt cur;
    int count;
    if constexpr (GROUPED) {
        const int span = slot / p.lay.H, head = slot - span * p.lay.H;
        if (span >= p.lay.spans || table_read(p.lay.span_walks, 1) == 0) return;
        const int* before = p.lay.vl + 2 * (p.lay.B + 1);
        const int total = table_read(before, p.lay.B);
        const int p0 = (int)((long long)span * total / p.lay.spans), p1 = (int)((long long)(span + 1) * total / p.lay.spans);
        if (span == 0 || p1 <= p0) return;
        // the sequence that holds chunk p0 is the one the span before ends in, unless it starts here
        const int e = min(max(table_read(p.lay.span_seq, span - 1), 0), p.lay.B - 1);
        const int b0 = table_read(before, e), b1 = min(table_read(before, e + 1), p1);
        if (b0 >= p0 || b1 <= p0) return;
        cur.bh = e * p.lay.H + head;
        cur.sv = seq_view<false, DK, DV>(p.lay, p.N, p.NC, cur.bh);
        cur.n = b1 - 1 - b0;
        count = b1 - p0;
    } else {
        if (slot >= p.BH) return;
        cur.bh = slot;
        cur.sv = seq_view<false, DK, DV, true>(p.lay, p.N, p.NC, slot);
        count = cur.sv.NC;
        cur.n = count - 1;
        if (count <= 0) return;
    }
    f32x16 accD[TPW];
#pragma unroll
    for (int j = 0; j < TPW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) accD[j][v] = 0.0f;
    RawGate<GATE_BF16> raw_f;
    u32x4 raw_q[2];
    Raw16<__bf16> raw_d;
    light_walk<DK, DV, GATE_BF16, GATED, NW, 1>(p, reinterpret_cast<__bf16*>(smem + L::lq), 0, reinterpret_cast<__bf16*>(smem + L::ld), 0,
                                                reinterpret_cast<float*>(smem + L::lt), cur, count, accD, p.span_decay + (size_t)slot * DK,
                                                raw_f, raw_q, raw_d, ww);
    if (NDT % NW == 0 || ww.w < NDT) {
        float* out = p.span_add + (size_t)slot * DK * DV + (size_t)(32 * ww.at + (tid & 31)) * DV + 4 * ((tid >> 5) & 1);
#pragma unroll
        for (int j = 0; j < TPW; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                *reinterpret_cast<f32x4*>(out + 32 * ((ww.w + NW * j) / NAT) + 8 * c) =
                    f32x4{accD[j][4 * c], accD[j][4 * c + 1], accD[j][4 * c + 2], accD[j][4 * c + 3]};
    }
}

// Two workgroups of eight waves to a compute unit (heads of 64: three of four).
template <int DK, int DV, bool GATE_BF16, bool GATED>
__global__ __launch_bounds__(64 * walk_waves(DK, DV), walk_waves(DK, DV) == 8 ? 4 : 3) void bwd_ends_kernel(BwdGradParams p)
{
    if (p.lay.vl && p.lay.spans > 0) ends_body<DK, DV, GATE_BF16, GATED, true>(p);
    else ends_body<DK, DV, GATE_BF16, GATED, false>(p);
}

template <int DK, int DV, bool GATED>
static hipError_t launch_ends_one(const SeqDims& d, const BwdGradParams& p, unsigned grid, hipStream_t stream)
{
    typedef WalkLds<DK, DV> L;
    auto kern = d.gate_bf16 ? bwd_ends_kernel<DK, DV, true, GATED> : bwd_ends_kernel<DK, DV, false, GATED>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)L::light_total);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * walk_waves(DK, DV)), L::light_total, stream, p);
    return hipGetLastError();
}

template <bool GATED>
static hipError_t launch_ends(const SeqDims& d, const BwdGradParams& p, unsigned grid, hipStream_t stream)
{
    if (d.dk == 128 && d.dv == 128) return launch_ends_one<128, 128, GATED>(d, p, grid, stream);
    if (d.dk == 64 && d.dv == 64) return launch_ends_one<64, 64, GATED>(d, p, grid, stream);
    if (d.dk == 128 && d.dv == 64) return launch_ends_one<128, 64, GATED>(d, p, grid, stream);
    if (d.dk == 64 && d.dv == 128) return launch_ends_one<64, 128, GATED>(d, p, grid, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_walk_ends(const SeqDims& d, const BwdGradParams& p, unsigned grid, hipStream_t stream)
{
    return p.beta ? launch_ends<true>(d, p, grid, stream) : launch_ends<false>(d, p, grid, stream);
}

}   // namespace hgrn2
