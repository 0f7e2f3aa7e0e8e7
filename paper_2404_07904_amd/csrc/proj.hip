// Input side of the HGRU2 token mixer (paper Section 2, Eq. 1): the three projections of the layer
// input and their activations,
//
//     z = U x + b_u   (pre-activation of the forget gate; Eq. 2 turns sigmoid(z) into f inside
//                      the recurrence kernels),
//     v = SiLU(V x + b_v)   (the paper's input vector i),
//     q = sigmoid(W x + b_w)   (the paper's output gate o),
//
// as ONE bf16 matrix product [M, d] x [d, 3d] on the matrix cores with bias and activation applied
// to the fp32 accumulators, written token-major ([B][N][H][dh] = [M][d]), which is the layout the
// recurrence takes with HGRN2_LAYOUT_BNHD: neither the pre-activations of q nor the gate ever
// reach memory.  The reverse mode is two more products, dx = dA W3 and dW3 = dA^T x, after one element-wise pass that
// forms dA = (dz, dv SiLU'(a_v), dq q (1 - q)) and the bias gradients.
//
// One matrix kernel (gemm_nt_kernel) for all three: both operands with the contraction index contiguous, which x W3^T has as it
// is; W3 and x are transposed first, and the element-wise pass writes dA in both orders (dW3 straight from dA and x,
// with LDS transpose reads, took 516 us at 16384 tokens and width 2048, this way 324 + 50).
#include "../../include/hgrn2.h"
#include "common.hpp"
#include "kernels.hpp"
#include "proj_plan.hpp"
#include <type_traits>

namespace hgrn2 {

constexpr int kUnits = 256;      // compute units: workgroups that walk tiles
constexpr int kBandRows = 4;     // row blocks per band of the workgroup -> tile order

enum GemmEpilogue { kEpiProj = 0, kEpiPlain = 1, kEpiFloat = 2 };

struct GemmParams {
    const __bf16* A;      // [M][K], row stride lda
    const __bf16* B;      // [N][K], row stride ldb
    long long lda, ldb;
    int M, N, K;          // K a multiple of 64, N of the tile width
    // outputs
    __bf16* C;            // kEpiPlain: [M][N] bf16, row stride ldc
    float* Cf;            // kEpiFloat: [splits][M][N] fp32, row stride ldc: the splits' shares of the contraction
    long long ldc;
    // kEpiProj: N = 3 d; columns [0, d) -> z, [d, 2d) -> v (and a_v), [2d, 3d) -> q, each [M][d]
    const float* bias;
    __bf16 *z, *v, *q, *av;
    int d;
};

// s_waitcnt: all but the youngest n vector loads have landed, and all LDS reads
constexpr int vm_lgkm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

// ---- the products: C = A B^T, both operands k-contiguous ------------------------------------------------------------
// A workgroup computes a TM x TN tile, WM x WN waves side by side (KG groups of them share the steps' four k-quarters between
// them and add up at the end: small tiles of long contractions).  K advances in steps of 64, whole 128-byte lines of every row,
// through a ring of NS tiles in LDS (A and B in turn) that `global_load_lds` fills, 16 bytes per lane, no registers in
// between.  Such a load writes the 64 lanes' vectors to consecutive LDS addresses, so a tile row is 128 bytes with no padding; the
// 16-byte piece c of row r is kept at position c ^ ((r >> 1) & 7), which the loading lane realises by fetching the piece that
// belongs at its position, and 16 consecutive rows then cover all 64 banks for any piece.
//   One barrier per step, before its last quarter: by then every wave has the last fragments of the step in registers, so the
// barrier retires the step's two tiles, which are refilled, and publishes those of the next step (each wave has waited for its
// own loads of them; loads are counted by hand, the compiler does not track them).  With NS = 5 the tile of A is requested 1 3/4 steps
// ahead, that of B 3/4.  Fragments are requested right after the first MFMAs of the quarter before (the compiler waits for
// all outstanding LDS reads before an MFMA that needs one), and the refill goes out one load at a time between the MFMAs.
//   16384 x 2048 x 6144 with bias, activations and four outputs: 342-359 us = 1.15-1.20 PFLOP/s (an earlier kernel with steps of 32, half
// lines, 372-400); dx 315 us = 1.31 PFLOP/s (369), dW3 324 (516).  What bounds the 256 x 256 tile (builds that leave work out): 217 us are MFMAs and LDS reads
// (1.9 PFLOP/s), 85 us the loads' way into LDS next to 192 KB of LDS reads a step (loads that never miss L2 save 14 us, no wait for them nothing), 38 us
// the epilogue.  Four waves of 128 x 128, with a third fewer LDS reads but one wave per SIMD: 365 us.
//   A workgroup of the projections' 256 x 256 tile has a compute unit to itself and walks several tiles (WALK): the ring goes on across their boundary,
// the loads of the next tile's first steps go out in the last ones of this, and nothing starts or drains in between.
// Rows leave through the slot that is free at that moment, each wave by itself, as whole lines (stored from the accumulators in
// pieces of 32 bytes, the write path takes 45 us more).  16384 x 2048 x 6144: 377 -> 359 us, 8192 rows 191 -> 176, 16384 x 1024 x 3072
// 109 -> 99, 4100 x 2048 x 6144 110.5 -> 108.  dx has three times the steps to a tile and half of the outputs, and gains nothing (8192 rows 426 -> 429 us
// for the whole reverse mode), so it keeps one tile to a workgroup.
constexpr bool nt_walks(int epi, int tm) { return epi == kEpiProj && tm == 256; }

// A wave's 32 NI x 64 part of a tile, from its accumulators to memory: acc[i][j][v] = C[row0 + 32 i + lane % 32][32 j + 8 (v / 4) + 4 (lane / 32) + v % 4],
// `part`: of the tile's 256 columns.  Rows before m_new are another tile's.  Every store is issued by every lane (rows that are not
// stored lie outside the buffer), 4 NI per output: the walk counts them.  `stage`: 4 KB of LDS of the wave's own.
template <int NI, int NJ>
__device__ __forceinline__ void store_tile(const GemmParams& p, const f32x16 (&acc)[NI][NJ], int row0, int m_new, int col, char* stage)
{
    static_assert(NJ == 2, "a row of the wave's part is one line of 128 bytes");
    const int lane = (int)threadIdx.x & 63, r32 = lane & 31, g = lane >> 5;
    const int which = col / p.d;
    const uint32_t pitch = (uint32_t)p.d * 2u;
    const int from = max(row0, m_new), rows = max(min(row0 + 32 * NI, p.M) - from, 0);
    // (of the row that is the buffer's first: rows before it wrap around to offsets past its end)
    const uint32_t at = (uint32_t)(row0 - from + (lane >> 3)) * pitch + 16u * (lane & 7);
    auto buffer = [&](__bf16* out) {
        return __builtin_amdgcn_make_buffer_rsrc(out + (size_t)from * (pitch / 2) + (col - which * p.d), 0, (int)((uint32_t)rows * pitch), 0x00020000);
    };
    // the 16-byte piece c of row r lies at c ^ ((r >> 1) & 7), as in the ring
    auto put = [&](const u32x4& u, int piece) {
        // the halves of the wave trade four columns for four: lanes 0 .. 31 get columns 8 piece .., the others 8 (piece + 1) ..
        const auto x = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
        *reinterpret_cast<u32x4*>(stage + r32 * 128 + (((piece + g) ^ ((r32 >> 1) & 7)) << 4)) = u32x4{x[0], y[0], x[1], y[1]};
    };
    // MODE 0: the sum itself; 1: SiLU of it; 2: sigmoid of it
    auto store = [&](auto MODE, const auto& to, int i) {
        constexpr int md = decltype(MODE)::value;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int c = 0; c < 4; c += 2) {
                union { __bf16 e[8]; u32x4 u; } y;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float a = acc[i][j][4 * c + e];
                    const float sg = md == 0 ? 0.0f : fast_rcp(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * a));
                    y.e[e] = (__bf16)(md == 0 ? a : md == 1 ? a * sg : sg);
                }
                put(y.u, 4 * j + c);
            }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int r = 8 * k + (lane >> 3);
            const u32x4 u = *reinterpret_cast<const u32x4*>(stage + r * 128 + (((lane & 7) ^ ((r >> 1) & 7)) << 4));
            __builtin_amdgcn_raw_buffer_store_b128(u, to, at + (uint32_t)(32 * i + 8 * k) * pitch, 0, 0);
        }
    };
    typedef std::integral_constant<int, 0> Plain;
    typedef std::integral_constant<int, 1> Silu;
    typedef std::integral_constant<int, 2> Sigmoid;
    if (which == 0) {
        const auto to = buffer(p.z);
#pragma unroll
        for (int i = 0; i < NI; ++i) store(Plain(), to, i);
    } else if (which == 1) {
        const auto to = buffer(p.v), to_av = buffer(p.av);
#pragma unroll
        for (int i = 0; i < NI; ++i) { store(Silu(), to, i); if (p.av) store(Plain(), to_av, i); }
    } else {
        const auto to = buffer(p.q);
#pragma unroll
        for (int i = 0; i < NI; ++i) store(Sigmoid(), to, i);
    }
}

template <int EPI, int TM, int TN, int WM, int WN, int KG, int NS>
__global__ __launch_bounds__(64 * WM * WN * KG, 2) void gemm_nt_kernel(GemmParams p)
{
    constexpr int NWV = WM * WN * KG, THREADS = 64 * NWV;
    static_assert(NWV == 8 && 4 % KG == 0 && NS >= 5 && NS % 2 == 1, "eight waves, a ring of whole steps and one tile");
    constexpr int SLOT = (TM > TN ? TM : TN) * 128;               // bytes of a slot of the ring
    constexpr int LA = TM / 8 / NWV, LB = TN / 8 / NWV;           // load instructions per wave for a tile of A, of B
    constexpr int NI = TM / WM / 32, NJ = TN / WN / 32, KPW = 4 / KG;
    constexpr bool WALK = nt_walks(EPI, TM);
    typedef Mma<__bf16> M;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    typedef const __attribute__((address_space(1))) void* global_ptr;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = w % WN, wm = w / WN % WM, kg = w / (WN * WM);
    const int n_bn = p.N / TN, n_bm = (p.M + TM - 1) / TM;
    // The tiles of an XCD lie together; its workgroups take them in turn, every `stride`-th (WALK), or one each.
    int t, t_end, stride;
    {
        const int tiles = n_bm * n_bn, grid = (int)gridDim.x, id = (int)blockIdx.x;
        const int per = tiles / kXcds, rem = tiles - per * kXcds, x = id % kXcds, from = x * per + min(x, rem);
        t = from + id / kXcds;
        t_end = from + per + (x < rem ? 1 : 0);
        stride = (grid + kXcds - 1 - x) / kXcds;
    }
    // Tile t: rows m0 .. of A and columns n0 .. of C.  WALK: the last tile of a column reaches back into the rows of the one before
    // (which it does not store again: m_new), so that all tiles are whole unless A is shorter than one, and a wave's offsets stay what they
    // are from tile to tile.  Others clamp: a row read over and over costs less than as many new ones (100 rows of width 3072, two
    // tiles of 64: 23.4 us reaching back, 22.2).
    struct Tile { int m0, m_new, n0; };
    auto tile_at = [&](int at) {
        const int band_tiles = kBandRows * n_bn, band = at / band_tiles, in_band = at - band * band_tiles;
        const int rows = min(kBandRows, n_bm - band * kBandRows), bn = in_band / rows;
        const int m = (band * kBandRows + in_band - bn * rows) * TM;
        return Tile{WALK ? max(min(m, p.M - TM), 0) : m, m, bn * TN};
    };
    Tile tile = tile_at(t);
    f32x16 acc[NI][NJ];
    // What the sums start from: zero, or (WALK) the biases of their columns.  These are scalar loads, a half wave's each, and kept apart from the
    // choice between them: folded into a vector load at a chosen address, they would wait for the ring's loads and the stores.
    auto scalar = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
    auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float b = 0.0f;
                    if constexpr (WALK) {
                        typedef const __attribute__((address_space(4))) float* scalar_ptr;
                        const scalar_ptr s = (scalar_ptr)(p.bias + tile.n0 + (TN / WN) * wn + 32 * j + 8 * c);
                        const float lo = scalar(s[e]), hi = scalar(s[4 + e]);
                        b = g ? hi : lo;
                    }
#pragma unroll
                    for (int i = 0; i < NI; ++i) acc[i][j][4 * c + e] = b;
                }
    };
    clear();
    // Load instruction j of a wave: eight rows, of A from row a0(j) on.  A row of dW3's operands is 2 bytes per token and may be long, so
    // the rows before are part of the scalar address; rows past the end of A re-read its last one (never stored).
    const int left = p.M - (WALK ? 0 : tile.m0);
    const bool whole = left >= TM;
    auto a_of = [&](const Tile& at) { return reinterpret_cast<const char*>(p.A) + (size_t)at.m0 * p.lda * 2; };
    auto b_of = [&](const Tile& at) { return reinterpret_cast<const char*>(p.B) + (size_t)at.n0 * p.ldb * 2; };
    const char *abase = a_of(tile), *bbase = b_of(tile), *anext = abase, *bnext = bbase;
    auto a0 = [&](int j) { return whole ? 8 * (LA * w + j) : 0; };
    uint32_t ao[LA], bo[LB];
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const int row = 8 * (LA * w + j) + (lane >> 3);
        ao[j] = (uint32_t)(min(row, left - 1) - a0(j)) * (uint32_t)(p.lda * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
        const int row = 8 * (LB * w + j) + (lane >> 3);
        bo[j] = (uint32_t)(lane >> 3) * (uint32_t)(p.ldb * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    // the steps of 64 of this workgroup's share of the contraction
    const int steps = p.K / 64, first = (int)((long long)blockIdx.y * steps / gridDim.y);
    const int nk = (int)((long long)(blockIdx.y + 1) * steps / gridDim.y) - first;
    // load instruction j of this wave for the A (B) tile of k-step ks into `slot`; steps past the last one are the next tile's (K has
    // four steps and more there), or the last one once more
    auto step_of = [&](const char* base, const char* next, int ks) {
        if constexpr (WALK) return ks < nk ? base + (size_t)ks * 128 : next + (size_t)(ks - nk) * 128;
        else return base + (size_t)(first + min(ks, nk - 1)) * 128;
    };
    auto load_a = [&](int slot, int ks, int j) {
        const char* s = step_of(abase, anext, ks) + (size_t)a0(j) * p.lda * 2;
        __builtin_amdgcn_global_load_lds((global_ptr)(s + ao[j]), (lds_ptr)(smem + slot * SLOT + 8 * (LA * w + j) * 128), 16, 0, 0);
    };
    auto load_b = [&](int slot, int ks, int j) {
        const char* s = step_of(bbase, bnext, ks) + (size_t)(8 * (LB * w + j)) * p.ldb * 2;
        __builtin_amdgcn_global_load_lds((global_ptr)(s + bo[j]), (lds_ptr)(smem + slot * SLOT + 8 * (LB * w + j) * 128), 16, 0, 0);
    };
    const int sw = (r32 >> 1) & 7;
    auto read_frags = [&](bf16x8 (&fa)[NI], bf16x8 (&fb)[NJ], int sa, int sb, int kk) {
        const int off = r32 * 128 + (((2 * kk + g) ^ sw) << 4);
        const char* a = smem + sa * SLOT + (TM / WM) * wm * 128 + off;
        const char* b = smem + sb * SLOT + (TN / WN) * wn * 128 + off;
#pragma unroll
        for (int j = 0; j < NJ; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(b + 32 * j * 128);
#pragma unroll
        for (int i = 0; i < NI; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(a + 32 * i * 128);
    };
    constexpr int NM = NI * NJ, HEAD = NM > 2 ? 2 : 1;
    bf16x8 fa[2][NI], fb[2][NJ];
    auto multiply = [&](int par, int from, int to) {
#pragma unroll
        for (int t = 0; t < NM; ++t)
            if (t >= from && t < to) M::mma(acc[t / NJ][t % NJ], fb[par][t % NJ], fa[par][t / NJ]);
    };
    // tiles 0 .. NS - 2 (A of step 0, B of step 0, A of step 1, ...); the first two have to be there
#pragma unroll
    for (int h = 0; h < NS - 1; ++h)
#pragma unroll
        for (int j = 0; j < ((h & 1) ? LB : LA); ++j) { if (h & 1) load_b(h, h >> 1, j); else load_a(h, h >> 1, j); }
    __builtin_amdgcn_s_waitcnt(vm_lgkm((NS - 3) / 2 * (LA + LB)));
    __builtin_amdgcn_s_barrier();
    auto wrap = [](int s) { return s >= NS ? s - NS : s; };
    int s0 = 0;                                   // slot of A of the step, B behind it
    read_frags(fa[0], fb[0], 0, 1, KPW * kg);
    // the loads that refill the two slots a step has freed: tile 2 k + NS (of B), then 2 k + NS + 1 (of A; steps taken as half of a
    // tile's number: written as sums, the scalar addresses cost small products 0.2 us)
    auto refill = [&](int slot, int k, int j) {   // j = 0 .. LB + LA - 1
        const int sl = j < LB ? slot : wrap(slot + 1), h = NS + (j < LB ? 0 : 1);
        if (h & 1) load_b(sl, k + (h >> 1), j < LB ? j : j - LB); else load_a(sl, k + (h >> 1), j < LB ? j : j - LB);
    };
    // a step: phases 0 .. KPW - 1; of the loads behind the barrier of step k, B's go out in its last phase and A's in the first phase of the next
    constexpr int NL = LB + LA, LAST = LB;
    int stores = 0;          // stores that went out behind the loads of this tile's first two steps
    for (;;) {
    Tile next = tile;
    if constexpr (WALK) {
        if (t + stride < t_end) next = tile_at(t + stride);
        anext = a_of(next); bnext = b_of(next);
    }
    for (int k = 0; k < nk; ++k) {
        const int sn = wrap(s0 + 2), sp = wrap(s0 + NS - 2);       // slots of the next and of the previous step
#pragma unroll
        for (int ph = 0; ph < KPW; ++ph) {
            const int par = KPW == 1 ? 0 : (ph & 1), nx = KPW == 1 ? 1 : par ^ 1;
            const bool last = ph == KPW - 1;
            if (last) {
                __builtin_amdgcn_sched_barrier(0);
                if (KPW == 1) {
#pragma unroll
                    for (int j = LAST; j < NL; ++j) refill(sp, k - 1, j);
                }
                // (the stores of the tile before are younger than what a tile's first step waits for)
                constexpr int NEW = (NS - 5) / 2 * (LA + LB) + LA;
                if (WALK && k == 0 && stores == 8 * NI) __builtin_amdgcn_s_waitcnt(vm_lgkm(NEW + 8 * NI));
                else if (WALK && k == 0 && stores == 4 * NI) __builtin_amdgcn_s_waitcnt(vm_lgkm(NEW + 4 * NI));
                else __builtin_amdgcn_s_waitcnt(vm_lgkm(NEW));
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
            }
            multiply(par, 0, HEAD);
            __builtin_amdgcn_sched_barrier(0);
            if (last) read_frags(fa[nx], fb[nx], sn, wrap(sn + 1), KPW * kg);
            else read_frags(fa[nx], fb[nx], s0, wrap(s0 + 1), KPW * kg + ph + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (last) {
#pragma unroll
                for (int j = 0; j < LAST; ++j) {
                    multiply(par, HEAD + (NM - HEAD) * j / LAST, HEAD + (NM - HEAD) * (j + 1) / LAST);
                    __builtin_amdgcn_sched_barrier(0);
                    refill(s0, k, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if (ph == 0) {
                constexpr int REST = NL - LAST;
#pragma unroll
                for (int j = 0; j < REST; ++j) {
                    multiply(par, HEAD + (NM - HEAD) * j / REST, HEAD + (NM - HEAD) * (j + 1) / REST);
                    __builtin_amdgcn_sched_barrier(0);
                    refill(sp, k - 1, LAST + j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                multiply(par, HEAD, NM);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (KPW == 1) {
#pragma unroll
            for (int i = 0; i < NI; ++i) fa[0][i] = fa[1][i];
#pragma unroll
            for (int j = 0; j < NJ; ++j) fb[0][j] = fb[1][j];
        }
        s0 = sn;
    }
    if constexpr (WALK) {
        char* stage = smem + wrap(s0 + NS - 1) * SLOT + 8 * LA * w * 128;        // (where this wave's next loads of A go)
        store_tile<NI, NJ>(p, acc, tile.m0 + (TM / WM) * wm, tile.m_new, tile.n0 + (TN / WN) * wn, stage);
        stores = 4 * NI * (tile.n0 / p.d == 1 && p.av ? 2 : 1);
        t += stride;
        if (t >= t_end) break;
        tile = next; abase = anext; bbase = bnext;
        clear();
    } else break;
    }
    __builtin_amdgcn_s_waitcnt(vm_lgkm(0));
    if constexpr (WALK) return;
    __builtin_amdgcn_s_barrier();
    const int m0 = tile.m0, n0 = tile.n0;

    // the groups' shares of the sum, added in order
    if constexpr (KG > 1) {
        float* red = reinterpret_cast<float*>(smem);
        constexpr int TILE = NI * NJ * 16 * 64;
        if (kg > 0) {
            float* d = red + (size_t)((kg - 1) * WM * WN + w % (WM * WN)) * TILE + lane * 4;
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        *reinterpret_cast<f32x4*>(d + ((i * NJ + j) * 4 + c) * 256) = f32x4{acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int k = 0; k < KG - 1; ++k) {
                const float* d = red + (size_t)(k * WM * WN + w) * TILE + lane * 4;
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const f32x4 t = *reinterpret_cast<const f32x4*>(d + ((i * NJ + j) * 4 + c) * 256);
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[i][j][4 * c + e] += t[e];
                        }
            }
        }
    }
    // acc[i][j][v] = C[m0 + (TM / WM) wm + 32 i + lane % 32][n0 + (TN / WN) wn + 32 j + 8 (v/4) + 4 g + v%4]
    if constexpr (EPI == kEpiFloat) {
        if (kg == 0) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int row = m0 + (TM / WM) * wm + 32 * i + r32;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (row < p.M)
                            *reinterpret_cast<f32x4*>(p.Cf + ((size_t)blockIdx.y * p.M + row) * p.ldc + n0 + (TN / WN) * wn + 32 * j + 8 * c + 4 * g) =
                                f32x4{acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
            }
        }
    } else {
        constexpr int PS = TN + 8, VPR = TN / 8;
        __bf16* St = reinterpret_cast<__bf16*>(smem + (KG > 1 ? (KG - 1) * TM * TN * 4 : 0));
        int which = 0;
        if constexpr (EPI == kEpiProj) which = n0 / p.d;
        const int n_pass = (EPI == kEpiProj && which == 1 && p.av != nullptr) ? 2 : 1;
        for (int pass = 0; pass < n_pass; ++pass) {
            // 0: the sum itself (plus bias in the projections); 1: SiLU; 2: sigmoid
            const int mode = (EPI != kEpiProj || pass == 1 || which == 0) ? 0 : which;
            auto stage_tile = [&](auto MODE) {
                constexpr int md = decltype(MODE)::value;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int col = (TN / WN) * wn + 32 * j + 8 * c + 4 * g;
                        f32x4 b = {0.0f, 0.0f, 0.0f, 0.0f};
                        if constexpr (EPI == kEpiProj) b = *reinterpret_cast<const f32x4*>(p.bias + n0 + col);
#pragma unroll
                        for (int i = 0; i < NI; ++i) {
                            const int row = (TM / WM) * wm + 32 * i + r32;
                            bf16x4 pk;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float a = acc[i][j][4 * c + e] + b[e];
                                float y = a;
                                if constexpr (md != 0) {
                                    const float sg = fast_rcp(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * a));
                                    y = (md == 1) ? a * sg : sg;
                                }
                                pk[e] = (__bf16)y;
                            }
                            *reinterpret_cast<bf16x4*>(St + (size_t)row * PS + col) = pk;
                        }
                    }
            };
            if (kg == 0) {
                if (mode == 0)      stage_tile(std::integral_constant<int, 0>());
                else if (mode == 1) stage_tile(std::integral_constant<int, 1>());
                else                stage_tile(std::integral_constant<int, 2>());
            }
            __syncthreads();
            __bf16* out;
            long long ld;
            int c0;
            if constexpr (EPI == kEpiProj) {
                out = (pass == 1) ? p.av : (which == 0) ? p.z : (which == 1) ? p.v : p.q;
                ld = p.d;
                c0 = n0 - which * p.d;
            } else {
                out = p.C; ld = p.ldc; c0 = n0;
            }
            constexpr int VECS = TM * VPR / THREADS, BATCH = VECS < 8 ? VECS : 8;
#pragma unroll
            for (int v0 = 0; v0 < VECS; v0 += BATCH) {
                u32x4 buf[BATCH];
#pragma unroll
                for (int k = 0; k < BATCH; ++k) {
                    const int vi = tid + (v0 + k) * THREADS;
                    buf[k] = *reinterpret_cast<const u32x4*>(St + (size_t)(vi / VPR) * PS + (vi % VPR) * 8);
                }
#pragma unroll
                for (int k = 0; k < BATCH; ++k) {
                    const int vi = tid + (v0 + k) * THREADS, row = vi / VPR;
                    if (m0 + row < p.M) *reinterpret_cast<u32x4*>(out + (size_t)(m0 + row) * ld + c0 + (vi % VPR) * 8) = buf[k];
                }
            }
            __syncthreads();
        }
    }
}

template <int EPI, int TM, int TN, int WM, int WN, int KG, int NS>
static hipError_t launch_nt(const GemmParams& p, int splits, hipStream_t stream)
{
    constexpr size_t ring = (size_t)NS * (TM > TN ? TM : TN) * 128;
    constexpr bool walk = nt_walks(EPI, TM);
    constexpr size_t tail = (size_t)(KG - 1) * TM * TN * 4 + (EPI == kEpiFloat || walk ? 0 : (size_t)TM * (TN + 8) * 2);
    constexpr size_t lds = ring > tail ? ring : tail;
    static_assert(lds <= 160 * 1024, "LDS budget");
    auto kern = gemm_nt_kernel<EPI, TM, TN, WM, WN, KG, NS>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds);
    if (e != hipSuccess) return e;
    const int tiles = ((p.M + TM - 1) / TM) * (p.N / TN);
    hipLaunchKernelGGL(kern, dim3((unsigned)(walk && tiles > kUnits ? kUnits : tiles), splits), dim3(64 * WM * WN * KG), lds, stream, p);
    return hipGetLastError();
}

template <int EPI>
static hipError_t launch_product(const GemmParams& p, const NtPlan& plan, hipStream_t stream)
{
    if (plan.tile == 64) return launch_nt<EPI, 64, 64, 1, 2, 4, 9>(p, plan.splits, stream);
    if (plan.tile == 128) return launch_nt<EPI, 128, 128, 2, 4, 1, 5>(p, plan.splits, stream);
    if constexpr (EPI == kEpiFloat) return launch_nt<EPI, 192, 256, 2, 4, 1, 5>(p, plan.splits, stream);
    else return launch_nt<EPI, 256, 256, 2, 4, 1, 5>(p, 1, stream);
}

// out = the sum of the shares, in order (n a multiple of 4)
__global__ __launch_bounds__(256) void proj_sum_kernel(const float* shares, float* out, size_t n, int splits)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    f32x4 s = *reinterpret_cast<const f32x4*>(shares + i);
#pragma unroll 4
    for (int k = 1; k < splits; ++k) s += *reinterpret_cast<const f32x4*>(shares + (size_t)k * n + i);
    *reinterpret_cast<f32x4*>(out + i) = s;
}

// ---- element-wise pass of the reverse mode -------------------------------------------------------
// dA[t][0:d] = dz, dA[t][d:2d] = dv * SiLU'(a_v), dA[t][2d:3d] = dq * q (1 - q), in this order (dx) and transposed, tokens padded
// with zeros to whole steps of 64 (dW3); and per block of ROWS tokens the column sums of dA (the bias gradients are
// their sum over the row blocks, in order).
//
// Bound by memory (16 bytes in and out per row and column triple, one reciprocal and exponential, and 6 for the transposed copy).  A
// workgroup takes 256 columns, which lie inside one of the three blocks (d is a multiple of 256), so what
// is read is chosen by a uniform branch; a thread holds V neighbouring columns and every V-th part of the
// rows, kActBatch rows requested at a time; the V parts' column sums meet in LDS, in order.
// V = 8 (16-byte vectors) needs 16-byte aligned arrays; others take V = 2.
// 16384 rows at width 2048: 540 MB 94 us without the transposed copy, 741 MB 120 us = 6.2 TB/s with it.
constexpr int kActBatch = 4;
constexpr int kActPitch = kActCols + 8;

// 8 consecutive rows (tokens) of one column of a [rows][pitch] LDS tile: lane -> column x0 + lane % 16, rows k0 + 8 (lane / 16) ..
__device__ __forceinline__ bf16x8 column_piece(const __bf16* tile, int pitch, int k0, int x0, int lane)
{
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const int i16 = lane & 15;
    const __bf16* p = tile + (k0 + 8 * (lane >> 4) + (i16 >> 2)) * pitch + x0 + 4 * (i16 & 3);
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 4 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int V, int ROWS>
__global__ __launch_bounds__(256) void proj_dact_kernel(const __bf16* dz, const __bf16* dv, const __bf16* dq, const __bf16* q,
                                                         const __bf16* av, __bf16* dA, __bf16* dAt, float* partial, int M, int Mp, int d)
{
    typedef __bf16 vec __attribute__((ext_vector_type(V)));
    constexpr int kPart = ROWS / V, kBatch = kPart < kActBatch ? kPart : kActBatch;      // rows of a thread; requested at a time
    static_assert(kPart % kBatch == 0 && ROWS % 32 == 0, "whole batches");
    __shared__ float sums[V][kActCols];
    extern __shared__ __align__(16) char smem[];
    __bf16* tile = reinterpret_cast<__bf16*>(smem);                       // [ROWS][kActPitch]
    const int tx = (int)threadIdx.x % (kActCols / V), ty = (int)threadIdx.x / (kActCols / V);
    const int col0 = (int)blockIdx.x * kActCols, which = col0 / d;
    const int c = col0 - which * d + tx * V;                              // of the block's own arrays
    const int t0 = (int)blockIdx.y * ROWS, r0 = t0 + ty * kPart;
    const __bf16* gsrc = which == 0 ? dz : which == 1 ? dv : dq;
    const __bf16* asrc = which == 1 ? av : q;
    float s[V];
#pragma unroll
    for (int e = 0; e < V; ++e) s[e] = 0.0f;
    for (int rb = r0; rb < r0 + kPart; rb += kBatch) {
        vec u[kBatch], a[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const size_t e = (size_t)min(rb + k, M - 1) * d + c;          // rows past the end re-read the last one (never used)
            u[k] = *reinterpret_cast<const vec*>(gsrc + e);
            if (which != 0) a[k] = *reinterpret_cast<const vec*>(asrc + e);
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            vec h;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                float g = (float)u[k][e];
                if (which == 1) {
                    const float x = (float)a[k][e];
                    const float sg = fast_rcp(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
                    g = g * sg * (1.0f + x * (1.0f - sg));
                } else if (which == 2) {
                    const float x = (float)a[k][e];
                    g = g * x * (1.0f - x);
                }
                h[e] = rb + k < M ? (__bf16)g : (__bf16)0.0f;             // tokens past the end contribute nothing
                s[e] += (float)h[e];                                      // the value the products will see (rounded to bf16)
            }
            if (rb + k < M) *reinterpret_cast<vec*>(dA + (size_t)(rb + k) * 3 * d + col0 + tx * V) = h;
            *reinterpret_cast<vec*>(tile + (size_t)(rb + k - t0) * kActPitch + tx * V) = h;
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) sums[ty][tx * V + e] = s[e];
    __syncthreads();
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < V; ++k) t += sums[k][threadIdx.x];
    partial[(size_t)blockIdx.y * 3 * d + col0 + (int)threadIdx.x] = t;
    // the transposed copy, 64 bytes of 16 columns a store
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int k0 = 0; k0 < ROWS; k0 += 32) {
            const bf16x8 v = column_piece(tile, kActPitch, k0, 64 * w + 16 * x, lane);
            const int tok = t0 + k0 + 8 * (lane >> 4);
            *reinterpret_cast<bf16x8*>(dAt + (size_t)(col0 + 64 * w + 16 * x + (lane & 15)) * Mp + tok) = v;
        }
}

template <int V, int ROWS>
static hipError_t launch_dact_rows(const void* dz, const void* dv, const void* dq, const void* q, const void* av, __bf16* dA,
                                   __bf16* dAt, float* partial, int M, int Mp, int d, hipStream_t stream)
{
    constexpr size_t lds = (size_t)ROWS * kActPitch * sizeof(__bf16);
    hipLaunchKernelGGL((proj_dact_kernel<V, ROWS>), dim3(3 * d / kActCols, Mp / ROWS), dim3(256), lds, stream,      // the padding of the transposed copy included
                       static_cast<const __bf16*>(dz), static_cast<const __bf16*>(dv), static_cast<const __bf16*>(dq),
                       static_cast<const __bf16*>(q), static_cast<const __bf16*>(av), dA, dAt, partial, M, Mp, d);
    return hipGetLastError();
}
template <int V>
static hipError_t launch_proj_dact(const void* dz, const void* dv, const void* dq, const void* q, const void* av, __bf16* dA,
                                   __bf16* dAt, float* partial, int M, int Mp, int d, hipStream_t stream)
{
    return act_rows(M, d) == 32 ? launch_dact_rows<V, 32>(dz, dv, dq, q, av, dA, dAt, partial, M, Mp, d, stream)
                                : launch_dact_rows<V, 64>(dz, dv, dq, q, av, dA, dAt, partial, M, Mp, d, stream);
}

// What the products of the reverse mode need besides dA, in one launch: workgroups 0 .. n_w3 - 1 transpose W3, the next n_x transpose x,
// the rest add up the bias gradients.

// dst [cols][ld] = src [rows][cols]^T (bf16), 64 x 64 tiles through LDS; cols and ld multiples of 64, rows past the end read as zero.
__device__ __forceinline__ void transpose_tile(__bf16* tile, const __bf16* src, __bf16* dst, int rows, int cols, int ld, int block)
{
    constexpr int P = 64 + 32;                     // rows 16 banks apart for the transpose reads
    const int r0 = block / (cols / 64) * 64, c0 = block % (cols / 64) * 64, tid = (int)threadIdx.x;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int r = (tid >> 3) + 32 * k, c = (tid & 7) * 8;
        u32x4 v = *reinterpret_cast<const u32x4*>(src + (size_t)min(r0 + r, rows - 1) * cols + c0 + c);
        if (r0 + r >= rows) v = u32x4{0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(tile + r * P + c) = v;
    }
    __syncthreads();
    const int lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int k0 = 0; k0 < 64; k0 += 32)
        *reinterpret_cast<bf16x8*>(dst + (size_t)(c0 + 16 * w + (lane & 15)) * ld + r0 + k0 + 8 * (lane >> 4)) =
            column_piece(tile, P, k0, 16 * w, lane);
}

// db[c] = sum over the row blocks of partial[block][c], in a fixed order: 32 columns per workgroup,
// the blocks in eight consecutive slices (one per 32 threads) that are then added in order.
constexpr int kBiasCols = 32, kBiasSlices = 8;

__global__ __launch_bounds__(kBiasCols * kBiasSlices) void proj_prepare_kernel(const __bf16* w3, __bf16* w3t, int n_w3, const __bf16* x,
                                                                               __bf16* xt, int n_x, int M, int Mp, int d,
                                                                               const float* partial, float* db, int n_blocks)
{
    __shared__ __align__(16) __bf16 tile[64 * (64 + 32)];
    const int id = (int)blockIdx.x;
    if (id < n_w3) { transpose_tile(tile, w3, w3t, 3 * d, d, 3 * d, id); return; }
    if (id < n_w3 + n_x) { transpose_tile(tile, x, xt, M, d, Mp, id - n_w3); return; }
    float (*part)[kBiasCols] = reinterpret_cast<float (*)[kBiasCols]>(tile);
    const int n = 3 * d, tx = (int)threadIdx.x % kBiasCols, ty = (int)threadIdx.x / kBiasCols;
    const int c = (id - n_w3 - n_x) * kBiasCols + tx;                // n is a multiple of 32
    const int per = (n_blocks + kBiasSlices - 1) / kBiasSlices;
    const int b0 = ty * per, b1 = min(n_blocks, b0 + per);
    float s = 0.0f;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += partial[(size_t)b * n + c];
    part[ty][tx] = s;
    __syncthreads();
    if (ty == 0) {
        float t = 0.0f;
#pragma unroll
        for (int k = 0; k < kBiasSlices; ++k) t += part[k][tx];
        db[c] = t;
    }
}

}   // namespace hgrn2

using namespace hgrn2;

namespace {
int proj_check(int32_t M, int32_t d)
{
    if (M < 0 || d < 0) return HGRN2_ERR_SHAPE;
    if ((long long)M * 3 * d > (long long)INT32_MAX * 8) return HGRN2_ERR_SHAPE;
    if (d % 256 != 0) return HGRN2_ERR_UNSUPPORTED;        // a 256-column block of the product lies inside one of z, v, q
    return HGRN2_OK;
}
size_t round256p(size_t x) { return (x + 255) & ~(size_t)255; }
size_t padded(int32_t M) { return ((size_t)M + 63) & ~(size_t)63; }        // tokens, in whole steps of the product that contracts over them

// workspace of the reverse mode: dA, row-block sums of dA, W3 transposed, dA and x transposed, the shares of dW3
struct ProjBwdLayout {
    size_t dA, partial, w3t, dAt, xt, shares;
    int rows;             // of a row block
    NtPlan plan_w;
    size_t total() const { return dA + partial + w3t + dAt + xt + shares; }
};
ProjBwdLayout proj_bwd_layout(int32_t M, int32_t d)
{
    ProjBwdLayout l = {};
    if (M == 0 || d == 0) return l;
    const size_t n = 3 * (size_t)d;
    l.rows = act_rows(M, d);
    l.plan_w = plan_nt(3 * d, d, (int)padded(M), true);
    l.dA = round256p((size_t)M * n * sizeof(__bf16));
    l.partial = round256p(padded(M) / l.rows * n * sizeof(float));
    l.w3t = round256p(n * d * sizeof(__bf16));
    l.dAt = round256p(padded(M) * n * sizeof(__bf16));
    l.xt = round256p(padded(M) * d * sizeof(__bf16));
    l.shares = l.plan_w.splits > 1 ? round256p(l.plan_w.splits * n * d * sizeof(float)) : 0;
    return l;
}
}   // namespace

extern "C" {

size_t hgru2_proj_bwd_workspace_bytes(int32_t M, int32_t d)
{
    if (proj_check(M, d) != HGRN2_OK) return 0;
    return proj_bwd_layout(M, d).total();
}

int hgru2_proj_fwd(int32_t M, int32_t d, const void* x, const void* w3, const float* b3, void* z, void* v, void* q,
                   void* av, void* hip_stream)
{
    const int rc = proj_check(M, d);
    if (rc != HGRN2_OK) return rc;
    if ((size_t)M * d == 0) return HGRN2_OK;
    if (!x || !w3 || !b3 || !z || !v || !q) return HGRN2_ERR_NULL;
    GemmParams p = {};
    p.A = static_cast<const __bf16*>(x); p.lda = d;
    p.B = static_cast<const __bf16*>(w3); p.ldb = d;
    p.M = M; p.N = 3 * d; p.K = d;
    p.bias = b3; p.z = static_cast<__bf16*>(z); p.v = static_cast<__bf16*>(v); p.q = static_cast<__bf16*>(q);
    p.av = static_cast<__bf16*>(av); p.d = d;
    return launch_product<kEpiProj>(p, plan_nt(M, 3 * d, d, false), static_cast<hipStream_t>(hip_stream)) == hipSuccess ? HGRN2_OK : HGRN2_ERR_HIP;
}

int hgru2_proj_bwd(int32_t M, int32_t d, const void* x, const void* w3, const void* q, const void* av, const void* grad_z,
                   const void* grad_v, const void* grad_q, void* grad_x, float* grad_w3, float* grad_b3, void* workspace,
                   size_t workspace_bytes, void* hip_stream)
{
    const int rc = proj_check(M, d);
    if (rc != HGRN2_OK) return rc;
    if (d == 0) return HGRN2_OK;
    if (!grad_w3 || !grad_b3) return HGRN2_ERR_NULL;
    if (M > 0 && (!x || !w3 || !q || !av || !grad_z || !grad_v || !grad_q || !grad_x)) return HGRN2_ERR_NULL;
    const size_t need = hgru2_proj_bwd_workspace_bytes(M, d);
    if (need > 0 && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))) return HGRN2_ERR_WORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (M == 0) {       // nothing contributes
        if (launch_zero_floats(grad_w3, (size_t)3 * d * d, stream) != hipSuccess ||
            launch_zero_floats(grad_b3, (size_t)3 * d, stream) != hipSuccess)
            return HGRN2_ERR_HIP;
        return HGRN2_OK;
    }
    const ProjBwdLayout l = proj_bwd_layout(M, d);
    char* at = static_cast<char*>(workspace);
    auto take = [&](size_t bytes) { char* r = at; at += bytes; return r; };
    __bf16* dA = reinterpret_cast<__bf16*>(take(l.dA));
    float* partial = reinterpret_cast<float*>(take(l.partial));
    __bf16* w3t = reinterpret_cast<__bf16*>(take(l.w3t));
    __bf16* dAt = reinterpret_cast<__bf16*>(take(l.dAt));
    __bf16* xt = reinterpret_cast<__bf16*>(take(l.xt));
    float* shares = reinterpret_cast<float*>(take(l.shares));
    const int Mp = (int)padded(M), blocks = Mp / l.rows;
    const bool aligned = (((uintptr_t)grad_z | (uintptr_t)grad_v | (uintptr_t)grad_q | (uintptr_t)q | (uintptr_t)av) & 15) == 0;
    if ((aligned ? launch_proj_dact<8>(grad_z, grad_v, grad_q, q, av, dA, dAt, partial, M, Mp, d, stream)
                 : launch_proj_dact<2>(grad_z, grad_v, grad_q, q, av, dA, dAt, partial, M, Mp, d, stream)) != hipSuccess)
        return HGRN2_ERR_HIP;
    const int n_w3 = 3 * d / 64 * (d / 64), n_x = Mp / 64 * (d / 64);
    hipLaunchKernelGGL(proj_prepare_kernel, dim3(n_w3 + n_x + 3 * d / kBiasCols), dim3(kBiasCols * kBiasSlices), 0, stream,
                       static_cast<const __bf16*>(w3), w3t, n_w3, static_cast<const __bf16*>(x), xt, n_x, M, Mp, d, partial, grad_b3, blocks);
    if (hipGetLastError() != hipSuccess) return HGRN2_ERR_HIP;
    // dx [M][d] = dA [M][3d] . W3 [3d][d]
    GemmParams px = {};
    px.A = dA; px.lda = 3 * d;
    px.B = w3t; px.ldb = 3 * d;
    px.M = M; px.N = d; px.K = 3 * d;
    px.C = static_cast<__bf16*>(grad_x); px.ldc = d;
    if (launch_product<kEpiPlain>(px, plan_nt(M, d, 3 * d, false), stream) != hipSuccess) return HGRN2_ERR_HIP;
    // dW3 [3d][d] = dA^T [3d][M] . x [M][d]
    GemmParams pw = {};
    pw.A = dAt; pw.lda = Mp;
    pw.B = xt; pw.ldb = Mp;
    pw.M = 3 * d; pw.N = d; pw.K = Mp;
    pw.Cf = l.plan_w.splits > 1 ? shares : grad_w3; pw.ldc = d;
    if (launch_product<kEpiFloat>(pw, l.plan_w, stream) != hipSuccess) return HGRN2_ERR_HIP;
    if (l.plan_w.splits > 1) {
        const size_t n = (size_t)3 * d * d;
        hipLaunchKernelGGL(proj_sum_kernel, dim3((unsigned)(n / 1024)), dim3(256), 0, stream, shares, grad_w3, n, l.plan_w.splits);
        if (hipGetLastError() != hipSuccess) return HGRN2_ERR_HIP;
    }
    return HGRN2_OK;
}

}   // extern "C"
