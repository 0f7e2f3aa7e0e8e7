// Per-chunk forward read-out of the chunkwise HGRN2 algorithm (paper Section 3.2, Eq. 3,
// unrolled inside one chunk of C tokens whose incoming state is S_n):
//
//     o_i = sum_{j<=i} ( sum_a q_i[a] k_j[a] prod_{j<s<=i} f_s[a] ) v_j  +  (q_i * G_i) S_n
//
// (q_i * G_i) S_n is evaluated as Q~_i (G_m * S_n): the state sweep stores G_m * S_n.
//
// The decay between two tokens is factored around the reference row m = C/2:
//     prod_{j<s<=i} f_s = (G_i / G_m) (G_m / G_j)  ->  P = tril(Q~ K~^T),  Q~ = q G/G_m,  K~ = k G_m/G
// so every cumulative product spans at most C/2 tokens, and the one that appears as a divisor is
// the product BETWEEN the row and the reference, formed directly by multiplication (no logs).
// One workgroup handles one chunk of one (batch, head); all chunks are independent because the
// state sweep has already written every S_n.  P is built transposed so that the accumulator
// registers already hold 4 consecutive j per lane and go to LDS as 8-byte vectors.
//
// From contributions (ADD, fp32 storage, few sequences of few chunks): instead of a sweep that walks the
// chunks in order -- one workgroup per sequence and column slab, 5 us a chunk, 20 of the 29 us of a
// forward pass over 256 tokens of one head -- a sweep launch takes every chunk from zero at once, and
// the workgroup of chunk n adds up the contributions of the chunks before it,
//     S_n = Diag(g_{n-1}) ( ... Diag(g_0) h0 + A_0 ... ) + A_{n-1},
// out of the cache.  What bounds it is the chain of one chunk, products on fp32 matrix instructions most of all
// (64 clocks each), so a workgroup takes 64 dv columns (half of a 128-wide head's: half of the contributions to
// add up and of the products, for P formed twice; see launch_fwd_out_add()), and the final state, h (G_m S_n) + K^^T V, is a workgroup of its
// own beside the last chunk's while all find a place at once.  us, one workgroup for all of it -> now: one head of 64 x 64,
// 64 / 256 / 4096 tokens 11.6 / 20.6 / 31.4 -> 9.9 / 18.3 / 29.2; of 128 x 128, 64 / 256 / 1024 tokens 20.0 / 30.7 / 39.9 -> 12.0 / 20.9 /
// 25.9; 32 heads of 128 x 128, 192 tokens 33.5 -> 26.1; 64 of 64 x 128 29.4 -> 26.0.
#include "common.hpp"
#include "kernels.hpp"

namespace hgrn2 {

struct FwdOutParams {
    const void* q;
    const void* f;
    const void* v;
    const void* ws;
    void* o;
    int BH, N, NC, gate_bf16;
    const float* beta;   // [H][dk] lower bounds, or null: the gate tensor holds f itself
    int H;
    TokenLayout lay;     // used when dense == 0
    int dense;           // sequence tensors are [B][H][N][d]
    int* flag;           // null, or set to 1 when a gate product falls below the floor of the reciprocals
    // ADD: what chunk j of sequence s adds from zero is at add + (s NC + j) dk dv, the product of its gates
    // at decay + s decay_stride + j dk (j < NC - 1); initial and final states as the C ABI's
    const float* add;
    const float* decay;
    size_t decay_stride;
    const float* h0;
    float* hT;
    int chunk_items;         // workgroups of chunks (chunk, slab of dv)
    int final_items;         // workgroups behind them that form the final states (sequence, slab); 0: the last chunks' do
};

template <typename T, int DK, int DV> struct FwdOutLds {
    static constexpr int C = kChunk;
    static constexpr int PK = DK + pad_elems<T>();
    static constexpr int PC = C + pad_elems<T>();
    static constexpr int PO = DV + pad_elems<T>();
    static constexpr size_t qm = 0;                                   // [C][PK]  Q~
    static constexpr size_t km = qm + (size_t)C * PK * sizeof(T);     // [C][PK]  K~, later [C][PO] output staging
    static constexpr size_t ost = km;
    static constexpr size_t vt = km + (size_t)C * (PK > PO ? PK : PO) * sizeof(T);   // [DV][PC] V transposed
    static constexpr size_t pm = vt + (size_t)DV * PC * sizeof(T);    // [C][PC]  P
    static constexpr size_t tot = pm + (size_t)C * PC * sizeof(T);    // [4][DK] fp32
    static constexpr size_t total = tot + (size_t)kWaves * DK * sizeof(float);
};

// ADD: 0, or the dv columns of a workgroup that adds up contributions
template <typename T, int DK, int DV, bool DENSE, int ADD>
__device__ __forceinline__ void fwd_out_body(const FwdOutParams& p)
{
    static_assert(!ADD || !is_bf16_type<T>(), "bf16 storage takes the fused walk");
    constexpr int C = kChunk, RW = C / kWaves;
    constexpr int DVW = ADD ? ADD : DV, NSPLIT = DV / DVW;           // dv columns of the workgroup
    typedef FwdOutLds<T, DK, DVW> L;
    constexpr int PK = L::PK, PC = L::PC, PO = L::PO;
    constexpr int NRT = C / 32, NBT = DVW / 32, NKS = DK / 16;
    typedef Mma<T> M;

    extern __shared__ __align__(16) char smem[];
    T* Qm = reinterpret_cast<T*>(smem + L::qm);
    T* Km = reinterpret_cast<T*>(smem + L::km);
    T* Vt = reinterpret_cast<T*>(smem + L::vt);
    T* Pm = reinterpret_cast<T*>(smem + L::pm);
    float* tot = reinterpret_cast<float*>(smem + L::tot);
    T* Ost = reinterpret_cast<T*>(smem + L::ost);   // output staging aliases K~ once P has been formed

    if (not_chosen(p.lay)) return;       // one of several chunk lengths, and not the one called for
    int n, bh, dv0 = 0;                  // dv0: first dv column of the workgroup
    bool final_only = false;             // a workgroup that only forms a final state
    if constexpr (ADD != 0) {
        int item = blockIdx.x;
        final_only = item >= p.chunk_items;
        if (final_only) item = ((item - p.chunk_items) / NSPLIT * p.NC + p.NC - 1) * NSPLIT + (item - p.chunk_items) % NSPLIT;
        dv0 = item % NSPLIT * DVW;
        if (!locate_chunk<DENSE>(p.lay, p.BH, p.NC, item / NSPLIT, bh, n)) return;
    } else {
        if (!locate_chunk<DENSE>(p.lay, p.BH, p.NC, blockIdx.x, bh, n)) return;
    }
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const bool k_act = 2 * lane < DK, v_act = 2 * lane < DVW;
    const SeqView sv = seq_view<DENSE, DK, DV>(p.lay, p.N, p.NC, bh);
    const size_t seq_k = sv.off_k, seq_v = sv.off_v;
    const int N = sv.N;
    const ChunkRows cr = chunk_rows(p.lay.sub, n, N);        // which tokens the chunk's rows stand for
    const int ld_k = DENSE ? DK : (int)p.lay.sn_k, ld_v = DENSE ? DV : (int)p.lay.sn_v;   // token stride, elements
    const bool gate_bf16 = p.gate_bf16 != 0;
    const T* qg = static_cast<const T*>(p.q);
    const T* vg = static_cast<const T*>(p.v);
    const T* wsn = static_cast<const T*>(p.ws) + (size_t)blockIdx.x * DK * DV;      // chunk indices are the workspace order

    // ---------------- loads ----------------
    // incoming state S_n, column block bt of this wave, as B-operand fragments (k runs over dk)
    static_assert(kWaves % NBT == 0 && (NRT * NBT) % kWaves == 0, "tile/wave mapping");
    const int bt = w % NBT;
    typename M::frag sfrag[NKS];
    if constexpr (ADD == 0) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            sfrag[ks] = *reinterpret_cast<const typename M::frag*>(
                wsn + state_frag_offset(ks >> 1, bt, NBT, ks & 1, lane));
    }
    f32x2 rf[RW], rq[RW], rv[RW];
    {
        RawRows<RW> raw_f, raw_q, raw_v;
        const int row0 = cr.tok0 + RW * w;
        const int col_k = k_act ? 2 * lane : 0, col_v = dv0 + (v_act ? 2 * lane : 0);
        load_rows<RW>(raw_f, p.f, seq_k, ld_k, col_k, row0, N, gate_bf16);
        load_rows<RW>(raw_q, qg, seq_k, ld_k, col_k, row0, N, is_bf16_type<T>());
        load_rows<RW>(raw_v, vg, seq_v, ld_v, col_v, row0, N, is_bf16_type<T>());
        convert_rows<RW>(rf, raw_f, row0, cr.end, k_act, gate_bf16, 1.0f, cr.first);
        if (p.beta) gate_rows<RW>(rf, p.beta + (size_t)(bh % p.H) * DK, col_k, k_act, row0, cr.end, cr.first);
        convert_rows<RW>(rq, raw_q, row0, cr.end, k_act, is_bf16_type<T>(), 0.0f, cr.first);
        convert_rows<RW>(rv, raw_v, row0, cr.end, v_act, is_bf16_type<T>(), 0.0f, cr.first);
    }
    if constexpr (ADD != 0) {
        // The sum goes over the whole workgroup in 16-byte vectors, several chunks' requested at a time
        // (what one request takes -- the values come from other XCDs -- is most of what a chunk costs:
        // 5 us each when every lane fetched its fragments chunk after chunk), and reaches the fragments
        // through the memory of the tiles that are written next.
        constexpr int NV = DK * DVW / 4 / kThreads, AHEAD = NV > 4 ? 4 : 6;
        f32x4 st[NV];
        const float* h0 = p.h0 ? p.h0 + (size_t)bh * DK * DV : nullptr;
        const float* add = p.add + (size_t)bh * p.NC * DK * DV;
        const float* dec = p.decay + (size_t)bh * p.decay_stride;
        auto at = [&](int i) { return 4 * (tid + kThreads * i); };               // in the workgroup's [DK][DVW]
        auto in_state = [&](int i) { return at(i) / DVW * DV + dv0 + at(i) % DVW; };
#pragma unroll
        for (int i = 0; i < NV; ++i) st[i] = h0 ? *reinterpret_cast<const f32x4*>(h0 + in_state(i)) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int j0 = 0; j0 < n; j0 += AHEAD) {
            f32x4 a[AHEAD][NV];
            float dm[AHEAD][NV];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const int j = min(j0 + u, n - 1);
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    a[u][i] = *reinterpret_cast<const f32x4*>(add + (size_t)j * DK * DV + in_state(i));
                    dm[u][i] = dec[j * DK + at(i) / DVW];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if (j0 + u >= n) break;
#pragma unroll
                for (int i = 0; i < NV; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[i][e] = fmaf(dm[u][i], st[i][e], a[u][i][e]);
            }
        }
        float* sum = reinterpret_cast<float*>(smem);
        static_assert((size_t)DK * DVW * sizeof(float) <= L::tot, "the state fits the memory of the tiles");
#pragma unroll
        for (int i = 0; i < NV; ++i) *reinterpret_cast<f32x4*>(sum + at(i)) = st[i];
        __syncthreads();
        // element s of fragment ks: row 16 ks + 8 (s / 4) + 4 g + s % 4 of column 32 bt + r32
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int s = 0; s < 8; ++s) sfrag[ks].v[s] = sum[(size_t)(16 * ks + 8 * (s >> 2) + 4 * g + (s & 3)) * DVW + 32 * bt + r32];
        // (the tiles are written after the next barrier)
    }

    // ---------------- gate products and scaled operands ----------------
    float a0[RW], a1[RW], z0[RW], z1[RW];
    {
        float run0 = 1.0f, run1 = 1.0f;
#pragma unroll
        for (int i = 0; i < RW; ++i) { run0 *= rf[i].x; run1 *= rf[i].y; a0[i] = run0; a1[i] = run1; }
        run0 = 1.0f; run1 = 1.0f;
#pragma unroll
        for (int i = RW - 1; i >= 0; --i) { z0[i] = run0; z1[i] = run1; run0 *= rf[i].x; run1 *= rf[i].y; }
    }
    float kz0[ADD ? RW : 1], kz1[ADD ? RW : 1];          // k z, for the final state
    if constexpr (ADD != 0) {
#pragma unroll
        for (int i = 0; i < RW; ++i) { kz0[i] = (1.0f - rf[i].x) * z0[i]; kz1[i] = (1.0f - rf[i].y) * z1[i]; }
    }
    if (k_act) {
        tot[w * DK + 2 * lane] = a0[RW - 1];
        tot[w * DK + 2 * lane + 1] = a1[RW - 1];
    }
    __syncthreads();
    if (k_act) {
        const BlockDecay d0 = block_decay(tot, DK, w, 2 * lane);
        const BlockDecay d1 = block_decay(tot, DK, w, 2 * lane + 1);
        {   // the smallest product this thread takes a reciprocal of: its first row after the reference, its last before
            const float s0 = d0.mid * (w >= 2 ? a0[RW - 1] : z0[0]), s1 = d1.mid * (w >= 2 ? a1[RW - 1] : z1[0]);
            if (p.flag && fminf(s0, s1) < kTinyProduct) *p.flag = 1;
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int row = RW * w + i;
            // m = product of the gates strictly between this row and the reference row C/2
            float m0, m1, qs0, qs1, ks0, ks1;
            if (w >= 2) {          // rows after the reference: G_i/G_m = m <= 1
                m0 = d0.mid * a0[i]; m1 = d1.mid * a1[i];
                const float i0 = fast_rcp(fmaxf(m0, kTinyProduct)), i1 = fast_rcp(fmaxf(m1, kTinyProduct));
                qs0 = rq[i].x * m0; qs1 = rq[i].y * m1;
                ks0 = (1.0f - rf[i].x) * i0; ks1 = (1.0f - rf[i].y) * i1;
            } else {               // rows up to the reference: G_m/G_j = m <= 1
                m0 = d0.mid * z0[i]; m1 = d1.mid * z1[i];
                const float i0 = fast_rcp(fmaxf(m0, kTinyProduct)), i1 = fast_rcp(fmaxf(m1, kTinyProduct));
                qs0 = rq[i].x * i0; qs1 = rq[i].y * i1;
                ks0 = (1.0f - rf[i].x) * m0; ks1 = (1.0f - rf[i].y) * m1;
            }
            store_pair_t<T>(Qm, (size_t)row * PK + 2 * lane, qs0, qs1);
            store_pair_t<T>(Km, (size_t)row * PK + 2 * lane, ks0, ks1);
        }
    }
    if (v_act) {
        float x0[RW], x1[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) { x0[i] = rv[i].x; x1[i] = rv[i].y; }
        store_run<T, RW>(Vt + (2 * lane) * PC + RW * w, x0);
        store_run<T, RW>(Vt + (2 * lane + 1) * PC + RW * w, x1);
    }
    __syncthreads();

    if constexpr (ADD != 0) {
        // the read-out takes G_m S_n (the totals are complete since the first barrier)
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int row = 16 * ks + 8 * c + 4 * g;
                const f32x4 t0 = *reinterpret_cast<const f32x4*>(tot + row), t1 = *reinterpret_cast<const f32x4*>(tot + DK + row);
#pragma unroll
                for (int s = 0; s < 4; ++s) sfrag[ks].v[4 * c + s] *= t0[s] * t1[s];
            }
    }

    // ---------------- P^T blocks: (J, I) with J <= I; wave w takes block w ----------------
    {
        constexpr int NBLK = NRT * (NRT + 1) / 2;
        for (int blk = final_only ? NBLK : w; blk < NBLK; blk += kWaves) {
            // enumerate (J, I): 0 -> (0,0), 1 -> (0,1), 2 -> (1,1)
            int I = 0, J = 0, cnt = 0;
            for (int ii = 0; ii < NRT; ++ii)
                for (int jj = 0; jj <= ii; ++jj) { if (cnt == blk) { I = ii; J = jj; } ++cnt; }
            f32x16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const typename M::frag fa = M::load(Km + (32 * J + r32) * PK + 16 * ks + 8 * g);
                const typename M::frag fb = M::load(Qm + (32 * I + r32) * PK + 16 * ks + 8 * g);
                M::mma(acc, fa, fb);    // acc[row j][col i]
            }
            const int i_glob = 32 * I + r32;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int j0 = 32 * J + 8 * c + 4 * g;
                float x[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) x[jj] = (j0 + jj <= i_glob) ? acc[4 * c + jj] : 0.0f;
                store_pair_t<T>(Pm, (size_t)i_glob * PC + j0, x[0], x[1]);
                store_pair_t<T>(Pm, (size_t)i_glob * PC + j0 + 2, x[2], x[3]);
            }
        }
    }
    if (!final_only) __syncthreads();

    if constexpr (ADD != 0) {
        // Final state, of the last chunk: h (G_m S_n) + K^^T V with K^_j = k_j prod_{s > j} f_s, as the sweep
        // forms it (K~ has a reciprocal in it, whose error the state would keep), in the tile the P blocks have
        // read K~ from.  Tiles (at, bt), the channel tiles dealt to the waves of a dv tile; fragments 2 at and
        // 2 at + 1 hold the state in accumulator order.
        if (final_only || (p.hT && p.final_items == 0 && n == p.NC - 1)) {
            if (k_act) {
                const float p0 = block_decay(tot, DK, w, 2 * lane).post, p1 = block_decay(tot, DK, w, 2 * lane + 1).post;
#pragma unroll
                for (int i = 0; i < RW; ++i) store_pair_t<T>(Km, (size_t)(RW * w + i) * PK + 2 * lane, kz0[i] * p0, kz1[i] * p1);
            }
            __syncthreads();
#pragma unroll
            for (int at = 0; at < DK / 32; ++at) {
                if (at % (kWaves / NBT) != w / NBT) continue;
                f32x16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int ch = 32 * at + acc_row(v, lane);
                    acc[v] = sfrag[2 * at + (v >> 3)].v[v & 7] * (tot[2 * DK + ch] * tot[3 * DK + ch]);
                }
#pragma unroll
                for (int ks = 0; ks < C / 16; ++ks)
                    M::mma(acc, M::load_kmajor(Km, PK, 16 * ks, 32 * at, lane), M::load(Vt + (32 * bt + r32) * PC + 16 * ks + 8 * g));
                float* out = p.hT + (size_t)bh * DK * DV + (size_t)(32 * at) * DV + dv0 + 32 * bt + r32;
#pragma unroll
                for (int v = 0; v < 16; ++v) out[(size_t)acc_row(v, lane) * DV] = acc[v];
            }
            if (final_only) return;
            __syncthreads();                 // (the O tiles take this memory)
        }
    }

    // ---------------- O tiles: P V + (q G) S_n ----------------
    // (NRT * NBT is a multiple of the wave count and NBT divides it, so every tile of a wave
    // shares the column block bt and the state fragments loaded at the top are reused.)
    for (int tix = w; tix < NRT * NBT; tix += kWaves) {
        const int rt = tix / NBT;
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
        for (int ks = 0; ks < 2 * (rt + 1); ++ks) {
            const typename M::frag fa = M::load(Pm + (32 * rt + r32) * PC + 16 * ks + 8 * g);
            const typename M::frag fb = M::load(Vt + (32 * bt + r32) * PC + 16 * ks + 8 * g);
            M::mma(acc, fa, fb);
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            // k-slot order of the state fragments: rows 16ks + {4g..4g+3, 8+4g..8+4g+3}
            const T* qrow = Qm + (32 * rt + r32) * PK + 16 * ks + 4 * g;
            const typename M::frag fa = M::load2(qrow, qrow + 8);
            M::mma(acc, fa, sfrag[ks]);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v)
            Ost[(size_t)(32 * rt + acc_row(v, lane)) * PO + 32 * bt + r32] = (T)acc[v];
    }
    __syncthreads();

    // ---------------- coalesced store of the [C][DV] tile ----------------
    {
        constexpr int VEC = 16 / (int)sizeof(T);         // elements per 16-byte vector
        constexpr int VPR = DVW / VEC;                    // vectors per row
        T* og = static_cast<T*>(p.o);
        for (int idx = tid; idx < C * VPR; idx += kThreads) {
            const int row = idx / VPR, cv = idx % VPR;
            const int grow = cr.tok0 + row;
            if (cr.holds(row)) {
                const uint4 val = *reinterpret_cast<const uint4*>(Ost + (size_t)row * PO + cv * VEC);
                *reinterpret_cast<uint4*>(og + seq_v + (size_t)grow * ld_v + dv0 + cv * VEC) = val;
            }
        }
    }
}

constexpr int kUnits = 256;      // compute units

// Workgroups that add up contributions for heads of 64 find two places on a compute unit: six chunks' values requested at
// a time instead of eight leave the registers for it (128 heads of 64, 192 tokens: 35.9 -> 28.7 us).
constexpr int add_places(int dk, int cols) { return dk == 64 && cols == 64 ? 2 : 1; }

template <typename T, int DK, int DV, int ADD>
__global__ __launch_bounds__(kThreads, ADD ? add_places(DK, ADD) : 1) void fwd_out_kernel(FwdOutParams p)
{
    if (p.dense) fwd_out_body<T, DK, DV, true, ADD>(p);
    else         fwd_out_body<T, DK, DV, false, ADD>(p);
}

template <typename T, int DK, int DV, int ADD>
static hipError_t launch_one(const SeqDims& d, const FwdOutParams& p, hipStream_t stream)
{
    constexpr int DVW = ADD ? ADD : DV, NSPLIT = DV / DVW;
    typedef FwdOutLds<T, DK, DVW> L;
    auto kern = fwd_out_kernel<T, DK, DV, ADD>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)L::total);
    if (e != hipSuccess) return e;
    FwdOutParams a = p;
    a.chunk_items = (int)d.total_chunks() * NSPLIT;
    a.final_items = 0;
    if constexpr (ADD != 0) {
        constexpr int places = add_places(DK, ADD);
        static_assert(places * L::total <= 160 * 1024, "LDS budget of the workgroups of a compute unit");
        // Final states beside the chunks, if all run at once on the 256 compute units; where a sequence is one chunk, only on a
        // unit each (192 heads of 64 x 64, 64 tokens: 13.4 us beside the chunks, two on a unit, 12.7 in them).
        const long long all = (long long)a.chunk_items + (long long)d.BH * NSPLIT;
        if (p.hT && all <= kUnits * (d.NC > 1 ? places : 1)) a.final_items = d.BH * NSPLIT;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.chunk_items + a.final_items)), dim3(kThreads), L::total, stream, a);
    return hipGetLastError();
}

// COLS: 0, or the dv columns of a workgroup that adds up contributions
template <typename T, int COLS>
static hipError_t launch_dims(const SeqDims& d, const FwdOutParams& p, hipStream_t stream)
{
    if (d.dk == 128 && d.dv == 128) return launch_one<T, 128, 128, COLS>(d, p, stream);
    if (d.dk == 64 && d.dv == 64) return launch_one<T, 64, 64, COLS>(d, p, stream);
    if (d.dk == 128 && d.dv == 64) return launch_one<T, 128, 64, COLS>(d, p, stream);
    if (d.dk == 64 && d.dv == 128) return launch_one<T, 64, 128, COLS>(d, p, stream);
    return hipErrorInvalidValue;
}

static FwdOutParams out_params(const SeqDims& d, const void* q, const void* f, const void* v, void* o)
{
    FwdOutParams p;
    p.q = q; p.f = f; p.v = v; p.ws = nullptr; p.o = o;
    p.BH = d.BH; p.N = d.N; p.NC = d.NC; p.gate_bf16 = d.gate_bf16 ? 1 : 0;
    p.beta = d.beta; p.H = d.H; p.lay = d.lay; p.dense = d.dense() ? 1 : 0; p.flag = d.domain_flag;
    p.add = nullptr; p.decay = nullptr; p.decay_stride = 0; p.h0 = nullptr; p.hT = nullptr; p.chunk_items = 0; p.final_items = 0;
    return p;
}

hipError_t launch_fwd_out(const SeqDims& d, const void* q, const void* f, const void* v, const void* ws_state,
                          void* o, hipStream_t stream)
{
    if (d.total_chunks() == 0) return hipSuccess;
    FwdOutParams p = out_params(d, q, f, v, o);
    p.ws = ws_state;
    return d.io_bf16 ? launch_dims<__bf16, 0>(d, p, stream) : launch_dims<float, 0>(d, p, stream);
}

hipError_t launch_fwd_out_add(const SeqDims& d, const void* q, const void* f, const void* v, const float* add,
                              const float* decay, size_t decay_stride, const float* h0, void* o, float* hT, hipStream_t stream)
{
    if (d.total_chunks() == 0) return hipSuccess;
    if (d.io_bf16 || d.packed) return hipErrorInvalidValue;
    FwdOutParams p = out_params(d, q, f, v, o);
    p.add = add; p.decay = decay; p.decay_stride = decay_stride; p.h0 = h0; p.hT = hT;
    // Heads of 64 x 128 are halved only while the halves find a unit each: two of them on a unit take longer than one workgroup
    // for all columns (us, halves / whole: 129 heads of 64 tokens 18.3 / 16.2, 192 19.2 / 16.8; 96 of 128 tokens 30.2 / 28.3, 48 of 256 tokens 29.8 / 27.5).
    if (d.dk == 64 && d.dv == 128 && 2 * d.total_chunks() > kUnits) return launch_one<float, 64, 128, 128>(d, p, stream);
    return launch_dims<float, 64>(d, p, stream);
}

}   // namespace hgrn2
