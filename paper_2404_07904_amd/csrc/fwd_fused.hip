// Fused forward pass of the chunkwise HGRN2 algorithm (paper Section 3.2, Eq. 3): the
// chunk-to-chunk state recurrence and the per-chunk read-out in ONE pass over q, f, v,
//
//     O_n     = tril(Q~ K~^T) V + Q~ (G_m S_n)
//     S_{n+1} = h (G_m S_n + K~^T V)
//
// with Q~ = q G/G_m, K~ = k G_m/G (k = 1 - f, G the cumulative gate product inside the chunk, G_m
// its value after the first half of the chunk, h the product over the second half), so that the
// per-chunk states never travel through HBM (the two-kernel path writes and re-reads 2*dk*dv
// bytes per chunk, as much again as the chunk's own q, f, v, o).  One workgroup (eight wave64s; heads
// of 64: four) walks the chunks of a (batch, head), or of a run or span of them (below), in order,
// software-pipelined in two stages per chunk with one barrier after each:
//
//   stage A(n):  store O(n-1) from its LDS staging tile; copy V(n) into LDS; rescale the state
//                to G_m(n) S_n and publish it (bf16, MFMA-fragment order) to LDS; first half of
//                the element-wise work of chunk n+1 (gate products, per-wave block totals);
//                P(n) = tril(Q~ K~^T) on three waves
//   stage B(n):  all remaining contractions of chunk n (Q~ (G_m S_n), P V, K~^T V) while the
//                second half of the element-wise work of chunk n+1 (Q~, K~ tiles) fills the
//                other tile buffer; O(n) into its staging tile
//
//   * the dk x dv state lives in fp32 MFMA accumulators, two 32x32 tiles per wave;
//   * wave w owns rows 8w..8w+7 of the chunk for the element-wise work (gate products along time
//     serially in registers, channel pair per lane) and the 32x32 output tile (w/4, w%4);
//   * V is a raw row-major [token][channel] copy (no arithmetic on its way in) and is read with LDS
//     transpose loads; K~ is kept transposed ([channel][token], which the row-block layout writes
//     as 16-byte vectors), so that the state update reads it with plain 16-byte loads; Q~ keeps
//     its columns in the order the state fragments hold the contraction index (bits 2 and 3 of
//     the channel swapped), so that its operand of the read-out is one 16-byte load too;
//   * rows are fetched two chunks ahead into two alternating register sets.
//   * with fewer sequences than compute units, two workgroups share a sequence, each owning one
//     half of the dv columns (of V, O and the state): the element-wise work on q and f and the
//     P blocks are done twice, everything that scales with dv is halved, and the whole chip is busy.
//   * heads of 64 channels take workgroups of four waves, two on a compute unit: a wave then owns
//     two row blocks, one per half wave, since a row has only 32 channel pairs.
//   * few or long sequences: a workgroup owns a run of a sequence's chunks.  The state that enters
//     the run comes from a light walk over the chunks before it (the recurrence alone: f, V and
//     about 0.4 of a chunk's time), either its own, from the sequence's initial state (cuts
//     placed so that all workgroups finish together), or -- for long sequences -- from walks
//     from zero, one per run, by run_ends_kernel, whose results the workgroup adds up first.
//   * a packed batch gives a workgroup a SPAN of a head's chunks, sequence after sequence, however
//     they lie: the pipeline runs on across the sequence boundaries (the rows of the next sequence's
//     first chunks are fetched while the current one ends), the state is replaced by the next
//     sequence's initial state where it starts and written out where one ends; a span that starts
//     inside a sequence finds its state as a run does, by a light walk or from run_ends_kernel.
//     Every workgroup walks equally many chunks, whatever the lengths are.
// Used for bf16 storage; fp32 storage takes the sweep + read-out path.
#include "common.hpp"
#include "kernels.hpp"
#include <type_traits>

namespace hgrn2 {

struct FwdFusedParams {
    const void* q;
    const void* f;
    const void* v;
    const float* h0;
    void* o;
    float* hT;
    void* save;          // null, or where every chunk's scaled incoming state G_m S_n goes for a later backward pass
    int N, NC, BH;
    const float* beta;   // [H][dk] lower bounds, or null: the gate tensor holds f itself
    int H;
    TokenLayout lay;     // used when dense == 0
    int dense;           // sequence tensors are [B][H][N][d]: token strides are the compile-time dk, dv
    int* flag;           // null, or set to 1 when a gate product falls below the floor of the reciprocals
    // Runs of a sequence.  R > 0: run r of sequence s is chunks cuts.bnd[r] .. bnd[r + 1] - 1 and the workgroup
    // numbered s R + r takes it, after a light walk over the chunks before it.
    int R;
    FwdCuts cuts;
    // Otherwise (TokenLayout::seg > 1), with `run_add` set: the state entering run r of sequence s is
    //   Diag(decay_{r-1}) ( ... Diag(decay_0) h0[s] + add_0 ... ) + add_{r-1},
    // run_add [s (seg - 1) + j][dk][dv], run_decay [s (seg - 1) + j][dk], j = 0 .. seg - 2.
    // (run_add null: h0 holds the state entering every run, one per run.)  Spans of a packed batch: entry
    // span * H + head is what the span adds to the last of its sequences, which goes on in later spans.
    float* run_add;
    float* run_decay;
    int walkers;         // sequences (runs of segmented ones, spans x heads) that get a workgroup, or R of them, each for NSPLIT slabs of dv
    int ends_per_seq;    // run_ends_kernel: how many of a sequence's runs are walked, the first ones
};

constexpr int fused_waves(int dk) { return dk == 128 ? 8 : 4; }

template <int DK_, int DVW_> struct FwdFusedLds {
    static constexpr int DK = DK_, DVW = DVW_, C = kChunk, NW = fused_waves(DK);   // DVW: dv columns of one workgroup
    // Row pitches in elements.  Tiles read row-major with 16-byte vectors want consecutive rows
    // 4 banks apart (+8 elements); tiles read with transpose loads (4 rows x 64 bytes per half
    // wave) want them 16 banks apart (+32 elements).
    static constexpr int PQ = DK + 8, PT = C + 8, PV = DVW + 32, PC = C + 8, PO = DVW + 8;
    static constexpr size_t qm = 0;                                     // Q~    [2][C][PQ], columns in fragment order
    static constexpr size_t km = qm + (size_t)2 * C * PQ * 2;           // K~^T  [2][DK][PT]
    static constexpr size_t vm = km + (size_t)2 * DK * PT * 2;          // V     [C][PV]
    static constexpr size_t pm = vm + (size_t)C * PV * 2;               // P   [C][PC]
    static constexpr size_t sb = pm + (size_t)C * PC * 2;               // G_m S_n, bf16, fragment order
    static constexpr bool late_qs = (C / 32) * (DVW / 32) < NW;         // see LATE_QS
    static constexpr int NSB = late_qs ? 2 : 1;                         // copies of the published state
    static constexpr size_t ost = sb + (size_t)NSB * DK * DVW * 2;      // O   [C][PO]
    static constexpr size_t tot = ost + (size_t)C * PO * 2;             // [8][DK] fp32 block totals + one row of ones
    static constexpr size_t ca = tot + (size_t)(kRowBlocks + 1) * DK * 4;    // [DK] fp32 state rescale
    static constexpr size_t ch = ca + (size_t)DK * 4;                   // [DK] fp32 h of the chunk before (grouped walks)
    static constexpr size_t cr = ch + (size_t)DK * 4;                   // [DK] fp32 r of a chunk that ends its sequence
    static constexpr size_t total = cr + (size_t)DK * 4;
    static_assert(total * (8 / NW) <= 160 * 1024, "LDS budget of the workgroups of a compute unit");
    // light walk (the same memory, before the walk proper)
    static constexpr size_t lk = 0;                                     // K^^T  [2][DK][PT]
    static constexpr size_t lv = lk + (size_t)2 * DK * PT * 2;          // V     [2][C][PV]
    static constexpr size_t lt = lv + (size_t)2 * C * PV * 2;           // [2][8][DK] fp32 block totals, then a row of ones
    static constexpr size_t lg = lt + (size_t)(2 * kRowBlocks + 1) * DK * 4;   // [2][DK] fp32 whole-chunk gate product
    static constexpr size_t light_total = lg + (size_t)2 * DK * 4;
    static_assert(light_total <= total, "the light walk fits the tiles of the walk proper");
};

// One chunk of the walk: tokens row0 .. row0 + C - 1 of a sequence of N tokens whose first token is
// token tok0 of the packed tensors (grouped walks; 0 otherwise).  N = 0: a pass past the end.
// `slot` is the chunk's place in an array with one entry per chunk of the batch (the kept states).
// Row r of the chunk stands for token row0 + r of the sequence where lo <= row0 + r < hi and for no
// token elsewhere (past the end of the sequence; in the small-gate modes, outside the chunk's middle
// rows: ChunkRows).
struct FusedChunk {
    int tok0, row0, N, bh, first, last, slot, lo, hi;
};
// What a walk over spans keeps of a chunk while it is in the window of its passes (scalar registers, of which it
// has too few): the rest of FusedChunk is computed from it.  n: chunk of sequence e.
struct SpanChunk {
    int tok0, N, n, e, slot;
};

// GROUPED: a span of a packed batch's chunks (else: a sequence, or a run of one).  ENDS: only the state
// that a run leaves when it starts from zero, and the product of its gates (run_ends_kernel).  RUNS: the
// workgroup may own a run that does not start with the sequence, and an odd number of chunks ends in
// a single pass of its own; without it the chunk loop always takes an even number of passes (a pass
// over a chunk past the end sees gates equal to one and is an exact no-op), which costs short odd walks
// a pass and saves long ones registers (128 sequences of 2048 tokens: 92.4 against 95.9 us).
// EXACT_END: the state a sequence ends in is wanted.  It is used on (decoding starts from it), and most of it is
// what the last few tokens add, whose 1 - f is exact in bf16 for bf16 gates of 0.5 and more, but K~ = (1 - f) G_m / G
// is not.  The products of a sequence's last chunk are therefore factored around G_m r instead of G_m, with
// r = h 2^-e in [1, 2): Q~ / r, K~ r, r G_m S_n, and 2^e for h.  K~ r is the product of the later gates times a power of
// two, so that it rounds as K^ = k prod_{s > j} f_s does (error of the final state against 64 bits, 32 heads of 1024
// tokens, gates from 0.5 to 1: 1.66e-3 -> 1.27e-3; up to 0.9 us a call, which calls without hT do not pay).
template <int DK, int DV, int DVW, bool GATE_BF16, bool DENSE, bool GROUPED, bool ENDS, bool RUNS = true, bool EXACT_END = false>
__device__ __forceinline__ void fwd_fused_body(const FwdFusedParams& p)
{
    static_assert(!(DENSE && GROUPED), "spans are a feature of packed batches");
    typedef __bf16 T;
    typedef Mma<T> M;
    typedef typename M::frag frag;
    typedef FwdFusedLds<DK, DVW> L;
    constexpr int NSPLIT = DV / DVW, C = L::C, NW = L::NW, NT = 64 * NW, RW = C / kRowBlocks;
    constexpr int PQ = L::PQ, PT = L::PT, PV = L::PV, PC = L::PC, PO = L::PO;
    constexpr int NBT = DVW / 32, NKS = DK / 16;
    constexpr int NST = (DK / 32) * NBT / NW;        // state tiles per wave: 2 (128 x 128) or 1
    constexpr int NOT = (C / 32) * NBT;              // output tiles of the workgroup: waves 0 .. NOT-1 own one
    constexpr int PW0 = (NOT == NW) ? 0 : NOT;       // first of the three waves that compute the P blocks
    // With 64 dv columns per workgroup of eight waves only four own an output tile; their read-out of
    // the incoming state, Q~ (G_m S_n), is then issued one stage late, in stage A of the next pass,
    // next to the P blocks the other waves compute there (the published state is double-buffered
    // for that, and O(n) leaves in stage B of pass n+1).  This evens out the matrix work of the
    // two stages.
    constexpr bool LATE_QS = L::late_qs;
    // With the smaller register footprint of the 64-column variants (and of bf16 gates), every MFMA chain requests all its
    // operand fragments first and the instruction scheduler is told not to sink those loads back
    // between the MFMAs: one LDS latency per chain instead of one per k-step pair.
    constexpr bool BATCH_LOADS = (DVW == 64) && GATE_BF16;
    constexpr int KB8 = BATCH_LOADS ? DK / 16 : 2, KB4 = BATCH_LOADS ? kChunk / 16 : 1;   // k-steps per batch
    static_assert(RW == 8 && NST * NW == (DK / 32) * NBT && NOT <= NW && PW0 + 3 <= NW, "tile/wave mapping");

    extern __shared__ __align__(16) char smem[];
    T* Qm = reinterpret_cast<T*>(smem + L::qm);
    T* Km = reinterpret_cast<T*>(smem + L::km);
    T* Vm = reinterpret_cast<T*>(smem + L::vm);
    T* Pm = reinterpret_cast<T*>(smem + L::pm);
    T* Sb = reinterpret_cast<T*>(smem + L::sb);
    T* Ost = reinterpret_cast<T*>(smem + L::ost);
    float* tot = reinterpret_cast<float*>(smem + L::tot);
    float* cA = reinterpret_cast<float*>(smem + L::ca);
    float* cH = reinterpret_cast<float*>(smem + L::ch);
    float* cR = reinterpret_cast<float*>(smem + L::cr);

    if (not_chosen(p.lay)) return;       // one of several chunk lengths, and not the one called for
    // workgroup -> (sequence, run, dv half): ids 8 apart land on the same XCD (ids are dealt to the 8
    // XCDs round-robin), so the workgroups of a sequence share an L2 for the rows several of them read (run_item())
    int bh, split, run = 0;
    const int n_run = (GROUPED || !RUNS || p.R == 0) ? 1 : p.R;
    if (NSPLIT == 1 && n_run == 1) { bh = blockIdx.x; split = 0; }
    else {
        const RunItem item = run_item(blockIdx.x, p.walkers, n_run * NSPLIT);
        bh = item.seq;
        split = item.sub % NSPLIT; run = item.sub / NSPLIT;
    }
    // padding of the grid (uniform, before any barrier)
    int ends_slot = bh;
    if constexpr (ENDS && !GROUPED) {
        // the first ends_per_seq of the seg runs of every sequence
        const int whole = bh / p.ends_per_seq;
        if (whole * p.lay.seg >= p.BH) return;
        bh = whole * p.lay.seg + (bh - whole * p.ends_per_seq);
    } else {
        if (bh >= (GROUPED ? p.lay.spans * p.lay.H : p.BH)) return;
    }
    const int* t_start = p.lay.vl;
    const int* t_len = p.lay.vl + (p.lay.B + 1);
    const int* t_before = p.lay.vl + 2 * (p.lay.B + 1);
    // GROUPED: the span is chunks p0 .. p1 - 1 of head `head`, counted over the sequences in order; it
    // starts with chunk cur_n of sequence cur_e
    int head = 0, cur_e = 0, cur_n = 0, span_id = 0;
    bool span_ends = false;                  // the spans' contributions are there
    SeqView sv;
    int NC;                                  // chunks of the walk
    int n0 = 0;                              // its first chunk, within the sequence (not GROUPED)
    if constexpr (GROUPED) {
        span_id = bh / p.lay.H;
        head = bh - span_id * p.lay.H;
        // addresses are formed from token numbers: the view is the head's slice of the whole tensor
        sv.off_k = (size_t)head * p.lay.sh_k; sv.off_v = (size_t)head * p.lay.sh_v; sv.chunk0 = 0;
        sv.N = 0; sv.NC = 0;
        const int total = table_read(t_before, p.lay.B);
        const int p0 = (int)((long long)span_id * total / p.lay.spans), p1 = (int)((long long)(span_id + 1) * total / p.lay.spans);
        NC = p1 - p0;
        span_ends = p.run_add && table_read(p.lay.span_walks, 0) != 0;
        if (ENDS && !span_ends) return;
        if (NC > 0) {
            // the sequence that holds chunk p0 (ENDS: the span's last chunk): the last one with at most
            // that many chunks before it
            const int at = ENDS ? p1 - 1 : p0;
            // (64 table entries a step, one per lane: every step waits for memory before the first chunk is
            // requested; against a bisection, 32 sequences of 512 tokens 75.8 -> 74.5 us, 256 of 64 96.7 -> 95.0)
            int lo = 0, hi = p.lay.B;        // invariant: before[lo] <= at < before[hi]
            while (hi - lo > 1) {
                const int stride = (hi - lo + 63) >> 6, i = lo + ((int)(threadIdx.x & 63) + 1) * stride;
                const bool below = i < hi && t_before[i] <= at;
                const int c = __builtin_amdgcn_readfirstlane(__popcll(__ballot(below)));
                hi = min(hi, lo + (c + 1) * stride);
                lo += c * stride;
            }
            cur_e = lo;
            const int before = table_read(t_before, lo);
            cur_n = max(p0 - before, 0);
            if constexpr (ENDS) {
                // that sequence's chunks inside the span, if it goes on in the next one
                if (table_read(t_before, lo + 1) == p1) return;
                NC = p1 - before - cur_n;
            }
        }
    } else {
        bh = sequence_of_workgroup<DENSE>(p.lay, bh);
        if constexpr (ENDS) { if (!DENSE && p.lay.vl) ends_slot = bh; }
        sv = seq_view<DENSE, DK, DV, true>(p.lay, p.N, p.NC, bh);
        NC = sv.NC;
        if (RUNS && n_run > 1) { n0 = p.cuts.bnd[run]; NC = p.cuts.bnd[run + 1] - n0; }
        head = bh / p.lay.seg % p.H;
    }
    // the sequence whose entries of h0 and hT the walk starts from and ends in
    const int whole = (RUNS && !ENDS && !GROUPED && p.run_add) ? bh / p.lay.seg : bh;
    const int dv0 = split * DVW;             // first dv column of this workgroup
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave index, in a scalar register
    // element-wise work: this lane's row block (of 8) and channel pair
    const int rb = (DK == 128) ? w : 2 * w + g, cl = (DK == 128) ? lane : r32;
    const int wrow = (C / NW) * w;           // first row of the wave
    const size_t seq_k = sv.off_k, seq_v = sv.off_v;
    const int ld_k = DENSE ? DK : (int)p.lay.sn_k, ld_v = DENSE ? DV : (int)p.lay.sn_v;   // token stride, elements
    const T* qg = static_cast<const T*>(p.q);
    const T* vg = static_cast<const T*>(p.v);
    T* og = static_cast<T*>(p.o);
    const int rt = w / NBT, bt = w % NBT;    // output tile (rt, bt) of this wave, if w < NOT
    const int at0 = NST * (w / NBT);         // its state tiles: (at0 .. at0 + NST - 1, bt)
    const bool has_o = (NOT == NW) || w < NOT;
    const bool is_p = w >= PW0 && w < PW0 + 3;
    const bool after = w >= NW / 2;          // rows of this wave lie after the mid-chunk reference

    // a sequence without tokens ends in the state it starts from
    auto pass_state_on = [&](int seq) {
        if (p.hT)
            for (int idx = tid; idx < DK * DVW; idx += NT) {
                const size_t e = (size_t)seq * DK * DV + (size_t)(idx / DVW) * DV + dv0 + idx % DVW;
                p.hT[e] = p.h0 ? p.h0[e] : 0.0f;
            }
    };
    if constexpr (GROUPED) {
        // (such sequences lie in no span: they are dealt out by their number)
        for (int e = ENDS ? p.lay.B : span_id; e < p.lay.B; e += p.lay.spans)
            if (table_read(t_len, e) == 0) pass_state_on(e * p.lay.H + head);
        if (NC == 0) return;                 // (uniform early exit, before any barrier)
    } else if (NC == 0) {
        if constexpr (!ENDS) pass_state_on(bh);
        return;
    }

    // ---- the chunks of the walk, in order.  Spans step through the sequences with a cursor that runs
    // three chunks ahead of the pass (everything here is wave-uniform).
    int cur_nc = 0, cur_tok = 0, cur_N = 0, cur_slot = 0, left = NC;
    auto open_sequence = [&](int e) {
        cur_e = e;
        cur_N = table_read(t_len, e); cur_nc = p.lay.chunks_of(cur_N); cur_tok = table_read(t_start, e);
        // the chunks of (sequence, head) lie together, the heads of a sequence one after the other
        cur_slot = table_read(t_before, e) * p.lay.H + head * cur_nc;
    };
    auto next_chunk = [&]() {
        SpanChunk c;
        if (left <= 0) {                     // past the end of the span, for good
            c.tok0 = 0; c.N = 0; c.n = 0; c.e = 0; c.slot = 0;
            return c;
        }
        c.tok0 = cur_tok; c.N = cur_N; c.n = cur_n; c.e = cur_e; c.slot = cur_slot + cur_n;
        if (--left > 0 && ++cur_n == cur_nc) {
            int e = cur_e + 1;
            while (table_read(t_len, e) == 0) ++e;       // (left > 0: a later sequence has tokens)
            open_sequence(e);
            cur_n = 0;
        }
        return c;
    };
    const int N_one = sv.N;
    auto chunk_at = [&](int c) {             // chunk c of the workgroup's sequence; rows of chunks outside the walk stand for no token
        FusedChunk k;
        const ChunkRows cr = chunk_rows(p.lay.sub, c, N_one);
        const bool in = !RUNS || (c >= n0 && c < n0 + NC);
        k.tok0 = 0; k.row0 = cr.tok0; k.lo = cr.first; k.hi = in ? cr.end : cr.first;
        k.N = N_one; k.bh = bh; k.first = c == 0; k.last = c == NC - 1; k.slot = sv.chunk0 + c;
        return k;
    };
    // window of the pass: ck[j] = chunk n - 1 + j of pass n (spans only)
    SpanChunk ck[5];
    const int first_n = cur_n;               // the span starts with this chunk of its first sequence
    int first_tok = 0, first_N = 0, first_bh = bh;
    if constexpr (GROUPED) {
        open_sequence(cur_e);
        first_tok = cur_tok; first_N = cur_N; first_bh = cur_e * p.lay.H + head;
        ck[0].tok0 = 0; ck[0].N = 0; ck[0].n = 0; ck[0].e = 0; ck[0].slot = 0;
#pragma unroll
        for (int j = 1; j < 5; ++j) ck[j] = next_chunk();
    }
    auto span_chunk = [&](const SpanChunk& s) {
        FusedChunk k;
        const ChunkRows cr = chunk_rows(p.lay.sub, s.n, s.N);
        k.tok0 = s.tok0; k.row0 = cr.tok0; k.lo = cr.first; k.hi = cr.end; k.N = s.N; k.bh = s.e * p.lay.H + head;
        k.first = s.n == 0 && s.N > 0; k.last = s.n == p.lay.chunks_of(s.N) - 1; k.slot = s.slot;
        return k;
    };
    auto chunk_rel = [&](int n, int rel) { return GROUPED ? span_chunk(ck[rel + 1]) : chunk_at(n0 + n + rel); };

    // ---- state: fp32 accumulators.  Between chunks they hold S_n / h(n-1); see stage A. ----
    f32x16 accS[NST];
    // Element (tile j, register v) of this lane in a [dk][dv] fp32 state: a wave-uniform address
    // (sequence, tile, group of four registers) plus one per-lane 32-bit byte offset plus a small
    // constant, so that no access needs an address register of its own.
    const uint32_t st_lane = (uint32_t)(4 * g * DV + dv0 + 32 * bt + r32) * 4u;
    auto state_rows = [&](const float* base, int seq, int j, int c) {
        return reinterpret_cast<const char*>(base) + ((size_t)seq * DK * DV + (size_t)(32 * (at0 + j) + 8 * c) * DV) * 4;
    };
    auto initial_state = [&](int seq) {
#pragma unroll
        for (int j = 0; j < NST; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const char* rows = state_rows(p.h0, seq, j, c);
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    accS[j][4 * c + jj] = p.h0 ? *reinterpret_cast<const float*>(rows + st_lane + jj * DV * 4) : 0.0f;
            }
    };
    // accumulators *= per-channel factors in LDS (channel = accumulator row)
    auto scale_state = [&](const float* factor) {
#pragma unroll
        for (int j = 0; j < NST; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 cm = *reinterpret_cast<const f32x4*>(factor + 32 * (at0 + j) + 8 * c + 4 * g);
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) accS[j][4 * c + jj] *= cm[jj];
            }
    };
    // the state after the chunk before: scale * accumulators, formed in place (what follows either
    // replaces the accumulators or is the end of the walk)
    auto final_state = [&](int seq, const float* scale) {
        scale_state(scale);
#pragma unroll
        for (int j = 0; j < NST; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                char* rows = const_cast<char*>(state_rows(p.hT, seq, j, c));
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) *reinterpret_cast<float*>(rows + st_lane + jj * DV * 4) = accS[j][4 * c + jj];
            }
    };
    if constexpr (ENDS) {
#pragma unroll
        for (int j = 0; j < NST; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) accS[j][v] = 0.0f;
    } else {
        initial_state(GROUPED ? first_bh : whole);
        if (RUNS && (GROUPED ? span_ends : p.run_add != nullptr)) {
            // what the runs before this one add, and how their gates decay what enters them
            int k0 = 0, k1 = bh - whole * p.lay.seg;
            if constexpr (GROUPED) {
                // the spans from the one in which the span's first sequence starts
                k1 = k0 = span_id;
                if (first_n > 0) {
                    const int total = table_read(t_before, p.lay.B), before = table_read(t_before, first_bh / p.lay.H);
                    while (k0 > 0 && (int)((long long)k0 * total / p.lay.spans) > before) --k0;
                }
            }
            // (the values come from other XCDs: what a request takes is most of what a run costs, so
            // several runs' are requested at a time)
            constexpr int AHEAD = NST == 1 ? 4 : 2;
            for (int k = k0; k < k1; k += AHEAD) {
                f32x4 dm[AHEAD][NST][4];
                float a[AHEAD][NST][16];
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const int ku = min(k + u, k1 - 1);
                    const int slot = GROUPED ? ku * p.lay.H + head : whole * (p.lay.seg - 1) + ku;
                    const float* dec = p.run_decay + (size_t)slot * DK;
#pragma unroll
                    for (int j = 0; j < NST; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            dm[u][j][c] = *reinterpret_cast<const f32x4*>(dec + 32 * (at0 + j) + 8 * c + 4 * g);
                            const char* rows = state_rows(p.run_add, slot, j, c);
#pragma unroll
                            for (int jj = 0; jj < 4; ++jj) a[u][j][4 * c + jj] = *reinterpret_cast<const float*>(rows + st_lane + jj * DV * 4);
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    if (k + u >= k1) break;
#pragma unroll
                    for (int j = 0; j < NST; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) accS[j][v] = fmaf(dm[u][j][v >> 2][v & 3], accS[j][v], a[u][j][v]);
                }
            }
        }
    }
    const f32x2 beta_pair = p.beta ? *reinterpret_cast<const f32x2*>(p.beta + (size_t)head * DK + 2 * cl) : f32x2{0.0f, 0.0f};
    float hprev0 = 1.0f, hprev1 = 1.0f;      // h of the previous chunk, channels 2*cl, 2*cl+1 (wave 0 only)

    // ---- row fetch, two chunks ahead, two register sets ----
    RawRows<RW> rawf[2], rawq[2];
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int VPR = DVW / 8;             // 16-byte vectors per V / O row
    constexpr int NVV = C * VPR / NT;        // vectors per thread
    constexpr int VRS = 64 / VPR;            // rows one wave covers per vector
    // V: two chunks ahead too, in alternating sets, where the registers allow it (fp32 gates take
    // twice the prefetch registers of bf16 ones; V is then fetched one chunk ahead)
    constexpr int VD = GATE_BF16 ? 2 : 1;
    u32x4 rawv[VD][NVV];
    const int vrow = wrow + lane / VPR, vcol = 8 * (lane % VPR);      // V copy: 16 bytes per lane, rows vrow (+ VRS)
    // Every load is issued unconditionally (a row past the end of the sequence re-reads the last
    // row), and the chunk loop takes two chunks per turn, so that its body is straight-line code:
    // the compiler can then count outstanding loads exactly and the two register sets never have
    // to be copied.  Row addresses are wave-uniform.
    const char* fbase = static_cast<const char*>(p.f) + seq_k * (GATE_BF16 ? 2 : 4);
    const char* qbase = reinterpret_cast<const char*>(qg + seq_k);
    const char* vbase = reinterpret_cast<const char*>(vg + seq_v + dv0);
    auto load_f = [&](RawRows<RW>& d, const FusedChunk& c) {
        load_block_rows<DK == 64, RW, GATE_BF16>(d, fbase + (size_t)c.tok0 * ((size_t)ld_k * (GATE_BF16 ? 2 : 4)), c.row0 + wrow,
                                           max(c.N - 1, 0), ld_k, lane);
    };
    auto load_q = [&](RawRows<RW>& d, const FusedChunk& c) {
        load_block_rows<DK == 64, RW, true>(d, qbase + (size_t)c.tok0 * ((size_t)ld_k * 2), c.row0 + wrow, max(c.N - 1, 0), ld_k, lane);
    };
    auto load_v = [&](u32x4 (&d)[NVV], const FusedChunk& c) {
        const int row0 = c.row0 + wrow, last_row = max(c.N - 1, 0);
        const char* vb = vbase + (size_t)c.tok0 * ((size_t)ld_v * 2);
#pragma unroll
        for (int j = 0; j < NVV; ++j) {
            const int rc = min(max(row0 + lane / VPR + VRS * j, 0), last_row);
            d[j] = *reinterpret_cast<const u32x4*>(vb + (size_t)rc * ((size_t)ld_v * 2) + 2 * vcol);
        }
    };
    // Rows past the end of the sequence need no masking here: their K~ is zero (f = 1 there), so
    // whatever finite values stand in for them never reach a stored output or the state.
    auto store_v = [&](const u32x4 (&s)[NVV]) {
#pragma unroll
        for (int j = 0; j < NVV; ++j) *reinterpret_cast<u32x4*>(Vm + (vrow + VRS * j) * PV + vcol) = s[j];
    };

    // ---- element-wise work of one chunk, split around the exchange of the block totals ----
    // With a = inclusive gate product from the start of this wave's 8-row block, z = exclusive
    // product to its end, t = a z the block total, mid = product of the blocks between this block
    // and the mid-chunk reference row, and m = product of the gates between the reference row and
    // this row:
    //   rows after the reference:  Q~ = q m,   K~ = k / m,   m = mid a,  1/m = z / (mid t)
    //   rows before it:            Q~ = q / m, K~ = k m,     m = mid z,  1/m = a / (mid t)
    // so Q~ = (q a) s_a and K~ = (k z) s_z with per-channel block factors s_a, s_z in {mid,
    // 1/(mid t)}: one reciprocal per channel and block, floored so that it stays finite outside
    // the supported gate range.
    // First half (before the totals are exchanged): q a, k z, t.
    float qa0[RW], qa1[RW], kz0[RW], kz1[RW], bt0, bt1;
    float below_floor = 1.0f;            // smallest product a reciprocal was taken of (reported once, at the end)
    auto prep_gates = [&](const RawRows<RW>& rf_raw, const RawRows<RW>& rq_raw, const FusedChunk& c) {
        f32x2 rf[RW];
        convert_rows<RW>(rf, rf_raw, c.row0 + RW * rb, c.hi, true, GATE_BF16, 1.0f, c.lo);
        if (p.beta) gate_rows<RW>(rf, beta_pair, true, c.row0 + RW * rb, c.hi, c.lo);
        float run0 = 1.0f, run1 = 1.0f;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const uint32_t u = __float_as_uint(rq_raw.r[i].x);
            run0 *= rf[i].x; run1 *= rf[i].y;
            qa0[i] = __uint_as_float(u << 16) * run0;
            qa1[i] = __uint_as_float(u & 0xffff0000u) * run1;
        }
        bt0 = run0; bt1 = run1;
        run0 = 1.0f; run1 = 1.0f;
#pragma unroll
        for (int i = RW - 1; i >= 0; --i) {      // k z = (1 - f) z = z_i - z_{i-1}
            const float n0 = run0 * rf[i].x, n1 = run1 * rf[i].y;
            kz0[i] = run0 - n0; kz1[i] = run1 - n1;
            run0 = n0; run1 = n1;
        }
        *reinterpret_cast<f32x2*>(tot + rb * DK + 2 * cl) = f32x2{bt0, bt1};
    };
    // x = significand(x) power_of_two(x) for normal numbers (h is 2^-100 to 1 in the gate domain)
    auto significand = [](float x) { return __uint_as_float((__float_as_uint(x) & 0x7fffffu) | 0x3f800000u); };
    auto power_of_two = [](float x) { return __uint_as_float(__float_as_uint(x) & 0xff800000u); };
    // Second half: block factors from the exchanged totals, tiles to LDS.
    auto prep_tiles = [&](int c, bool starts_sequence, bool ends) {      // c: only its parity matters (which tile buffer)
        // product of the (at most three) block totals between this block and the reference row;
        // an absent factor reads the row of ones
        const float* ones = tot + kRowBlocks * DK;
        const float* r1 = after ? (rb > 4 ? tot + 4 * DK : ones) : (rb < 3 ? tot + 3 * DK : ones);
        const float* r2 = after ? (rb > 5 ? tot + 5 * DK : ones) : (rb < 2 ? tot + 2 * DK : ones);
        const float* r3 = after ? (rb > 6 ? tot + 6 * DK : ones) : (rb < 1 ? tot + 1 * DK : ones);
        const f32x2 m1 = *reinterpret_cast<const f32x2*>(r1 + 2 * cl);
        const f32x2 m2 = *reinterpret_cast<const f32x2*>(r2 + 2 * cl);
        const f32x2 m3 = *reinterpret_cast<const f32x2*>(r3 + 2 * cl);
        const float mid0 = m1.x * m2.x * m3.x, mid1 = m1.y * m2.y * m3.y;
        const float R0 = fast_rcp(fmaxf(mid0 * bt0, kTinyProduct));
        const float R1 = fast_rcp(fmaxf(mid1 * bt1, kTinyProduct));
        below_floor = fminf(below_floor, fminf(mid0 * bt0, mid1 * bt1));
        float sa0 = after ? mid0 : R0, sa1 = after ? mid1 : R1;             // multiplies q a
        float sz0 = after ? R0 : mid0, sz1 = after ? R1 : mid1;             // multiplies k z
        if (EXACT_END && ends) {
            f32x2 h = {1.0f, 1.0f};
#pragma unroll
            for (int i = kRowBlocks / 2; i < kRowBlocks; ++i) {
                const f32x2 t = *reinterpret_cast<const f32x2*>(tot + i * DK + 2 * cl);
                h.x *= t.x; h.y *= t.y;
            }
            const float e0 = significand(h.x), e1 = significand(h.y);
            sz0 *= e0; sz1 *= e1;
            sa0 *= fast_rcp(e0); sa1 *= fast_rcp(e1);
            if (rb == 0) *reinterpret_cast<f32x2*>(cR + 2 * cl) = f32x2{e0, e1};
        }
        // Q~: row-major, channel pair (2l, 2l+1) at column position sigma(2l) (bits 2 and 3 swapped);
        // K~^T: this thread's 8 tokens of each of its two channels as one 16-byte vector
        const int qcol = ((2 * cl) & ~12) | (((2 * cl) & 4) << 1) | (((2 * cl) & 8) >> 1);
        T* Qd = Qm + (size_t)(c & 1) * C * PQ + (size_t)(RW * rb) * PQ + qcol;
        T* Kd = Km + (size_t)(c & 1) * DK * PT + (size_t)(2 * cl) * PT + RW * rb;
        float k0[RW], k1[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            store_pair_t<T>(Qd, (size_t)i * PQ, qa0[i] * sa0, qa1[i] * sa1);
            k0[i] = kz0[i] * sz0; k1[i] = kz1[i] * sz1;
        }
        *reinterpret_cast<frag*>(Kd) = M::pack(k0);
        *reinterpret_cast<frag*>(Kd + PT) = M::pack(k1);
        // state rescale of the chunk, by wave 0: h of the previous chunk times G_m of this one
        if (w == 0) {
            f32x2 t[kRowBlocks];
#pragma unroll
            for (int i = 0; i < kRowBlocks; ++i) t[i] = *reinterpret_cast<const f32x2*>(tot + i * DK + 2 * cl);
            const float gm0 = (t[0].x * t[1].x) * (t[2].x * t[3].x), gm1 = (t[0].y * t[1].y) * (t[2].y * t[3].y);
            if constexpr (GROUPED) {
                // the state of a sequence's first chunk is its initial state, not what the walk carries;
                // and h alone turns the carried accumulators into the state a sequence ends in
                *reinterpret_cast<f32x2*>(cH + 2 * cl) = f32x2{hprev0, hprev1};
                if (starts_sequence) { hprev0 = 1.0f; hprev1 = 1.0f; }
            }
            *reinterpret_cast<f32x2*>(cA + 2 * cl) = f32x2{hprev0 * gm0, hprev1 * gm1};
            hprev0 = (t[4].x * t[5].x) * (t[6].x * t[7].x); hprev1 = (t[4].y * t[5].y) * (t[6].y * t[7].y);
            if (EXACT_END && ends) { hprev0 = power_of_two(hprev0); hprev1 = power_of_two(hprev1); }
        }
    };

    // O leaves with non-temporal stores (this library does not read it.  us, ordinary -> non-temporal: 32 x 16 heads of 128, 2048 tokens, six
    // sets of buffers in turn 235 -> 228, inputs just written 235 -> 239, o read and written by a kernel right behind 331 -> 331; training pair of 8 x 16
    // heads 262 -> 261, 8 x 32 heads of 64 273 -> 270) through registers that stay reserved for the whole pass (see the end of stage B):
    // a global store reads its data registers late, and overwriting them earlier would make the
    // wave wait for the store, and with it for every prefetch issued before it, to complete.
    u32x4 obuf[C * VPR / NT];
    auto store_o = [&](const FusedChunk& c) {
#pragma unroll
        for (int k = 0; k < C * VPR / NT; ++k) {
            const int idx = tid + k * NT;
            const int row = idx / VPR, cv = idx % VPR;
            const int grow = c.row0 + row;
            obuf[k] = *reinterpret_cast<const u32x4*>(Ost + (size_t)row * PO + cv * 8);
            if (grow >= c.lo && grow < c.hi)       // also false for the chunk "-1" of the first pass
                __builtin_nontemporal_store(obuf[k], reinterpret_cast<u32x4*>(og + seq_v + ((size_t)c.tok0 + grow) * ld_v + dv0 + cv * 8));
        }
    };


    // ---- light walk: the recurrence alone over chunks c0 .. c1 - 1 of one sequence (N tokens from token
    // tok0 of the packed tensors), in place in the accumulators, which hold the true state before and
    // after:  S <- Diag(g) S + K^^T V,  K^_j = k_j prod_{s > j in chunk} f_s  (no quotients).  One
    // barrier per chunk: pass n writes the tiles of chunk n and the block totals of chunk n + 1, and
    // after the barrier multiplies while the other waves go on to the next pass.  The LDS pipe is what
    // a pass waits for (about 1 us; rows fetched four chunks ahead instead of two change nothing); an
    // odd number of chunks starts with a pass over a chunk without tokens, which keeps the code small
    // (a short walk meets most of it cold).
    auto light_walk = [&](int tok0, int N, int c0, int c1, float* decay_out) {
        T* Kl = reinterpret_cast<T*>(smem + L::lk);
        T* Vl = reinterpret_cast<T*>(smem + L::lv);
        float* tl = reinterpret_cast<float*>(smem + L::lt);
        float* gl = reinterpret_cast<float*>(smem + L::lg);
        const float* ones = tl + 2 * kRowBlocks * DK;
        constexpr int AH = 2;
        RawRows<RW> lf[AH];
        u32x4 lv[AH][NVV];
        float kz0[RW], kz1[RW], t0, t1, dec0 = 1.0f, dec1 = 1.0f;
        auto at = [&](int c) {
            FusedChunk k;
            const ChunkRows cr = chunk_rows(p.lay.sub, c, N);
            k.tok0 = tok0; k.row0 = cr.tok0; k.lo = cr.first; k.hi = (c >= c0 && c < c1) ? cr.end : cr.first; k.N = N;
            k.bh = 0; k.first = 0; k.last = 0; k.slot = 0;
            return k;
        };
        auto gates = [&](const RawRows<RW>& raw, const FusedChunk& c, int par) {
            f32x2 rf[RW];
            convert_rows<RW>(rf, raw, c.row0 + RW * rb, c.hi, true, GATE_BF16, 1.0f, c.lo);
            if (p.beta) gate_rows<RW>(rf, beta_pair, true, c.row0 + RW * rb, c.hi, c.lo);
            float run0 = 1.0f, run1 = 1.0f;
#pragma unroll
            for (int i = RW - 1; i >= 0; --i) {
                const float n0 = run0 * rf[i].x, n1 = run1 * rf[i].y;
                kz0[i] = run0 - n0; kz1[i] = run1 - n1;
                run0 = n0; run1 = n1;
            }
            t0 = run0; t1 = run1;
            *reinterpret_cast<f32x2*>(tl + (par * kRowBlocks + rb) * DK + 2 * cl) = f32x2{t0, t1};
        };
        auto pass = [&](auto SET, int n) {
            constexpr int set = decltype(SET)::value, par = set & 1;
            float post0 = 1.0f, post1 = 1.0f;
#pragma unroll
            for (int i = 1; i < kRowBlocks; ++i) {
                const float* src = (i > rb) ? tl + (par * kRowBlocks + i) * DK : ones;
                const f32x2 t = *reinterpret_cast<const f32x2*>(src + 2 * cl);
                post0 *= t.x; post1 *= t.y;
            }
            if (rb == 0) {
                *reinterpret_cast<f32x2*>(gl + par * DK + 2 * cl) = f32x2{post0 * t0, post1 * t1};
                dec0 *= post0 * t0; dec1 *= post1 * t1;
            }
            float k0[RW], k1[RW];
#pragma unroll
            for (int i = 0; i < RW; ++i) { k0[i] = kz0[i] * post0; k1[i] = kz1[i] * post1; }
            T* Kd = Kl + (size_t)par * DK * PT + (size_t)(2 * cl) * PT + RW * rb;
            *reinterpret_cast<frag*>(Kd) = M::pack(k0);
            *reinterpret_cast<frag*>(Kd + PT) = M::pack(k1);
#pragma unroll
            for (int j = 0; j < NVV; ++j)
                *reinterpret_cast<u32x4*>(Vl + (size_t)par * C * PV + (vrow + VRS * j) * PV + vcol) = lv[set][j];
            load_v(lv[set], at(n + AH));
            gates(lf[(set + 1) % AH], at(n + 1), 1 - par);
            load_f(lf[(set + 1) % AH], at(n + 1 + AH));
            __syncthreads();
            scale_state(gl + par * DK);
            const T* Kc = Kl + (size_t)par * DK * PT;
#pragma unroll
            for (int ks = 0; ks < C / 16; ++ks) {
                const frag vf = M::load_kmajor(Vl + (size_t)par * C * PV, PV, 16 * ks, 32 * bt, lane);
#pragma unroll
                for (int j = 0; j < NST; ++j) M::mma(accS[j], M::load(Kc + (32 * (at0 + j) + r32) * PT + 16 * ks + 8 * g), vf);
            }
        };
        if (tid < DK) tl[2 * kRowBlocks * DK + tid] = 1.0f;
        const int n0 = c1 - ((c1 - c0 + 1) & ~1);
        load_f(lf[0], at(n0)); load_v(lv[0], at(n0));
        load_f(lf[1], at(n0 + 1)); load_v(lv[1], at(n0 + 1));
        gates(lf[0], at(n0), 0);
        load_f(lf[0], at(n0 + AH));
        __syncthreads();
        for (int n = n0; n < c1; n += 2) {
            pass(std::integral_constant<int, 0>(), n);
            pass(std::integral_constant<int, 1>(), n + 1);
        }
        if (decay_out && rb == 0) *reinterpret_cast<f32x2*>(decay_out + 2 * cl) = f32x2{dec0, dec1};
        __syncthreads();                     // the tiles make room for those of the walk proper
    };
    if constexpr (ENDS) {
        light_walk(first_tok, GROUPED ? first_N : N_one, first_n, first_n + NC, split == 0 ? p.run_decay + (size_t)ends_slot * DK : nullptr);
#pragma unroll
        for (int j = 0; j < NST; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                char* rows = const_cast<char*>(state_rows(p.run_add, ends_slot, j, c));
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) *reinterpret_cast<float*>(rows + st_lane + jj * DV * 4) = accS[j][4 * c + jj];
            }
        return;
    }
    if (RUNS && !(GROUPED && span_ends) && (GROUPED ? first_n > 0 : n0 > 0)) {
        light_walk(first_tok, GROUPED ? first_N : N_one, 0, GROUPED ? first_n : n0, nullptr);
        // Keeps the compiler from computing the chunk loop's lane-dependent values ahead of the light
        // walk and carrying them through it in registers.
        int opaque = lane;
        asm volatile("" : "+v"(opaque));
    }

    // ---- prologue: rows of chunks 0 and 1 in flight, element-wise work of chunk 0 ----
    // the never-written block of P (rows 0..31 x columns 32..63) must read as zero
    for (int idx = tid; idx < 32 * 32; idx += NT) Pm[(idx >> 5) * PC + 32 + (idx & 31)] = (T)0.0f;
    if (tid < DK) tot[kRowBlocks * DK + tid] = 1.0f;
    load_f(rawf[0], chunk_rel(0, 0)); load_q(rawq[0], chunk_rel(0, 0)); load_v(rawv[0], chunk_rel(0, 0));
    load_f(rawf[1], chunk_rel(0, 1)); load_q(rawq[1], chunk_rel(0, 1));
    if (VD == 2) load_v(rawv[VD - 1], chunk_rel(0, 1));
    prep_gates(rawf[0], rawq[0], chunk_rel(0, 0));
    load_f(rawf[0], chunk_rel(0, 2)); load_q(rawq[0], chunk_rel(0, 2));
    __syncthreads();
    // whether chunk n + rel of the walk ends its sequence and the state is wanted
    const bool ends_here = EXACT_END && !GROUPED && (!RUNS || (p.run_add ? bh - whole * p.lay.seg == p.lay.seg - 1 : run == n_run - 1));
    auto ends = [&](int n, int rel) { return GROUPED ? span_chunk(ck[rel + 1]).last != 0 : (ends_here && n + rel == NC - 1); };
    prep_tiles(0, true, ends(0, 0));
    __syncthreads();

    // output tile accumulator, transposed: accO[v] = O[token 32 rt + r32][channel 32 bt + 8 (v/4) + 4 g + v%4]
    f32x16 accO;
#pragma unroll
    for (int v = 0; v < 16; ++v) accO[v] = 0.0f;
    // (all operand fragments are requested before the first MFMA, so that one LDS latency is paid,
    // not one per k-step)
    auto read_out_state = [&](const T* Qx, const T* Sx) {        // accO += ((G_m S)^T Q~^T) tile (bt, rt)
#pragma unroll
        for (int k0 = 0; k0 < NKS; k0 += KB8) {
            frag sa[KB8], qa[KB8];
#pragma unroll
            for (int k = 0; k < KB8; ++k) {
                const int ks2 = k0 + k;
                sa[k] = *reinterpret_cast<const frag*>(Sx + state_frag_offset(ks2 >> 1, bt, NBT, ks2 & 1, lane));
                qa[k] = M::load(Qx + (32 * rt + r32) * PQ + 16 * ks2 + 8 * g);
            }
            if (BATCH_LOADS) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < KB8; ++k) M::mma(accO, sa[k], qa[k]);
        }
    };
    auto stage_o = [&]() {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            bf16x4 pk;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) pk[jj] = (T)accO[4 * c + jj];
            *reinterpret_cast<bf16x4*>(Ost + (size_t)(32 * rt + r32) * PO + 32 * bt + 8 * c + 4 * g) = pk;
        }
    };
    auto pin_obuf = [&]() {
#pragma unroll
        for (int k = 0; k < C * VPR / NT; ++k) asm volatile("" :: "v"(obuf[k]));
    };

    // The published state holds, per lane, 8 channels of one dv column (the read-out contracts over
    // the channels).  A backward pass contracts over dv and wants 8 dv columns of one channel per
    // lane: the same bf16 values, regrouped by LDS transpose reads -- 16 lanes fetch 4 consecutive
    // channels of 4 dv columns each and get back 4 dv columns of one channel -- and written to
    // global memory as fragments (tile (channel tile, dv tile), half, lane) of 16 bytes per lane.
    constexpr int NSF = (DK / 32) * NBT * 2 / NW;        // fragments per wave and chunk
    auto save_state = [&](const T* Sx, int slot) {
        typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
        T* dst = static_cast<T*>(p.save) + (size_t)slot * DK * DV;
        const int i16 = lane & 15;
        const int m = ((lane & 16) >> 2) + (i16 & 3);    // which 4 channels of the tile's 32 this lane fetches
        const int hs = m >> 2, q4 = (m >> 1) & 1, gs = m & 1;
#pragma unroll
        for (int j = 0; j < NSF; ++j) {
            const int id = w * NSF + j, half = id & 1, tb = (id >> 1) % NBT, ta = (id >> 1) / NBT;
            const int dl = 32 * tb + 16 * half + 4 * g + (i16 >> 2);        // local dv column this lane fetches (first read)
            const T* src = Sx + state_frag_offset(ta, tb, NBT, hs, 32 * gs + (dl & 31)) + 4 * q4;
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(src));
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(src + 8 * 8));   // dv column + 8: lane + 8
            const frag out = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4, out), reinterpret_cast<u32x4*>(dst + state_frag_offset(ta, dv0 / 32 + tb, DV / 32, half, lane)));
        }
    };

    auto chunk = [&](auto PAR, int n) {
        constexpr int par = decltype(PAR)::value;
        const T* Qc = Qm + (size_t)par * C * PQ;
        const T* Kc = Km + (size_t)par * DK * PT;
        T* Sp = Sb + (LATE_QS ? (size_t)par * DK * DVW : 0);      // where this pass publishes G_m(n) S_n
        // ======================= stage A =======================
        if (!LATE_QS) store_o(chunk_rel(n, -1));
        store_v(rawv[VD == 2 ? par : 0]);
        load_v(rawv[VD == 2 ? par : 0], chunk_rel(n, VD));
        if constexpr (GROUPED) {
            // sequence boundary: the walk's accumulators, times h of the chunk before, are the state
            // the sequence before ends in; this chunk starts from its own sequence's initial state
            const FusedChunk before = chunk_rel(n, -1), here = chunk_rel(n, 0);
            if (before.last && p.hT) final_state(before.bh, cH);
            if (here.first && n > 0) initial_state(here.bh);
        }
        // G_m(n) S_n = c(n) * accumulators, published as the bf16 operand of the read-out
        auto publish = [&]() {
#pragma unroll
            for (int j = 0; j < NST; ++j) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    float x[8];
#pragma unroll
                    for (int s = 0; s < 8; ++s) x[s] = accS[j][8 * half + s];
                    *reinterpret_cast<frag*>(Sp + state_frag_offset(at0 + j, bt, NBT, half, lane)) = M::pack(x);
                }
            }
        };
        scale_state(cA);
        if (EXACT_END && ends(n, 0) && !p.save) scale_state(cR);
        publish();
        prep_gates(rawf[1 - par], rawq[1 - par], chunk_rel(n, 1));
        load_f(rawf[1 - par], chunk_rel(n, 3)); load_q(rawq[1 - par], chunk_rel(n, 3));
        if (LATE_QS) {
            // O(n-1) is completed here: its P V part was accumulated in stage B of the previous pass
            if (has_o) {
                read_out_state(Qm + (size_t)(1 - par) * C * PQ, Sb + (size_t)(1 - par) * DK * DVW);
                stage_o();
            }
            pin_obuf();
        }
        // P^T blocks (J <= I), one per wave
        if (is_p) {
            const int pb = w - PW0;
            const int I = (pb == 0) ? 0 : 1, J = (pb == 2) ? 1 : 0;   // 0:(0,0) 1:(0,1) 2:(1,1) as (J,I)
            f32x16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
            // K~ operand: lane (token 32 J + r32, g) needs the channels of k-step ks in fragment order,
            // 16 ks + 4 g + {0..3} and 16 ks + 8 + 4 g + {0..3}: two transpose reads of K~^T rows
            typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
            const int i16 = lane & 15;
            const T* kp = Kc + (size_t)(4 * g + (i16 >> 2)) * PT + 32 * J + (lane & 16) + 4 * (i16 & 3);
#pragma unroll
            for (int k0 = 0; k0 < NKS; k0 += KB8) {
                frag ka[KB8], qf[KB8];
#pragma unroll
                for (int k = 0; k < KB8; ++k) {
                    const int ks = k0 + k;
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(kp + (size_t)(16 * ks) * PT));
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(kp + (size_t)(16 * ks + 8) * PT));
                    ka[k] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    qf[k] = M::load(Qc + (32 * I + r32) * PQ + 16 * ks + 8 * g);
                }
                if (BATCH_LOADS) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < KB8; ++k) M::mma(acc, ka[k], qf[k]);     // acc[row j][col i]
            }
            const int i_glob = 32 * I + r32;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int j0 = 32 * J + 8 * c + 4 * g;
                float x[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) x[jj] = (j0 + jj <= i_glob) ? acc[4 * c + jj] : 0.0f;
                bf16x4 pk;
                pk[0] = (T)x[0]; pk[1] = (T)x[1]; pk[2] = (T)x[2]; pk[3] = (T)x[3];
                *reinterpret_cast<bf16x4*>(Pm + (size_t)i_glob * PC + j0) = pk;
            }
        }
        __syncthreads();
        // ======================= stage B =======================
        // O^T tile (bt, rt) = V^T P^T + (G_m S)^T Q~^T   and   accumulators += K~^T V
        if (LATE_QS) store_o(chunk_rel(n, -1));
        if (p.save && n < NC) {
            save_state(Sp, chunk_rel(n, 0).slot);
            if (EXACT_END && ends(n, 0)) {       // (kept states are G_m S_n whatever the chunk: r comes once they are out)
                __syncthreads();
                scale_state(cR);
                publish();
                __syncthreads();
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) accO[v] = 0.0f;
#pragma unroll
        for (int k0 = 0; k0 < C / 16; k0 += KB4) {
            frag vf[KB4], kf[KB4][NST], pf[KB4];
#pragma unroll
            for (int k = 0; k < KB4; ++k) {
                const int ks = k0 + k;
                vf[k] = M::load_kmajor(Vm, PV, 16 * ks, 32 * bt, lane);
#pragma unroll
                for (int j = 0; j < NST; ++j) kf[k][j] = M::load(Kc + (32 * (at0 + j) + r32) * PT + 16 * ks + 8 * g);
                if (has_o) pf[k] = M::load(Pm + (32 * rt + r32) * PC + 16 * ks + 8 * g);   // zero block included
            }
            if (BATCH_LOADS) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < KB4; ++k) {
#pragma unroll
                for (int j = 0; j < NST; ++j) M::mma(accS[j], kf[k][j], vf[k]);
                if (has_o) M::mma(accO, vf[k], pf[k]);
            }
        }
        if (!LATE_QS) read_out_state(Qc, Sp);
        prep_tiles(n + 1, chunk_rel(n, 1).first != 0, ends(n, 1));
        if (!LATE_QS) {
            if (has_o) stage_o();
            pin_obuf();
        }
        if constexpr (GROUPED) {             // the window moves on by one chunk
#pragma unroll
            for (int j = 0; j < 4; ++j) ck[j] = ck[j + 1];
            ck[4] = next_chunk();
        }
        __syncthreads();
    };

    int n_end = 0;
    for (; RUNS ? n_end + 1 < NC : n_end < NC; n_end += 2) {
        chunk(std::integral_constant<int, 0>(), n_end);
        chunk(std::integral_constant<int, 1>(), n_end + 1);
    }
    if (RUNS && n_end < NC) { chunk(std::integral_constant<int, 0>(), n_end); ++n_end; }
    if (LATE_QS && n_end == NC) {
        // the last chunk is still without its state read-out (a pass over an empty chunk has done it)
        if (has_o) {
            read_out_state(Qm + (size_t)((NC - 1) & 1) * C * PQ, Sb + (size_t)((NC - 1) & 1) * DK * DVW);
            stage_o();
        }
        __syncthreads();
    }
    if (!LATE_QS || n_end == NC) store_o(chunk_rel(n_end, -1));

    if (p.flag && below_floor < kTinyProduct) *p.flag = 1;
    if (p.hT) {
        // S_N = pending rescale * accumulators (the chunk after the last one has G_m = 1).  A span has
        // written the state of every sequence that a further pass followed.
        if constexpr (GROUPED) {
            const FusedChunk before = span_chunk(ck[0]);
            if (before.last) final_state(before.bh, cH);
        } else {
            if (!RUNS || (p.run_add ? bh - whole * p.lay.seg == p.lay.seg - 1 : run == n_run - 1)) final_state(whole, cA);
        }
    }
}

// (a workgroup of four waves shares a compute unit with another: two waves per SIMD either way)
template <int DK, int DV, int DVW, bool GATE_BF16, bool RUNS, bool EXACT_END>
__global__ __launch_bounds__(64 * fused_waves(DK), 2) void fwd_fused_kernel(FwdFusedParams p)
{
    if (p.dense) fwd_fused_body<DK, DV, DVW, GATE_BF16, true, false, false, RUNS, EXACT_END>(p);
    else         fwd_fused_body<DK, DV, DVW, GATE_BF16, false, false, false, RUNS, EXACT_END>(p);
}

// The walk over spans of a packed batch's chunks (a kernel of its own: its register needs are not
// those of the walk over one sequence).
template <int DK, int DV, int DVW, bool GATE_BF16, bool EXACT_END>
__global__ __launch_bounds__(64 * fused_waves(DK), 2) void fwd_fused_grouped_kernel(FwdFusedParams p)
{
    fwd_fused_body<DK, DV, DVW, GATE_BF16, false, true, false, true, EXACT_END>(p);
}

// What every run of a sequence (every span of a packed batch) adds to the state from zero, and the
// product of its gates.
template <int DK, int DV, int DVW, bool GATE_BF16>
__global__ __launch_bounds__(64 * fused_waves(DK), 2) void run_ends_kernel(FwdFusedParams p)
{
    if (p.lay.vl && p.lay.spans > 0) fwd_fused_body<DK, DV, DVW, GATE_BF16, false, true, true>(p);
    else if (p.dense) fwd_fused_body<DK, DV, DVW, GATE_BF16, true, false, true>(p);
    else         fwd_fused_body<DK, DV, DVW, GATE_BF16, false, false, true>(p);
}

static bool fused_grouped(const SeqDims& d) { return d.lay.vl && d.lay.spans > 0; }

// (heads of 64 so many that 16 rows are more than an int apart, 524288 with fp32 gates, take sweep and read-out)
bool fwd_fused_supported(const SeqDims& d) { return d.io_bf16 && (d.dk != 64 || halves_near<8>(d.lay.sn_k, d.gate_bf16 ? 2 : 4)); }

typedef void (*FusedKernel)(FwdFusedParams);

template <int DK, int DV, int DVW, bool GATE_BF16>
static FusedKernel fused_kernel(bool ends, bool grouped, bool runs, bool exact_end)
{
    if (ends) return run_ends_kernel<DK, DV, DVW, GATE_BF16>;
    if (grouped) return exact_end ? fwd_fused_grouped_kernel<DK, DV, DVW, GATE_BF16, true> : fwd_fused_grouped_kernel<DK, DV, DVW, GATE_BF16, false>;
    if (runs) return exact_end ? fwd_fused_kernel<DK, DV, DVW, GATE_BF16, true, true> : fwd_fused_kernel<DK, DV, DVW, GATE_BF16, true, false>;
    // (the walk that takes many 128 x 128 sequences whole is bound by its registers and never had the exact end)
    constexpr bool EXACT = DK != 128 || DV != 128;
    return exact_end ? fwd_fused_kernel<DK, DV, DVW, GATE_BF16, false, EXACT> : fwd_fused_kernel<DK, DV, DVW, GATE_BF16, false, false>;
}

template <int DK, int DV, int DVW>
static hipError_t launch_fused(const SeqDims& d, const FwdFusedParams& p, bool ends, hipStream_t stream)
{
    typedef FwdFusedLds<DK, DVW> L;
    constexpr int NSPLIT = DV / DVW;
    // (walks of a few, odd chunks: the pass over an empty chunk that the other variant takes would be felt)
    const bool runs = p.R > 0 || p.run_add || (d.NC < 16 && d.NC % 2 == 1), grouped = fused_grouped(d), exact_end = p.hT != nullptr;
    const FusedKernel kern = d.gate_bf16 ? fused_kernel<DK, DV, DVW, true>(ends, grouped, runs, exact_end)
                                         : fused_kernel<DK, DV, DVW, false>(ends, grouped, runs, exact_end);
    const int lds = (int)(ends ? L::light_total : L::total);
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    const int per = NSPLIT * (p.R > 0 ? p.R : 1);
    const unsigned grid = per == 1 ? (unsigned)p.walkers : (unsigned)run_grid(p.walkers, per);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * L::NW), lds, stream, p);
    return hipGetLastError();
}

static hipError_t launch_fused_dims(const SeqDims& d, FwdFusedParams& p, int walkers, bool ends, hipStream_t stream)
{
    p.walkers = walkers;
    // Two workgroups per walk (each half of the dv columns) keep twice as many compute units busy,
    // but only as long as all of them run at once (144 sequences of 2048 tokens, 128-wide heads: 137 us
    // halved against 84 us whole; up to 128 sequences halving wins).
    const int all = walkers * (p.R > 0 ? p.R : 1);
    if (d.dk == 128 && d.dv == 128)
        return 2 * all > 256 ? launch_fused<128, 128, 128>(d, p, ends, stream)
                             : launch_fused<128, 128, 64>(d, p, ends, stream);
    if (d.dk == 64 && d.dv == 64) return launch_fused<64, 64, 64>(d, p, ends, stream);
    if (d.dk == 128 && d.dv == 64) return launch_fused<128, 64, 64>(d, p, ends, stream);
    if (d.dk == 64 && d.dv == 128) return launch_fused<64, 128, 64>(d, p, ends, stream);
    return hipErrorInvalidValue;
}

static FwdFusedParams fused_params(const SeqDims& d, const void* q, const void* f, const void* v)
{
    FwdFusedParams p;
    p.q = q; p.f = f; p.v = v; p.h0 = nullptr; p.o = nullptr; p.hT = nullptr; p.save = nullptr;
    p.N = d.N; p.NC = d.NC; p.BH = d.BH; p.beta = d.beta; p.H = d.H; p.lay = d.lay; p.dense = d.dense() ? 1 : 0;
    p.flag = d.domain_flag;
    p.R = 0; p.run_add = nullptr; p.run_decay = nullptr; p.walkers = 0; p.ends_per_seq = 1;
    return p;
}

FwdRuns plan_fwd_runs(const SeqDims& d, bool light_walks, bool kept)
{
    if (!d.io_bf16 || d.packed) { FwdRuns r; r.run_chunks = d.NC; return r; }
    return plan_fwd_runs(d.BH, d.NC, d.dk, d.dv, light_walks, kept);
}

hipError_t launch_fwd_fused(const SeqDims& d, const void* q, const void* f, const void* v, const float* h0,
                            void* o, float* hT, void* save_states, hipStream_t stream, int light_runs, const float* run_add,
                            const float* run_decay)
{
    if (d.BH == 0) return hipSuccess;
    FwdFusedParams p = fused_params(d, q, f, v);
    p.h0 = h0; p.o = o; p.hT = hT; p.save = save_states;
    if (light_runs > 1) {
        p.R = light_runs;
        fused_cuts(d.NC, p.R, &p.cuts);
    }
    p.run_add = const_cast<float*>(run_add); p.run_decay = const_cast<float*>(run_decay);
    return launch_fused_dims(d, p, fused_grouped(d) ? d.lay.spans * d.lay.H : d.BH, false, stream);
}

hipError_t launch_run_ends(const SeqDims& d, int ends_per_seq, const void* q, const void* f, const void* v, float* run_add,
                           float* run_decay, hipStream_t stream)
{
    if (d.BH == 0 || ends_per_seq <= 0) return hipSuccess;
    FwdFusedParams p = fused_params(d, q, f, v);
    p.run_add = run_add; p.run_decay = run_decay; p.ends_per_seq = ends_per_seq;
    return launch_fused_dims(d, p, fused_grouped(d) ? d.lay.spans * d.lay.H : d.BH / d.lay.seg * ends_per_seq, true, stream);
}

}   // namespace hgrn2
