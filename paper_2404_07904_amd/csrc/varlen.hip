// Variable-length batches: B sequences packed back to back along the token axis.  The kernels
// find a sequence's tokens and its slots in the per-chunk workspaces through a small device table
// (TokenLayout::vl) that this kernel builds from the caller's cumulative sequence lengths:
//
//   table[0 .. B]            first token of sequence b            (entry B: end of the last one)
//   table[B+1 .. 2B+1]       length of sequence b                 (entry B: 0)
//   table[2B+2 .. 3B+2]      chunks of the sequences before b     (entry B: chunks of all)
//   table[3B+3 .. 4B+3]      the sequences ordered by falling length (entry B unused)
// The last array is for the kernels that give a whole sequence to one workgroup: workgroups start
// in index order, so handing out the longest sequences first keeps the longest one from being the
// last to start (for more than kSortMax sequences the order is left as it is).
//
// The offsets are clamped to [0, T] and replaced by their running maximum, so the table always
// describes disjoint, ordered pieces of the T tokens, whatever the caller's array holds: a wrong
// array gives wrong results, never an access outside the tensors or the workspaces.
#include "common.hpp"
#include "kernels.hpp"

namespace hgrn2 {

constexpr int kTabThreads = 256;
constexpr int kSortMax = 8192;
constexpr int kSortLds = 2048;
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Group g of G starts at the first entry e whose chunks-before count reaches g / G of all chunks
// (bisection over the table's non-decreasing third array); the last group ends at the last entry,
// so that empty entries at the end belong to a group too.  Behind the G + 1 group starts: the choice
// between the two backward passes, then, for each of the G equal spans of chunks the walks over spans
// take, the entry the span ends in, then two ints: whether the forward walk's spans, the reverse walk's spans
// carry the state over spans by walks from zero (TokenLayout::span_walks).
// (Called by all threads of a one-workgroup kernel, after a barrier that follows the table's writes.)
// `before`: the table's third array, or the caller's copy of it in LDS.
template <typename Before>
__device__ __forceinline__ void build_groups(Before before, int n_entries, int G, int* groups, int heads64)
{
    const long long total = before[n_entries];
    for (int grp = threadIdx.x; grp <= G; grp += kTabThreads) {
        int first = n_entries;
        if (grp < G) {
            int lo = -1, hi = n_entries;                 // invariant: before[lo] G < grp total <= before[hi] G
            const long long want = (long long)grp * total;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if ((long long)before[mid] * G >= want) hi = mid; else lo = mid;
            }
            first = hi;
        }
        groups[grp] = first;
    }
    __syncthreads();
    // Which backward pass of a stateless call.  The reverse walk gives every workgroup a span of total / G chunks of a
    // head and has it first walk, at a quarter of the cost, the chunks between the end of its span and the end of the sequence
    // the span ends in, or add up what walks from zero found there; the other pass takes two sweeps, as long as the longest
    // sequence, then the per-chunk kernel.  The walk is chosen while the longest such tail is at most four spans long: where the two met
    // before the walk took 7 us a chunk.  It is ahead on the other side of the line too by now; us, walk / other pass, 16 heads,
    // 16384 tokens, one document of 4 and of 8 spans among short ones: 128 x 128 386 / 468 and 534 / 658, 64 x 64 274 / 333 and 455 / 512,
    // 128 x 64 318 / 356 and 488 / 518, 64 x 128 297 / 431 and 446 / 601.
    int tail = 0, head = 0;
    for (int s = threadIdx.x; s < G; s += kTabThreads) {
        const long long p0 = (long long)s * total / G, p1 = (long long)(s + 1) * total / G;
        if (p1 <= p0) { groups[G + 2 + s] = 0; continue; }
        int lo = 0, hi = n_entries;                      // invariant: before[lo] <= p1 - 1 < before[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (before[mid] <= p1 - 1) lo = mid; else hi = mid;
        }
        groups[G + 2 + s] = lo;                          // the sequence span s ends in
        const int after = (int)(before[lo + 1] - p1);    // chunks of sequence `lo` after the span's last one
        tail = max(tail, after);
        if (after > 0) head = max(head, (int)(p1 - before[lo]));          // and before the next span's first one
    }
    // The longest of all, over the waves' longest.
    __shared__ int longest[2][kTabThreads / 64];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { tail = max(tail, __shfl_xor(tail, d, 64)); head = max(head, __shfl_xor(head, d, 64)); }
    if ((threadIdx.x & 63) == 0) { longest[0][threadIdx.x >> 6] = tail; longest[1][threadIdx.x >> 6] = head; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 1; j < kTabThreads / 64; ++j) { tail = max(tail, longest[0][j]); head = max(head, longest[1][j]); }
        const long long share = (total + G - 1) / G;
        groups[G + 1] = (tail <= 4 * share) ? 1 : 0;
        // Walks from zero take a span's chunks, and some more for the states they leave; light walks the chunks of a
        // sequence outside a span.  us, walks from zero / light, 16384 tokens, spans of 16, 16 heads, that many chunks outside a span:
        //   128 x 128  forward 24: 97 to 100 / 103, 32: 96 / 112      backward 20: 200 / 189, 32: 186 to 201 / 200 to 208, 48: 198 / 234
        //    64 x 64   forward 24: 67 / 70, 32: 67 / 75               backward 16: 89 / 88, 20: 91 / 93, 32: 90 / 105
        //   128 x 64   forward 24: 78 / 79, 32: 78 / 84               backward 20: 149 / 120, 32: 137 to 140 / 134 to 143, 48: 141 / 152
        //    64 x 128  forward 24: 78 to 81 / 75 to 80, 32: 78 / 80   backward 20: 144 / 119, 32: 131 / 134, 48: 135 / 152
        // Over 392 batches of 4 to 64 heads and 8192 to 32768 tokens what is chosen takes 1% more than the better of the two, forward of heads of
        // 64 x 128 2.7% (spans of 32: light walks are ahead up to 64 chunks outside, 133 / 151).
        // (Fewer chunks than spans: spans without one leave nothing.)
        groups[2 * G + 2] = (total >= G && head > share + 9) ? 1 : 0;
        groups[2 * G + 3] = (total >= G && tail > (heads64 ? share / 3 + 2 : share + 8)) ? 1 : 0;
    }
}

__global__ __launch_bounds__(kTabThreads) void varlen_groups_kernel(const int* tab, int n_entries, int G, int* groups,
                                                                    int heads64, const int* choice, int path)
{
    if (choice && table_read(choice, 0) != path) return;        // one of several alternatives, and not the one called for
    build_groups(tab + 2 * (n_entries + 1), n_entries, G, groups, heads64);
}

// Exclusive prefix (sum, or running maximum of non-negative values) of one value per thread over the
// workgroup: inside a wave by shuffles, across the waves through `wave_tot` (one int per wave).
template <bool MAX>
__device__ __forceinline__ int block_prefix(int v, int* wave_tot)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d, 64);
        if (lane >= d) inc = MAX ? max(inc, o) : inc + o;
    }
    __syncthreads();                    // (the previous use of wave_tot is over)
    if (lane == 63) wave_tot[w] = inc;
    __syncthreads();
    int before = 0;
    for (int j = 0; j < w; ++j) before = MAX ? max(before, wave_tot[j]) : before + wave_tot[j];
    int exc = __shfl_up(inc, 1, 64);
    if (lane == 0) exc = 0;
    return MAX ? max(before, exc) : before + exc;
}

// With `groups` (null: none) the group array of the table is built in the same launch.
// What the one workgroup takes is the chain of trips to memory: with up to kSortLds sequences (LDS) every array is also kept in LDS, where
// the later steps read it, and the one trip left is the one that fetches `cu`.  Up to kSortMax the lengths are, for the order.  (21 sequences, 16 groups, with the profiler's 5 us a launch: 9.4 -> 7.2 us, forward of 21 sequences in 16384 tokens 93.7 -> 91.2, of 500 151 -> 121, of 2048 801 -> 302, of 2049 1396 -> 334).
template <bool LDS>
__global__ __launch_bounds__(kTabThreads) void varlen_table_kernel(const int* cu, int B, int T, int* tab, int G, int* groups, int heads64,
                                                                   int sub, const int* choice, int path)
{
    if (choice && table_read(choice, 0) != path) return;        // one of several alternatives, and not the one called for
    const int shift = 31 - __builtin_clz((unsigned)sub);         // sub is a power of two
    __shared__ int wave_tot[kTabThreads / 64];
    __shared__ __align__(16) int slen[(LDS ? kSortLds : kSortMax) + 4];
    __shared__ int sstart[LDS ? kSortLds + 4 : 1], sbefore[LDS ? kSortLds + 4 : 1];
    const int n = B + 1, tid = threadIdx.x;
    const int per = (n + kTabThreads - 1) / kTabThreads;
    const int lo = min(tid * per, n), hi = min(lo + per, n);      // this thread's entries
    auto clamped = [&](int i) { return min(max(cu[i], 0), T); };
    auto start_of = [&](int i) { if constexpr (LDS) return sstart[i]; else return tab[i]; };
    const bool sorted = LDS || B <= kSortMax;

    // starts: running maximum of the clamped offsets
    int m = 0;
    for (int i = lo; i < hi; ++i) m = max(m, clamped(i));
    int run = block_prefix<true>(m, wave_tot);
    for (int i = lo; i < hi; ++i) {
        run = max(run, clamped(i));
        tab[i] = run;
        if constexpr (LDS) sstart[i] = run;
    }
    if (sorted)
        for (int j = n + tid; j < ((n + 3) & ~3); j += kTabThreads) slen[j] = -1;      // padding never counts
    __syncthreads();                                              // starts of the neighbouring slices are visible

    // lengths, and the chunk counts before every sequence
    int c = 0;
    for (int i = lo; i < hi; ++i) {
        const int len = i < B ? start_of(i + 1) - start_of(i) : 0;
        tab[n + i] = len;
        if (sorted) slen[i] = i < B ? len : -1;
        c += (len + sub - 1) >> shift;
    }
    run = block_prefix<false>(c, wave_tot);
    for (int i = lo; i < hi; ++i) {
        tab[2 * n + i] = run;
        if constexpr (LDS) sbefore[i] = run;
        run += ((LDS ? (i < B ? slen[i] : 0) : tab[n + i]) + sub - 1) >> shift;
    }
    __syncthreads();                                              // all lengths are visible

    // order by falling length: the rank of sequence b is the number of sequences that come before
    // it (longer, or as long with a smaller index), counted directly in LDS, four at a time: with whole vectors before b
    // counting from its own length on and the others above it, what is missing is equal lengths before b in its own vector
    int* order = tab + 3 * n;
    for (int b = tid; b < B; b += kTabThreads) {
        int rank = b;
        if (sorted) {
            const int mine = slen[b];
            rank = 0;
#pragma unroll 4
            for (int j = 0; j < B; j += 4) {
                const i32x4 l = *reinterpret_cast<const i32x4*>(slen + j);
                const int above = j + 4 <= b ? mine - 1 : mine;
#pragma unroll
                for (int e = 0; e < 4; ++e) rank += l[e] > above ? 1 : 0;
            }
            for (int e = b & ~3; e < b; ++e) rank += slen[e] == mine ? 1 : 0;
        }
        order[rank] = b;
    }
    if (groups) {
        __syncthreads();
        if constexpr (LDS) build_groups((const int*)sbefore, B, G, groups, heads64);
        else build_groups((const int*)(tab + 2 * n), B, G, groups, heads64);
    }
}

// Long sequences of a packed batch are walked in runs of at most `run_chunks` chunks: the kernels
// then get a table whose entries are the runs (same four arrays, R entries, those past the last
// run empty), in which a run is a sequence like any other; only the carried states know which
// runs make up a sequence, through first_run[b] = number of runs of the sequences before b
// (B + 1 entries).  Runs are whole chunks, so the chunk counts of the run table add up as those of
// the sequence table do.  The runs keep their order (no sorting by length: none is long).
__global__ __launch_bounds__(kTabThreads) void varlen_run_table_kernel(const int* seq_tab, int B, int T, int run_chunks,
                                                                       int R, int* run_tab, int* first_run, int sub,
                                                                       const int* choice, int path)
{
    if (choice && table_read(choice, 0) != path) return;
    const int shift = 31 - __builtin_clz((unsigned)sub);         // sub is a power of two
    __shared__ int part[kTabThreads];
    const int n = B + 1, tid = threadIdx.x;
    const int per = (n + kTabThreads - 1) / kTabThreads;
    const int lo = min(tid * per, n), hi = min(lo + per, n);
    const int* start = seq_tab;
    const int* len = seq_tab + n;
    const int* before = seq_tab + 2 * n;
    auto runs_of = [&](int b) {
        const int nc = b < B ? (len[b] + sub - 1) >> shift : 0;
        return (nc + run_chunks - 1) / run_chunks;
    };
    int c = 0;
    for (int b = lo; b < hi; ++b) c += runs_of(b);
    part[tid] = c;
    __syncthreads();
    int first = 0;
    for (int j = 0; j < tid; ++j) first += part[j];
    const int m = R + 1, run_tokens = run_chunks * sub;
    for (int b = lo; b < hi; ++b) {
        first_run[b] = first;
        const int nr = runs_of(b);
        for (int k = 0; k < nr && first + k < R; ++k) {           // R bounds the runs of any batch of T tokens
            const int r = first + k;
            run_tab[r] = start[b] + k * run_tokens;
            run_tab[m + r] = min(run_tokens, len[b] - k * run_tokens);
            run_tab[2 * m + r] = before[b] + k * run_chunks;
            run_tab[3 * m + r] = r;
        }
        first += nr;
    }
    __syncthreads();
    const int used = min(first_run[B], R);
    for (int r = used + tid; r <= R; r += kTabThreads) {           // empty entries, and entry R of every array
        run_tab[r] = T;
        run_tab[m + r] = 0;
        run_tab[2 * m + r] = before[B];
        run_tab[3 * m + r] = r;
    }
}

// Zero fill as a kernel: a caller may have the stream under graph capture, where a memset node is
// not an option.
__global__ void zero_floats_kernel(float* dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0.0f;
}

hipError_t launch_zero_floats(float* dst, size_t n, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_floats_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, dst, n);
    return hipGetLastError();
}

// *out = src[0] + ... + src[n - 1] (a few ints)
__global__ void sum_ints_kernel(const int* src, int n, int* out)
{
    int t = 0;
    for (int i = 0; i < n; ++i) t += src[i];
    *out = t;
}

hipError_t launch_sum_ints(const int* src, int n, int* out, hipStream_t stream)
{
    hipLaunchKernelGGL(sum_ints_kernel, dim3(1), dim3(1), 0, stream, src, n, out);
    return hipGetLastError();
}

size_t varlen_table_bytes(int B) { return 4 * ((size_t)B + 1) * sizeof(int); }

hipError_t launch_varlen_table(const int* cu_seqlens, int B, int T, int* table, hipStream_t stream, int G, int* groups, bool heads64,
                               int sub, const int* choice, int path)
{
    auto kern = B <= kSortLds ? varlen_table_kernel<true> : varlen_table_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(kTabThreads), 0, stream, cu_seqlens, B, T, table, G, groups, heads64 ? 1 : 0, sub, choice, path);
    return hipGetLastError();
}

size_t varlen_groups_bytes(int G) { return (2 * (size_t)G + 4) * sizeof(int); }

hipError_t launch_varlen_groups(const int* table, int n_entries, int G, int* groups, bool heads64, hipStream_t stream, const int* choice, int path)
{
    hipLaunchKernelGGL(varlen_groups_kernel, dim3(1), dim3(kTabThreads), 0, stream, table, n_entries, G, groups, heads64 ? 1 : 0, choice, path);
    return hipGetLastError();
}

size_t varlen_run_table_bytes(int B, int R) { return varlen_table_bytes(R) + ((size_t)B + 1) * sizeof(int); }

hipError_t launch_varlen_run_table(const int* seq_table, int B, int T, int run_chunks, int R, int* run_table,
                                   int* first_run, hipStream_t stream, int sub, const int* choice, int path)
{
    hipLaunchKernelGGL(varlen_run_table_kernel, dim3(1), dim3(kTabThreads), 0, stream, seq_table, B, T, run_chunks, R,
                       run_table, first_run, sub, choice, path);
    return hipGetLastError();
}

}   // namespace hgrn2
