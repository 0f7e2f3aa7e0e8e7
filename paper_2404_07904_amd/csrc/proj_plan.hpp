// The tiles and shares of the projections' products: plain host arithmetic on a few sizes, in a header of its own so that it can
// be compiled and checked without a GPU.
#pragma once

namespace hgrn2 {

// Which tile a product takes, and (fp32 result) into how many shares its contraction is cut: by what they take, us, fitted to 100 to
// 16384 tokens at widths 256 to 2048.  256 x 256 has the best rate but needs 256 tiles to fill the chip; 128 x 128 finds two
// places on a compute unit, and so does 64 x 64, which has the shortest steps where a few workgroups have to do (a step
// is 1.5 / 1.1 / 0.45 us with all places taken, 1.1 / 0.45 / 0.26 us on a unit of its own).
// 575 tokens of width 1024, 256 / 128 / 64: projection 26.7 / 12.4 / 12.2 us, dx 59 / 28 / 17; 2048 tokens, projection 27.6 / 20.1 / 29.3;
// 16384 tokens, projection 94 / 119 / 214; width 2048 322 / 419 / 702.  (The constants of 256 are from before the projections' tiles were walked,
// which takes up to 10% off several tiles to a workgroup: 8192 tokens of width 1024 take 128, 60.2, where 256 takes 53.5.)
struct NtPlan { int tile, splits; };
inline double nt_time(int tile, long long tiles, double steps)
{
    if (tile == 256) {
        const long long rest = tiles % 256;
        return 3.5 + (double)(tiles / 256) * (1.5 * steps + 10.0) + (rest == 0 ? 0.0 : rest <= 192 ? 1.1 * steps + 9.0 : 1.5 * steps + 10.0);
    }
    const double full = tile == 128 ? 1.12 : 0.45, most = tile == 128 ? 0.95 : 0.45, half = tile == 128 ? 0.45 : 0.26, end = tile == 128 ? 2.0 : 1.0;
    const long long rest = tiles % 512;
    return 3.5 + (double)(tiles / 512) * (full * steps + end) + (rest == 0 ? 0.0 : (rest <= 256 ? half : most) * steps + end);
}
inline NtPlan plan_nt(int M, int N, int K, bool may_split)
{
    NtPlan best = {256, 1};
    double least = 1e30;
    const int steps = K / 64;
    for (int tile = 64; tile <= 256; tile *= 2) {
        // (fp32 results take 192 rows instead of 256: 3 d rows are a multiple of both, and 32 x 8 tiles fill the chip at width 2048 where 24 x 8 do not)
        const int rows = tile == 256 && may_split ? 192 : tile;
        const long long tiles = (long long)((M + rows - 1) / rows) * (N / tile);
        for (int s = 1; s <= 16 && (s == 1 || (may_split && steps >= 8 * s)); s *= 2) {
            // (the shares are written and read once more, and added up by a launch of their own)
            const double share_mb = 4e-6 * M * (double)N * s;
            if (s > 1 && share_mb > 64.0) break;
            const double t = nt_time(tile, tiles * s, (double)steps / s) * (rows == 192 ? 0.8 : 1.0) + (s > 1 ? 4.0 + share_mb * 0.5 : 0.0);
            if (t < least) { least = t; best = NtPlan{tile, s}; }
        }
    }
    return best;
}

// Element-wise pass of the reverse mode: columns of a workgroup, and its tokens: 64, or 32 while there are few (a workgroup's
// batches wait for memory one after the other: 204 tokens of width 256 in 128s 10.2 us, in 32s 5.4).
constexpr int kActCols = 256;
inline int act_rows(int M, int d) { return (long long)(3 * d / kActCols) * ((M + 63) / 64) < 256 ? 32 : 64; }

}   // namespace hgrn2
