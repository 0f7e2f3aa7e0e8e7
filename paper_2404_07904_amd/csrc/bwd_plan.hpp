// The cut of the fused reverse walk of an equal-length batch: plain host arithmetic on a few sizes, in a header
// of its own so that it can be compiled and checked without a GPU.
#pragma once

namespace hgrn2 {

constexpr int kMaxLightRuns = 16;

// How the reverse walk cuts every sequence: into R runs.  light: run r is chunks bnd[r] .. bnd[r + 1] - 1, and its
// workgroup first takes a light walk over the chunks after it (the state gradient alone).  Otherwise runs of rc
// chunks, and the state gradients at their ends come from walks from zero over the tokens after run 0, seg_tail
// sub-runs of sub_chunks chunks (s_sub to a run), and a carry over them.
struct BwdFusedPlan { int R, rc, s_sub, sub_chunks, seg_tail, light, bnd[kMaxLightRuns + 1]; };

// places: the workgroups the runs are to fill.  0: as many as run at once; kOnePerUnit: one per compute unit and at
// least four chunks to a run (fewer run boundaries to keep); 1: sequences are not cut.
constexpr int kOnePerUnit = 256;

inline BwdFusedPlan uncut_bwd(int NC)
{
    BwdFusedPlan pl = {};
    pl.R = 1; pl.rc = NC; pl.s_sub = 1; pl.sub_chunks = NC;
    return pl;
}

// R runs with a light walk each, which costs `rho` of a chunk's full work per chunk; the cuts let all runs
// take the same time T: len_r = T - rho (NC - end_r) from the last run (len = T) backwards, so T sum_{i<R} (1 - rho)^i = NC.
// rho is the balance that measured best with the bf16 walk before the present one, and still does for heads of 128: 128 sequences of
// 32 chunks in two runs, 12 + 20 chunks 157 us, 13 + 19 152, 14 + 18 (taken) 152, 15 + 17 158; 64 chunks 27 + 37 310, 28 + 36 (taken) 307, 29 + 35 310.
// Heads of 64 x 64 would take a larger one (256 sequences of 32 chunks: 12 + 20 124 us, 14 + 18, which are taken, 130).  A light chunk alone
// costs 0.23 to 0.26 of a full one.
constexpr double kBwdLightCost = 0.24;

// longest: what the longest run takes, at `cost` a light chunk.
inline BwdFusedPlan light_bwd(int NC, int R, double cost, double* longest)
{
    BwdFusedPlan pl = {};
    double sum = 0.0, x = 1.0;
    for (int r = 0; r < R; ++r) { sum += x; x *= 1.0 - kBwdLightCost; }
    const double T = NC / sum;
    double end = NC;
    pl.bnd[R] = NC;
    for (int r = R - 1; r >= 1; --r) {
        end -= T - kBwdLightCost * (NC - end);
        int b = (int)(end + 0.5);
        if (b < r) b = r;                              // every run keeps at least one chunk
        if (b > pl.bnd[r + 1] - 1) b = pl.bnd[r + 1] - 1;
        pl.bnd[r] = b;
    }
    *longest = 0.0;
    for (int r = 0; r < R; ++r) {
        const double t = pl.bnd[r + 1] - pl.bnd[r] + cost * (NC - pl.bnd[r + 1]);
        if (t > *longest) *longest = t;
    }
    pl.light = 1; pl.R = R; pl.s_sub = 1;
    return pl;
}

// Runs of equal length whose boundaries are walked to from zero, in sub-runs of about eight chunks: fewer, longer
// walks and fewer states to carry.
inline BwdFusedPlan ends_bwd(int NC, int R)
{
    BwdFusedPlan pl = {};
    int rc = (NC + R - 1) / R;
    int s = rc / 8;
    if (s < 1) s = 1;
    if (R > 1) rc = (rc + s - 1) / s * s;              // whole sub-runs per run
    pl.rc = rc;
    pl.R = rc > 0 ? (NC + rc - 1) / rc : 1;
    if (pl.R < 1) pl.R = 1;
    pl.s_sub = s;
    pl.sub_chunks = rc / s;
    pl.seg_tail = pl.R > 1 ? (NC - rc + pl.sub_chunks - 1) / pl.sub_chunks : 0;
    return pl;
}

// What the walks take besides the full walk of their run, in chunks of it: a chunk of a light walk; the two more launches of the walks
// from zero; a megabyte of states that those write and read twice.
// Fitted with the constants of plan_bwd_runs() to 1750 timings of the bf16 walk before the present one (7.5 us a chunk of 128 x 128, 5 us of
// 64 x 64): 1 to 250 sequences of 2 to 256 chunks, gates given and formed, every cut tried at each size; the chosen cut took 0.1 to
// 0.2% more than the best on average.  With the present walk (5.9 and 3.5 us a chunk) it takes 0.3% more with heads 128 channels wide, at most 1.16
// times the best, and 1.5% with heads of 64 channels, whose light chunks now cost 0.26 of a full one: few sequences of 8 to 12 chunks are walked
// from zero where light walks would do (8 heads of 64 x 128, 8 chunks: 20.2 us, light 15.3), and 56 to 128 heads of 64 x 64 take more runs than pay
// (128 heads of 12 chunks in four 34.7, in two 29.9).
struct BwdCost { double light, ends, mb; };
inline BwdCost bwd_cost(int dk, int dv)
{
    if (dk == 64 && dv == 64) return {0.17, 0.49, 0.23};
    if (dk == 128 && dv == 128) return {0.27, 2.2, 0.055};
    if (dk == 128) return {0.29, 2.0, 0.037};
    return {0.28, 1.3, 0.051};
}

// fine: fewer than 64 tokens per chunk.  Where the length is chosen on the device, such a pass is enqueued behind the one of 64 and as a
// rule returns at once; named by the caller, it has to give the same results, so it is cut the same way.
inline BwdFusedPlan plan_bwd_runs(int BH, int NC, int dk, int dv, bool io_bf16, int places, bool fine = false)
{
    if (places == 1 || BH <= 0 || NC <= 1) return uncut_bwd(NC);
    const bool pairs = dk == 64 && dv == 64 && io_bf16;        // workgroups of four waves, two on a compute unit
    double longest;
    if (places == kOnePerUnit || !io_bf16) {
        int R = kOnePerUnit / BH;
        if (R > NC / 4) R = NC / 4;
        if (R >= 2 && R <= 4) return light_bwd(NC, R, kBwdLightCost, &longest);
        return R < 2 ? uncut_bwd(NC) : ends_bwd(NC, R);
    }
    // Runs of one, two or four chunks and more, as many as find a place; light walks or walks from zero, by what they take (two
    // workgroups on a compute unit: 1.4 times as long).  1, 16 and 64 heads; us with runs of at
    // least four chunks -> with these:
    //   128 x 128:  4 chunks 26.5 -> 13.3, 27.0 -> 13.9, 27.9 -> 16.1 (light)  16 chunks 38.4 -> 26.7, 40.0 -> 34.3 (from zero; light 31.8), 47.5
    //              32 chunks 46.8 -> 30.4, 51.8 -> 43.7 (from zero), 84        64 chunks 48.7 -> 37.3, 60.4 (from zero)
    //   64 x 64:    4 chunks 17.1 -> 9.5, 17.6 -> 9.7, 17.8 -> 10.0 (light)    16 chunks 25.3 -> 16.9, 25.8 -> 19.8 (from zero), 28.9 -> 32.2
    // Runs of one chunk only, as long as they find a place, are too many for few long sequences (one head of 256 chunks: 64 x 64 39.2 us
    // in 64 runs, 60.4 in 256; 128 x 128 59.1 and 75.3, 56.1 in 128): every run's state is added up by one after the other.
    const BwdCost cost = bwd_cost(dk, dv);
    const int most = (pairs ? 2 : 1) * kOnePerUnit;
    // Three launches that return at once take 6.7 us, one 1.9: where few runs have four chunks, fine lengths take light walks
    // (length chosen on the device, ordinary gates, 128 heads of 64 x 64 and 12 chunks of 64: 39.4 us, 34.8 with the length named).
    const bool ends_ok = !fine || (most / BH > 4 && NC / 4 > 4);
    BwdFusedPlan best = uncut_bwd(NC);
    double least = NC;
    for (int at_once = kOnePerUnit; at_once <= most; at_once += kOnePerUnit)
        for (int shortest = 1; shortest <= 4; shortest *= 2) {
            int R = at_once / BH;
            if (R > NC / shortest) R = NC / shortest;
            if (R < 2) continue;
            const double crowd = R * BH > kOnePerUnit ? 1.4 : 1.0;
            if (shortest == 1) {
                const BwdFusedPlan light = light_bwd(NC, R < kMaxLightRuns ? R : kMaxLightRuns, cost.light, &longest);
                const double t = (light.R * BH > kOnePerUnit ? 1.4 : 1.0) * longest;
                if (t < least) { least = t; best = light; }
            }
            // (two or three runs per sequence: the walks from zero read most of q, f and grad_o once more while the
            // memory system is busy already; 128 x 128, 85 heads of 128 chunks 464 us light, 474 us from zero, but 64 heads, four runs each, 370 and 352)
            if (R < 4 || !ends_ok) continue;
            const BwdFusedPlan ends = ends_bwd(NC, R);
            const double mb = 4e-6 * dk * dv * (double)BH * ends.seg_tail;
            const double t = crowd * ends.rc + cost.ends + 0.3 * ends.sub_chunks + 0.037 * ends.seg_tail + cost.mb * mb;
            if (ends.R > 1 && t < least) { least = t; best = ends; }
        }
    return best;
}

}   // namespace hgrn2
