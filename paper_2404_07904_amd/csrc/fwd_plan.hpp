// The cut of the fused forward walk of an equal-length batch: plain host arithmetic on four sizes, in a
// header of its own so that it can be compiled and checked without a GPU.
#pragma once

namespace hgrn2 {

constexpr int kMaxFwdRuns = 16;

// How the fused forward walk of an equal-length batch cuts its sequences.  light > 1: into that many
// runs, each of whose workgroups finds the state it starts from by a light walk of its own over the
// chunks before the run.  seg > 1: into runs of run_chunks chunks (TokenLayout::seg), whose entering
// states launch_run_ends provides.
struct FwdRuns { int light = 1, seg = 1, run_chunks = 0; };

// Cost of a chunk of a light walk in chunks of the walk proper (measured: 1.0 us against 2.0 us in the
// 128 x 64 variant, and less next to other workgroups that stream).
constexpr double kLightCost = 0.42;

// Runs with a light walk each: the cuts that let all of them finish together,
// len_r + rho start_r = T for every run r, so that start_{r+1} = T + (1 - rho) start_r.
// (Chunk numbers are ints throughout: 86 to 128 heads of 64 are cut into two such runs however long they
// are, and a sequence of 262144 tokens has 32768 chunks of 8.)
struct FwdCuts { int bnd[kMaxFwdRuns + 1]; };      // run r is chunks bnd[r] .. bnd[r + 1] - 1
inline void fused_cuts(int NC, int R, FwdCuts* cuts)
{
    int* bnd = cuts->bnd;
    const double rho = 0.33;         // (below the cost: the last run, with the longest light walk, has one chunk anyway)
    double sum = 0.0, x = 1.0;
    for (int r = 0; r < R; ++r) { sum += x; x *= 1.0 - rho; }
    const double T = NC / sum;
    double end = 0.0;
    bnd[0] = 0;
    for (int r = 1; r < R; ++r) {
        end = T + (1.0 - rho) * end;
        int b = (int)(end + 0.5);
        if (b < bnd[r - 1] + 1) b = bnd[r - 1] + 1;
        if (b > NC - (R - r)) b = NC - (R - r);
        bnd[r] = b;
    }
    bnd[R] = NC;
}

// Workgroup -> sequence and item of the sequence (light run and half of dv, `per` of them).
// Workgroups are dealt to the 8 XCDs round-robin; the items of a sequence go to one XCD, so that they
// share an L2 for the rows several of them read, sequence s to XCD s % 8 -- but for the last BH % 8 sequences, whose
// items are dealt out one by one: with those whole, 11 of 85 sequences in three runs made 33 workgroups on some
// XCDs, for 32 compute units, and the pass took two rounds (85 heads of 2048 tokens: 92 us, uncut 70.6, so 55).
// (a workgroup past the last item gets seq >= BH)
constexpr int kXcds = 8;         // accelerator dies; consecutive workgroup ids land on consecutive dies
struct RunItem { int seq, sub; };
constexpr int run_grid(int BH, int per) { return kXcds * ((BH * per + kXcds - 1) / kXcds); }
constexpr RunItem run_item(int block, int BH, int per)
{
    const int x = block % kXcds, r = block / kXcds, whole = BH / kXcds, at = r - whole * per;
    const int i = at < 0 ? r : at * kXcds + x, q = i / per;
    return RunItem{at < 0 ? q * kXcds + x : whole * kXcds + q, i - q * per};
}

// light_walks = false: no light walks (whose workgroups all read the sequence's initial state, while one of
// them writes the final one: not for a state that is continued in place).
// kept: the walk keeps the chunk states for a backward pass.
inline FwdRuns plan_fwd_runs(int BH, int NC, int dk, int dv, bool light_walks = true, bool kept = false)
{
    FwdRuns r;
    r.run_chunks = NC;
    if (BH == 0 || NC < 2) return r;
    // The candidates and what they take, in chunks of the 64-column variants (2 us each), fitted to runs of
    // 1 to 128 heads of 128 and 64 and 2 to 256 chunks; the start-up they share is left out.  "halves": two
    // workgroups per run, each half of dv (the only way for 64 x 128 heads, no way for dv = 64); "whole": twice
    // the runs, whose chunks take 1.5 to 1.6 times as long.  Beyond 256 workgroups nothing gains: heads of 64
    // find two places on a compute unit, but two runs there slow each other down as much (256 heads of 2000
    // tokens: 70 us, in two runs each 73 us).
    //   light walks (all runs finish together):  NC rho / (1 - (1 - rho)^R)
    //   walks from zero: the second launch and the states in between cost as much as 5 to 9 chunks
    // e.g. 16 heads, 13 chunks: 27.9 us with 8 light walks (halves), 31 us whole, 28.8 us from zero;
    // 32 heads: 32 chunks 40 / 41.5 us (light / from zero), 64 chunks 65 us from zero in halves, 256 chunks
    // 209 us in halves, 182 us whole; 64 heads whole, 16 / 32 / 64 chunks: 30.5 / 52 / 96 us light, 39 / 55 / 91 us from zero.
    double best = NC;                                    // one run (128 x 128: in halves up to 128 heads)
    if (dk == 128 && dv == 128 && BH > 128) return r;
    // Two light runs that nearly fill the chip pay only while the walk is not bound by memory, to which kept states
    // add 2 dk dv bytes a chunk: 128 heads with kept states, us uncut / in two runs: 32 chunks 79.2 / 76.0, 48 chunks 131 / 123,
    // 64 chunks 169 / 177, 128 chunks 335 / 365; 112 heads: 64 chunks 157.8 / 156.6, 128 chunks 309 / 311.
    if (kept && dk == 128 && dv == 128 && BH > 112 && NC >= 56) return r;
    auto consider = [&](int places, double light_factor, double ends_cost, double per_chunk) {
        int R = places / BH;
        if (R > kMaxFwdRuns) R = kMaxFwdRuns;
        if (R > NC) R = NC;
        if (light_walks && R >= 2) {
            double keep = 1.0;
            for (int i = 0; i < R; ++i) keep *= 1.0 - kLightCost;
            const double t = light_factor * NC * kLightCost / (1.0 - keep);
            if (t < best) { best = t; r.light = R; r.seg = 1; r.run_chunks = NC; }
        }
        int seg = places / BH;
        if (seg > NC / 3) seg = NC / 3;                  // at least three chunks each
        if (seg >= 2) {
            const double t = ends_cost + per_chunk * NC / seg;
            if (t < best) {
                best = t;
                r.light = 1;
                r.run_chunks = (NC + seg - 1) / seg;
                r.seg = (NC + r.run_chunks - 1) / r.run_chunks;
            }
        }
    };
    const bool halves = dv == 128;
    consider(halves ? 128 : 256, 1.1, 5.0, 1.5);
    if (dk == 128 && halves) consider(256, 1.47, 9.0, 2.2);
    return r;
}

}   // namespace hgrn2
