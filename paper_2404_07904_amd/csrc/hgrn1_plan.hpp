// The cut of HGRN1's sequences into runs: plain host arithmetic on a few sizes, in a header of its own so that it can be compiled
// and checked without a GPU.
#pragma once

namespace hgrn2 {

constexpr int kH1Waves = 8;                       // waves per workgroup
constexpr int kH1Threads = 64 * kH1Waves;
constexpr int kH1Chan = 64;                       // channels per workgroup: a pair per lane of a half-wave
constexpr int kH1Segs = 2 * kH1Waves;             // segments per block: one per half-wave
constexpr int kH1SegLong = 32;                    // tokens per segment
constexpr int kH1SegShort = 16;                   // ... of the backward with activations (it holds more per token)

inline int h1_blocks(int N, int seg) { return (N + kH1Segs * seg - 1) / (kH1Segs * seg); }

// Runs of a sequence of NBLK blocks.  While the channels give fewer workgroups than the chip takes, as many as find a place; a
// run costs the launch and the walk of hgrn1_ends_kernel on top, as much as 0.8 and 0.6 blocks (5 us each), so three and fewer
// blocks stay together, and so do sequences that would only be halved.
constexpr int kH1Places = 256, kH1MaxRuns = 64;
inline int h1_runs(int B, int d, int NBLK, int* blocks_per_run)
{
    *blocks_per_run = NBLK;
    const long long groups = (long long)B * (d / kH1Chan);
    if (groups <= 0 || NBLK < 4) return 1;
    long long R = kH1Places / groups;
    if (R > NBLK) R = NBLK;
    if (R > kH1MaxRuns) R = kH1MaxRuns;
    if (R < 3) return 1;
    const int rb = (int)((NBLK + R - 1) / R);
    if (0.8 + 1.6 * rb >= NBLK) return 1;
    *blocks_per_run = rb;
    return (NBLK + rb - 1) / rb;
}

}   // namespace hgrn2
