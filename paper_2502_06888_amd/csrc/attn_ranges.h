// How many ranges the cached positions of a sequence are cut into: plain host code, no HIP.
#pragma once

namespace kattn {

// Attention workgroup: wavefronts, row groups each of them loads together, and wavefronts per SIMD.
// Query and output slices of a lane take 16 registers per query head.  Up to four heads fit the 128
// registers that four wavefronts leave; more would spill, so those run with fewer wavefronts and keep
// their loads in flight by requesting the next chunk before using this one.
constexpr int kAttnWaves = 4, kChunk = 2;
constexpr int attn_waves_per_simd(int G) { return G <= 4 ? 4 : G <= 6 ? 3 : 2; }

// Ranges of a cache of `len` positions in a launch over `pairs` (sequence, key-value head) pairs of G
// query heads of hd elements.  A function of the sequence's own length and of the size of the launch, as
// the splits of the projections are: what a sequence attends to is summed in the same order whatever
// the lengths of the others.  A range costs its loop passes plus a fixed part (query load, slot merge,
// partial sums written and read: about four passes, kRangeCost); the chip holds `slots` workgroups at a
// time, so the launch costs ceil(pairs * n / slots) rounds of that, priced as if all caches were as long
// as this one.  The merge launch counts as kMergeCost passes.  Counts beyond kMostRounds rounds are not
// tried; with more pairs than that the cache stays whole.
inline int attn_ranges(int len, long pairs, int G, int hd, int max_ranges) {
    constexpr int kRangeCost = 4, kMergeCost = 8, kMostRounds = 2;
    const int step = kAttnWaves * (512 / hd) * kChunk;  // positions of a loop pass
    const long slots = 256L * attn_waves_per_simd(G);
    long best = 0;
    int ranges = 1;
    for (int n = 1; n <= max_ranges && (long)(n - 1) * step < len && (n == 1 || pairs * n <= kMostRounds * slots); ++n) {
        const long passes = ((len + n - 1) / n + step - 1) / step;
        const long cost = (pairs * n + slots - 1) / slots * (passes + kRangeCost) + (n > 1 ? kMergeCost : 0);
        if (n == 1 || cost < best) {
            best = cost;
            ranges = n;
        }
    }
    return ranges;
}

}  // namespace kattn
