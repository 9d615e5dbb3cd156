// Choice of the tile and the split of K for a launch of the MFMA tile
// kernels (linear layers, convolution): host code only.
#pragma once
#include <math.h>
#include <stdint.h>

#include <algorithm>

namespace regenvc {

// One tile shape: a workgroup's fixed time (launch, first copies, epilogue;
// unsplit and split) and its time per 64-deep K step, in us, and a factor on
// rounds of n_cu workgroups (the clock that the power limit leaves, shared LDS
// and memory).  Fitted, all together, to the times of whole launches.  Rounds
// are counted as if each compute unit ran one workgroup at a time; the small
// tiles, two or three of which it runs side by side, have the gain of that in
// their factor, which is then below one.
struct TileCost {
    int32_t tile, bm, bn, waves;
    double fixed, fixed_split, step, load;
    bool splits;  // has a split-K form
};
// The second kernel of a split: its launch (us) and the rate (bytes per us) at
// which partials are written, read and the result stored.
struct SplitCost {
    double launch, rate;
    int64_t out_bytes;  // per output element, read and written
};
struct TilePlan {
    int32_t tile, splits;
    int32_t bm, bn, waves;
};

// The tile and number of K ranges (at most 8, of at least 8 steps each) with
// the smallest estimated time: whole rounds of n_cu workgroups and one last,
// partly filled round.  A split needs one f32 plane of the output per range
// in ws_bytes, and at most two rounds of workgroups.
template <int N_COSTS>
TilePlan plan_tiles(const TileCost (&costs)[N_COSTS], const SplitCost &sc, int64_t M, int64_t N, int nk, int n_cu,
                    int64_t ws_bytes)
{
    const int64_t plane = M * N * (int64_t)sizeof(float);
    TilePlan best{costs[0].tile, 1, costs[0].bm, costs[0].bn, costs[0].waves};
    double best_t = INFINITY;
    for (const TileCost &c : costs) {
        const int64_t tiles = (M + c.bm - 1) / c.bm * ((N + c.bn - 1) / c.bn);
        if (tiles > 0x7fffffff / 8) continue;
        const int max_splits = c.splits ? std::min(8, nk / 8) : 1;
        for (int s = 1; s <= std::max(1, max_splits); ++s) {
            if (s > 1 && (s * plane > ws_bytes || tiles * s > 2 * (int64_t)n_cu)) break;
            const double one = (s > 1 ? c.fixed_split : c.fixed) + (double)((nk + s - 1) / s) * c.step;
            const int64_t full = tiles * s / n_cu, rest = tiles * s % n_cu;
            double t = (double)full * one * c.load;
            if (rest > 0) t += one * (1.0 + (c.load - 1.0) * (double)rest / n_cu);
            if (s > 1) t += sc.launch + ((double)plane * 2 * s + (double)M * N * (double)sc.out_bytes) / sc.rate;
            if (t < best_t) best_t = t, best = TilePlan{c.tile, s, c.bm, c.bn, c.waves};
        }
    }
    return best;
}

}  // namespace regenvc
