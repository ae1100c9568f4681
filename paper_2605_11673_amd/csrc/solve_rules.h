// How a solve is launched (host only).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace sta {

constexpr int kCgNeighbours = 16;   // of a node, held at a fixed place; the others are read again in each iteration
constexpr int kCgSmallRound = 32;   // nodes that the one workgroup of a small solve takes at a time
constexpr int kCgSmallRounds = 11;  // of which it holds the blocks

// Whether a system's solve is one launch of one workgroup.  rowptr: of its
// 3 `nodes` rows.  An iteration there takes some 2 us, 0.3 for each round of nodes
// and 0.45 for each trip over further neighbours, of all rounds one after the
// other; by two launches 8.5 to 9.5, and 0.4 a trip, all rounds side by side.
// Whole solves, one workgroup / launches, in us: fracture meshes and refinement
// supersets of up to 343 nodes 185 / 341 and 175 / 204, a vertex of 325
// neighbours 1,060 / 1,605; 100 nodes of 40 to 60 674 / 945, of all 918 / 743; 200 and
// 350 of 150 to 200 1,830 / 835 and 22,500 / 2,170.
inline bool cg_small_pays(int64_t nodes, const int32_t* rowptr)
{
    const int64_t rounds = (nodes + kCgSmallRound - 1) / kCgSmallRound;
    if (rounds > kCgSmallRounds)
        return false;
    int64_t trips = 0, most = 0;
    for (int64_t w = 0; w < rounds; ++w) {
        int64_t round = 0;
        for (int64_t i = w * kCgSmallRound; i < std::min(nodes, (w + 1) * kCgSmallRound); ++i) {
            const int64_t further = (rowptr[3 * i + 1] - rowptr[3 * i]) / 3 - kCgNeighbours;
            round = std::max(round, (further + kCgNeighbours - 1) / kCgNeighbours);
        }
        trips += round;
        most = std::max(most, round);
    }
    return 9 * trips + 6 * rounds <= 150 + 8 * most;
}

// Iterations to launch before the next look at the residual (rr = |r|^2), after
// `launched` of them: what is left at the mean rate so far, at least 4 and at most
// twice as many as have run (the rate changes on the way) and 256.  While the
// residual is not below |b| (CG lets it rise at first), is not a number or
// infinite, there is no rate to go by: 16.  A look costs about 18 us of idle GPU, a
// launch pair past convergence about 3.  Counted on residuals of cubes of 8 to 12
// cells, these looks against one per 16 iterations, in us: 46 iterations 42 / 60,
// 524 282 / 606, 989 819 / 1,125, 4,735 of which 1,693 above |b| 1,599 / 5,331
// (6,255 with a look every 4 there).
inline int cg_chunk(double rr, double bnorm2, double tol2, int launched)
{
    const double rate = std::log(rr / bnorm2) / launched;  // per iteration
    if (!(rate < 0.0) || std::isinf(rate))
        return 16;
    const double left = std::log(tol2 / rr) / rate;
    const int most = launched < 128 ? 2 * launched : 256;
    if (!(left < most))
        return most;
    return left > 4.0 ? (int)std::ceil(left) : 4;
}

}  // namespace sta
