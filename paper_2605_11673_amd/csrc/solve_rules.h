// How a solve is launched (host only).
#pragma once

#include <cmath>

namespace sta {

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
