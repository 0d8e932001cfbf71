// When the host looks at the norms of a little solve.  Plain C++, shared by the
// solve and a CPU test.
#pragma once

#include <algorithm>
#include <cmath>

namespace dfl {

// Iterations between two looks, at most: a look costs about 12 us, an iteration
// 30 on small systems and up to 130 on large ones (24^3 x 48, N_s = 20, 24
// right-hand sides), and the iterations after the one that converged are wasted.
constexpr int LOOK = 4;

// Iterations to the first look: an iteration gains about one digit at best, so as
// many as the digits asked for.  Looking after four in any case, a solve of one
// iteration to 0.3 took 374 us instead of 240 (24^3 x 48, N_s = 12, 24 right-hand
// sides).
inline int first_look(double tol) {
    if (!(tol > 0)) return LOOK;
    return (int)std::min<double>(LOOK, std::max(1.0, std::ceil(-std::log10(tol) - 1e-6)));
}

// Iterations to the next look after `iters` iterations have brought the residual
// to `rel`: those that the same gain per iteration needs.
inline int next_look(int iters, double rel, double tol) {
    if (!(rel > tol && rel < 1 && tol > 0)) return LOOK;
    const double left = iters * std::log(tol / rel) / std::log(rel);
    return (int)std::min<double>(LOOK, std::max(1.0, std::ceil(left - 1e-6)));
}

}  // namespace dfl
