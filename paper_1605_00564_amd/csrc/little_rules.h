// How the products with the little operator's rows are split over the device, and
// when the host looks at the norms of a little solve.  Plain C++, shared by the
// solve and a CPU test.
#pragma once

#include <algorithm>
#include <cmath>

namespace dfl {

// Tiles of a product of nrows rows with n right-hand sides: 16 of a row's N_s by 8
// (narrow) or 16 (wide) right-hand sides, with `waves` waves on a tile.
struct RowTiles {
    bool wide;
    int nmt, ng;   // tiles along N_s, groups of right-hand sides
    int waves;
};
constexpr int ROW_WAVES = 4;   // waves of a workgroup: on one tile, or on a tile each
inline RowTiles row_tiles(int nrows, int Ns, int n) {
    RowTiles t{};
    // narrow tiles where they hold fewer columns: 24 right-hand sides, 24^3 x 48:
    // 30.4 us against the 34 of two wide tiles
    t.wide = n > 8 && (n <= 16 || n > 24);
    t.nmt = (Ns + 15) / 16;
    t.ng = t.wide ? (n + 15) / 16 : (n + 7) / 8;
    // four waves share a tile as long as the tiles alone leave the device idle, two
    // waves per SIMD: a solve to 1e-8 with 1536 tiles a product takes 260 us so and
    // 293 with a wave per tile, with 2592 tiles 337 and 313, with 3888 406 and 348
    t.waves = (long)nrows * t.nmt * t.ng <= 2048 ? ROW_WAVES : 1;
    return t;
}

// Tile of a workgroup's `tile`-th group of waves.  The tiles of a row lie in
// consecutive workgroups eight apart: one XCD, whose L2 then holds its couplings.
struct RowTile {
    int row, m, r;   // row (nrows or more: none), tile along N_s, group of right-hand sides
};
constexpr RowTile row_tile(unsigned block, int tile, int tiles, int nmt, int ng) {
    const int at = (int)(block / 8) * tiles + tile, per = nmt * ng;
    return {at / per * 8 + (int)(block % 8), at % per / ng, at % ng};
}
constexpr unsigned row_workgroups(int nrows, int tiles, int nmt, int ng) {
    return (unsigned)(((nrows + 7) / 8 * nmt * ng + tiles - 1) / tiles) * 8;
}

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
