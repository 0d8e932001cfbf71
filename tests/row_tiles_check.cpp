// For each "nrows Ns n" line on stdin, walks the workgroups of the product's grid and
// counts how often each tile is taken; prints the waves per tile, the tiles along
// N_s, the groups of right-hand sides and whether every tile was taken once
// (tests/test_little_rules.py).
#include <cstdio>
#include <vector>

#include "little_rules.h"

int main() {
    int nrows, Ns, n;
    while (std::scanf("%d %d %d", &nrows, &Ns, &n) == 3) {
        const dfl::RowTiles t = dfl::row_tiles(nrows, Ns, n);
        const int tiles = dfl::ROW_WAVES / t.waves;
        std::vector<int> seen((size_t)nrows * t.nmt * t.ng, 0);
        bool ok = t.nmt * 16 >= Ns && t.ng * (t.wide ? 16 : 8) >= n;
        for (unsigned b = 0; b < dfl::row_workgroups(nrows, tiles, t.nmt, t.ng); ++b)
            for (int k = 0; k < tiles; ++k) {
                const dfl::RowTile x = dfl::row_tile(b, k, tiles, t.nmt, t.ng);
                if (x.row < 0 || x.m < 0 || x.m >= t.nmt || x.r < 0 || x.r >= t.ng) ok = false;
                if (ok && x.row < nrows) ++seen[((size_t)x.row * t.nmt + x.m) * t.ng + x.r];
            }
        for (int s : seen) ok = ok && s == 1;
        std::printf("%d %d %d %d\n", t.waves, t.nmt, t.ng, ok ? 1 : 0);
    }
    return 0;
}
