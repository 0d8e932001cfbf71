// For each "positions-per-block blocks" line on stdin, prints the positions of a tile
// of the canonical-vector stencil and whether it is used (tests/test_tile_rule.py).
#include <cstdio>

#include "block_tables.h"

int main() {
    int Vbh, Nb;
    while (std::scanf("%d %d", &Vbh, &Nb) == 2) {
        const int P = dfl::tile_positions(Vbh, Nb, 128);
        std::printf("%d %d\n", P, dfl::tiles_fill(P, 128) ? 1 : 0);
    }
    return 0;
}
