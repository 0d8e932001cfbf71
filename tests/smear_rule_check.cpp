// Prints the groups of four of each "sites vectors" line on stdin
// (tests/test_smear_rule.py).
#include <cstdio>

#include "smear_rules.h"

int main() {
    long V;
    int n;
    while (std::scanf("%ld %d", &V, &n) == 2) std::printf("%d\n", dfl::gauss_groups(V, n));
    return 0;
}
