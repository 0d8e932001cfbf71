// Follows the host's looks through solves whose residual falls by a constant
// factor: for each "tol rate" line on stdin, prints the steps that the solve
// needs, the steps that it runs and its looks (tests/test_little_rules.py checks
// them).
#include <cmath>
#include <cstdio>

#include "little_rules.h"

int main() {
    double tol, rate;
    while (std::scanf("%lf %lf", &tol, &rate) == 2) {
        int need = 1;
        while (!(std::pow(rate, need) <= tol) && need < 500) ++need;
        int steps = 0, looks = 0, want = dfl::first_look(tol);
        for (;;) {
            if (want < 1 || want > dfl::LOOK) return 1;
            steps += want;
            ++looks;
            if (steps >= need) break;
            want = dfl::next_look(steps, std::pow(rate, steps), tol);
        }
        std::printf("%d %d %d\n", need, steps, looks);
    }
    return 0;
}
