// Host-only check of the plan of the direct kernel's form with shared weights (csrc/shared_plan.h).  Without arguments: walks
// the words of a tap for every word count and prints "mismatches: N", exit status 0 = none.  With an argument: reads calls
// from standard input, one a line (m c_out cw ks stride kind kind staged, kind as in direct_plan.h and, for this form, as in
// shared_plan.h), prints the tile and the words per load of each, and the tile and the K walk of the other choice; with "branches": m c_out cw branches tail half, prints form,
// tile and words per load.
#include "shared_plan.h"

#include <cstdio>
#include <cstring>
#include <vector>

using namespace bcnn;

int main(int argc, char** argv)
{
    if (argc > 1 && !strcmp(argv[1], "branches")) {
        int m, c_out, cw, branches, tail, half;
        while (scanf("%d %d %d %d %d %d", &m, &c_out, &cw, &branches, &tail, &half) == 6) {
            const BranchChoice c = branches_choose(m, c_out, cw, branches, tail != 0, half != 0);
            printf("%d %d %d\n", c.form, c.tile, SharedWalk::make(cw, branches).wide);
        }
        return 0;
    }
    if (argc > 1) {
        int m, c_out, cw, ks, stride, kind, mine, staged;
        while (scanf("%d %d %d %d %d %d %d %d", &m, &c_out, &cw, &ks, &stride, &kind, &mine, &staged) == 8) {
            const DirectChoice other = direct_estimate(m, c_out, cw, ks, kind, staged != 0);
            printf("%d %d %d %d\n", shared_choose(m, c_out, cw, ks, stride, mine, other), SharedWalk::make(cw, ks * ks).wide, other.tile, direct_mode(cw));
        }
        return 0;
    }
    long bad = 0;
    for (int taps : {1, 2, 3, 9, 16})
        for (int cw = 1; cw <= 200; ++cw) {
            const SharedWalk w = SharedWalk::make(cw, taps);
            std::vector<int> seen(taps * cw, 0);
            long steps = 0;
            for (int g = 0; g < w.groups; ++g)
                for (int i = 0; i < (w.wide < 3 ? 4 : w.wide); ++i) {
                    const int tap = w.wide < 3 ? g * (4 / w.wide) + i / w.wide : g / w.per_tap;
                    const int k = w.wide < 3 ? i % w.wide : (g % w.per_tap) * w.wide + i;    // within a half
                    if (tap >= taps) continue;
                    ++steps;
                    if (k < w.half) ++seen[tap * cw + k];
                    if (k < cw - w.half) ++seen[tap * cw + w.half + k];
                }
            bool ok = steps == w.steps(taps) && w.half <= w.per_tap * w.wide;
            for (int n : seen) ok = ok && n == 1;
            if (!ok) { ++bad; printf("wrong: %d words, %d taps\n", cw, taps); }
        }
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
