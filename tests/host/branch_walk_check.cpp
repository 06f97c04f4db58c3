// Host-only check of the branch mode's word walk (csrc/branch_walk.h): for every word count up to 4096, walk a tap as the
// kernel does, through the functions that the kernel uses, and check that
//   - every word of the tap is read exactly once, by one lane half,
//   - no whole group of four, which is loaded without a check, leaves the tap,
//   - both halves take the same number of K-steps, half_words of them, and the positions that are zero on both sides
//     are the 64 * half_words - 32 * cw that the kernel's start value allows for,
//   - no group is empty, and none of more than four K-steps.
// Prints "mismatches: N"; exit status 0 = none.
#include "branch_walk.h"

#include <cstdio>
#include <vector>

using namespace bcnn;

int main()
{
    long bad = 0;
    for (int cw = 1; cw <= 4096; ++cw) {
        const BranchWalk w = BranchWalk::make(cw);
        std::vector<int> seen(cw, 0);
        long before = bad;
        int steps = 0, zero_words = 0;
        for (int g = 0; g < w.groups(); ++g) {
            if (w.steps(g) < 1 || w.steps(g) > 4) ++bad;
            steps += w.steps(g);
            for (int h = 0; h < 2; ++h)
                for (int i = 0; i < w.steps(g); ++i) {
                    const int word = w.first(h, g) + i;
                    if (g >= w.full && !w.real(word)) { ++zero_words; continue; }   // reads as zero on both sides
                    if (word < 0 || word >= cw) ++bad;                               // another tap's, pixel's or branch's word
                    else ++seen[word];
                }
        }
        for (int n : seen)
            if (n != 1) ++bad;
        if (steps != w.half_words || 32 * zero_words != 64 * w.half_words - 32 * cw) ++bad;
        if (bad != before) printf("wrong at %d words\n", cw);
    }
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
