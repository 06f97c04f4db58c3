// Host-only check of how the kernel whose weights stay in LDS splits a call (csrc/resident_plan.h): every column of 32 pixels of
// every channel tile is taken by exactly one pass of one wave, passes hold one to RESIDENT_PASS columns, a launch has at
// most 256 workgroups unless there are more channel tiles, and places lie inside their LDS table.  Prints "mismatches: N"; exit
// status 0 = none.  With lines "m c_out cw taps bits own nothing_outside" on stdin and an argument, "calls" (bits of a filter) or "branches": whether
// the kernel takes each of them, and the words of a load.
#include "resident_plan.h"

#include <cstdio>
#include <vector>

using namespace bcnn;

static long check(int m, int c_out, int most = RESIDENT_PASS, int table = RESIDENT_COLUMNS)
{
    const ResidentSplit split = resident_split(m, c_out);
    long bad = 0;
    if (split.n_ctiles * RESIDENT_CHANNELS < c_out || (split.n_ctiles - 1) * RESIDENT_CHANNELS >= c_out) ++bad;
    if (split.n_ranges < 1 || (split.n_ctiles < 256 && split.n_ctiles * split.n_ranges > 256)) ++bad;
    const int quotient = split.columns / split.n_ranges, rest = split.columns % split.n_ranges;
    std::vector<int> seen(split.columns, 0);
    for (int range = 0; range < split.n_ranges; ++range) {
        const ResidentRun columns = resident_run(quotient, rest, range);
        for (int done = 0; done < columns.count; done += table) {
            const int here = columns.count - done < table ? columns.count - done : table;
            for (int wave = 0; wave < RESIDENT_WAVES; ++wave) {
                const ResidentRun mine = resident_run(here / RESIDENT_WAVES, here % RESIDENT_WAVES, wave);
                for (int place = mine.first, left = mine.count; left > 0;) {
                    const int take = resident_take(left, most);
                    if (take < 1 || take > most || take > left || place + take > here) return bad + 1;
                    for (int k = 0; k < take; ++k) ++seen[columns.first + done + place + k];
                    place += take;
                    left -= take;
                }
            }
        }
    }
    for (int n : seen)
        if (n != 1) ++bad;
    return bad;
}

int main(int argc, char** argv)
{
    if (argc > 1) {
        int m, c_out, cw, taps, bits, own, nothing;
        while (scanf("%d %d %d %d %d %d %d", &m, &c_out, &cw, &taps, &bits, &own, &nothing) == 7)
            printf("%d %d\n", (int)(argv[1][0] == 'c' ? resident_takes(m, c_out, cw, taps == 9 ? 3 : 1) : resident_takes_branches(m, c_out, cw, taps, bits, own, nothing)),
                   SharedWalk::make(cw, taps).wide);
        return 0;
    }
    long bad = 0;
    for (int c_out : {1, 32, 64, 65, 130, 256, 700, 1024, 5000, 20000})
        for (int m : {1, 31, 32, 33, 1000, 3136, 12544, 50176, 50177, 426000, 1000001}) bad += check(m, c_out) + check(m, c_out, 2, RESIDENT_BRANCH_COLUMNS);
    for (int m = 1; m < 60000; m += 37) bad += check(m, 256);
    printf("mismatches: %ld\n", bad);
    return bad != 0;
}
