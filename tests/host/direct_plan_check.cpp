// Host-only check of the direct kernel's tile choice (csrc/direct_plan.h).  Without arguments: measured calls go to the kernel
// that is faster on them; prints "mismatches: N", exit status 0 = none.  With "conv" or "branches": reads calls from standard
// input, one a line (m c_out cw ks kind staged, or m c_out cw branches tail half), prints the tile and the K walk of each.
#include "direct_plan.h"

#include <cstdio>
#include <cstring>

using namespace bcnn;

int main(int argc, char** argv)
{
    int m, c_out, cw, a, b, c;
    if (argc > 1 && !strcmp(argv[1], "conv")) {
        while (scanf("%d %d %d %d %d %d", &m, &c_out, &cw, &a, &b, &c) == 6)
            printf("%d %d\n", direct_choose(m, c_out, cw, a, b, c != 0), direct_mode(cw));
        return 0;
    }
    if (argc > 1 && !strcmp(argv[1], "branches")) {
        while (scanf("%d %d %d %d %d %d", &m, &c_out, &cw, &a, &b, &c) == 6)
            printf("%d %d\n", branches_direct_choose(m, c_out, cw, a, b != 0, c != 0), BranchWalk::make(cw).rest);
        return 0;
    }
    // calls that the staged kernel covers: pixels, channels out, words, filter, kind, whether it is the faster one
    const struct { int m, c_out, cw, ks, kind; bool staged; } calls[] = {
        {13328, 960, 8, 1, KIND_BITS_OUT, true}, {41552, 126, 32, 1, KIND_BITS_OUT, true}, {50176, 128, 4, 1, KIND_BITS_OUT, true},
        {50176, 100, 8, 1, KIND_BITS_OUT, true}, {45423, 576, 32, 1, KIND_SUMS_OUT, true}, {50176, 128, 32, 1, KIND_MODULE_PLAIN, true},
        {50176, 256, 32, 1, KIND_MODULE_PLAIN, true}, {50176, 128, 16, 1, KIND_MODULE_PLAIN, true}, {50176, 128, 8, 3, KIND_MODULE_PLAIN, true}, {23520, 640, 4, 3, KIND_MODULE_PLAIN, true},
        {15680, 1024, 12, 3, KIND_MODULE_GENERAL, true}, {50176, 256, 32, 3, KIND_MODULE_GENERAL, true},
        {49, 1024, 32, 3, KIND_BITS_OUT, false}, {196, 128, 4, 3, KIND_SUMS_OUT, false}, {100352, 256, 8, 1, KIND_SUMS_OUT, false},
        {784, 128, 16, 1, KIND_MODULE_PLAIN, false}, {6272, 512, 16, 1, KIND_MODULE_GENERAL, false},
    };
    long bad = 0;
    for (const auto& t : calls)
        if ((direct_choose(t.m, t.c_out, t.cw, t.ks, t.kind, true) == DIRECT_NONE) != t.staged) {
            ++bad;
            printf("wrong: %d pixels, %d channels, %d words, %d x %d, kind %d\n", t.m, t.c_out, t.cw, t.ks, t.ks, t.kind);
        }
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
