// Host-only check of the choice between the matrix-core kernels (csrc/direct_plan.h, then csrc/shared_plan.h, as the entry points ask them):
// measured calls go to the kernel that is faster on them, or stay on the one that took them before there was the third; prints "mismatches: N", exit status 0 = none.
#include "shared_plan.h"

#include <cstdio>

using namespace bcnn;

enum { STAGED, DIRECT, SHARED };

int main()
{
    // calls that the staged kernel covers: pixels, channels out, words, filter, kind, kind for shared weights, who takes them; us of
    // the staged or direct kernel and of the form with shared weights
    const struct { int m, c_out, cw, ks, kind, mine, who; } calls[] = {
        {13328, 960, 8, 1, KIND_BITS_OUT, SHARED_BITS, SHARED},                 // 5.49, 5.27
        {41552, 126, 32, 1, KIND_BITS_OUT, SHARED_BITS, SHARED},                // 6.63, 6.08
        {50176, 128, 4, 1, KIND_BITS_OUT, SHARED_BITS, SHARED},                 // 4.61, 3.85
        {50176, 100, 8, 1, KIND_BITS_OUT, SHARED_BITS, SHARED},                 // 4.40, 3.97
        {45423, 576, 32, 1, KIND_SUMS_OUT, SHARED_SUMS, STAGED},
        {50176, 128, 32, 1, KIND_MODULE_PLAIN, SHARED_FLOAT, STAGED},           // 17.3, 16.7
        {50176, 256, 32, 1, KIND_MODULE_PLAIN, SHARED_FLOAT, STAGED},           // 26.4, 25.8
        {50176, 128, 16, 1, KIND_MODULE_PLAIN, SHARED_HALF, SHARED},            // 12.3, 11.9
        {50176, 128, 16, 1, KIND_MODULE_PLAIN, SHARED_FLOAT, SHARED},           // 15.5, 14.0
        {50176, 128, 8, 3, KIND_MODULE_PLAIN, SHARED_HALF, SHARED},             // 16.5, 16.5
        {23520, 640, 4, 3, KIND_MODULE_PLAIN, SHARED_HALF, STAGED},             // 22.9, 22.9
        {23520, 640, 4, 3, KIND_MODULE_PLAIN, SHARED_FLOAT, STAGED},            // 29.9, 28.0
        {15680, 1024, 12, 3, KIND_MODULE_GENERAL, SHARED_HALF, SHARED},         // 37.0, 36.1
        {50176, 256, 32, 3, KIND_MODULE_GENERAL, SHARED_HALF, STAGED},          // 63.0, 66.8
        {50176, 256, 32, 3, KIND_MODULE_GENERAL, SHARED_FLOAT, STAGED},         // 62.1, 67.5
        {49, 1024, 32, 3, KIND_BITS_OUT, SHARED_BITS, DIRECT},                  // 5.1, 10.2
        {196, 128, 4, 3, KIND_SUMS_OUT, SHARED_SUMS, DIRECT},                   // 3.1, 4.5
        {100352, 256, 8, 1, KIND_SUMS_OUT, SHARED_SUMS, DIRECT},                // 19.2, 18.6
        {784, 128, 16, 1, KIND_MODULE_PLAIN, SHARED_HALF, DIRECT},              // 3.4, 4.4
        {784, 128, 16, 1, KIND_MODULE_PLAIN, SHARED_FLOAT, DIRECT},             // 3.3, 4.6
        {6272, 512, 16, 1, KIND_MODULE_GENERAL, SHARED_HALF, DIRECT},           // 6.8, 6.9
        {6272, 512, 16, 1, KIND_MODULE_GENERAL, SHARED_FLOAT, DIRECT},          // 7.6, 7.8
    };
    long bad = 0;
    for (const auto& t : calls) {
        const DirectChoice other = direct_estimate(t.m, t.c_out, t.cw, t.ks, t.kind, true);
        const int shared = shared_choose(t.m, t.c_out, t.cw, t.ks, 1, t.mine, other);
        if ((shared != SHARED_NONE ? SHARED : other.tile != DIRECT_NONE ? DIRECT : STAGED) != t.who) {
            ++bad;
            printf("wrong: %d pixels, %d channels, %d words, %d x %d, kind %d, %d\n", t.m, t.c_out, t.cw, t.ks, t.ks, t.kind, t.mine);
        }
    }
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
