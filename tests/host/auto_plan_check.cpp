// Host-only check of AUTO's rules (csrc/auto_plan.h): measured calls go where they were faster.  Prints "mismatches: N"; exit
// status 0 = none.
#include "auto_plan.h"

#include <cstdio>

using namespace bcnn;

static long bad = 0;
static void check(bool got, bool want, const char* what)
{
    if (got != want) { ++bad; printf("wrong: %s\n", what); }
}

int main()
{
    check(direct_behind_on_bits(1, 2, 802816ll * 64), true, "bits 64 -> 64, 256 maps of 56 x 56");
    check(direct_behind_on_bits(1, 1, 200704ll * 128), true, "bits 32 -> 128, 64 maps of 56 x 56");
    check(direct_behind_on_bits(1, 2, 200704ll * 512), true, "bits 64 -> 512, 64 maps of 56 x 56");
    check(direct_behind_on_bits(1, 1, 3136ll * 256), false, "bits 32 -> 256, one map of 56 x 56");
    check(direct_behind_on_bits(1, 2, 50176ll * 256), false, "bits 64 -> 256, 16 maps of 56 x 56");
    check(direct_behind_on_bits(1, 3, 802816ll * 256), false, "bits 96 -> 256, 256 maps of 56 x 56");
    check(direct_behind_on_bits(3, 1, 802816ll * 256), false, "bits 3x3, 32 -> 256, 256 maps of 56 x 56");
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
