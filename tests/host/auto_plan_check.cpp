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
    check(direct_behind_on_float_module(1, 2, 64, true, false, true, 802816ll * 64), true, "module without stream, 64 -> 64");
    check(direct_behind_on_float_module(1, 1, 64, true, true, false, 95648ll * 64), true, "module without bits, 15 -> 64");
    check(direct_behind_on_float_module(1, 2, 512, false, true, true, 752640ll * 512), true, "module without identity, 64 -> 512");
    check(direct_behind_on_float_module(1, 4, 512, false, true, true, 376320ll * 512), true, "module without identity, 128 -> 512");
    check(direct_behind_on_float_module(1, 2, 256, false, true, true, 200704ll * 256), false, "module without identity, 64 -> 256, 64 maps");
    check(direct_behind_on_float_module(1, 4, 64, true, false, true, 802816ll * 64), false, "module without stream, 128 -> 64");
    check(direct_behind_on_float_module(1, 2, 64, true, false, true, 12544ll * 64), false, "module without stream, small");
    check(direct_behind_on_float_module(3, 2, 717, true, true, true, 94080ll * 717), true, "module 3x3, 64 -> 717");
    check(direct_behind_on_float_module(3, 2, 512, true, true, true, 200704ll * 512), false, "module 3x3, 64 -> 512");
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
