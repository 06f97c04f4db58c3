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
    check(direct_behind_on_bits(1, 2, 64, 802816ll * 64), true, "bits 64 -> 64, 256 maps of 56 x 56");
    check(direct_behind_on_bits(1, 1, 128, 200704ll * 128), true, "bits 32 -> 128, 64 maps of 56 x 56");
    check(direct_behind_on_bits(1, 2, 512, 200704ll * 512), true, "bits 64 -> 512, 64 maps of 56 x 56");
    check(direct_behind_on_bits(1, 1, 256, 3136ll * 256), false, "bits 32 -> 256, one map of 56 x 56");
    check(direct_behind_on_bits(1, 2, 256, 50176ll * 256), false, "bits 64 -> 256, 16 maps of 56 x 56");
    check(direct_behind_on_bits(1, 2, 16, 802816ll * 16), true, "bits 64 -> 16, 256 maps of 56 x 56");
    check(direct_behind_on_bits(1, 3, 256, 802816ll * 256), false, "bits 96 -> 256, 256 maps of 56 x 56");
    check(direct_behind_on_bits(3, 1, 256, 802816ll * 256), false, "bits 3x3, 32 -> 256, 256 maps of 56 x 56");
    check(direct_behind_on_float_module(1, 2, 64, true, false, true, 802816ll * 64), true, "module without stream, 64 -> 64");
    check(direct_behind_on_float_module(1, 1, 64, true, true, false, 95648ll * 64), true, "module without bits, 15 -> 64");
    check(direct_behind_on_float_module(1, 2, 512, false, true, true, 752640ll * 512), true, "module without identity, 64 -> 512");
    check(direct_behind_on_float_module(1, 4, 512, false, true, true, 376320ll * 512), true, "module without identity, 128 -> 512");
    check(direct_behind_on_float_module(1, 2, 256, false, true, true, 200704ll * 256), false, "module without identity, 64 -> 256, 64 maps");
    check(direct_behind_on_float_module(1, 4, 64, true, false, true, 802816ll * 64), false, "module without stream, 128 -> 64");
    check(direct_behind_on_float_module(1, 2, 64, true, false, true, 12544ll * 64), false, "module without stream, small");
    check(direct_behind_on_float_module(3, 2, 717, true, true, true, 94080ll * 717), false, "module 3x3, 64 -> 717");
    check(direct_behind_on_float_module(3, 2, 512, true, true, true, 200704ll * 512), false, "module 3x3, 64 -> 512");
    check(direct_behind_on_float_module(1, 2, 511, false, true, true, 752640ll * 511), false, "module without identity, 64 -> 511");
    check(direct_behind_on_float_module(1, 2, 65, true, false, true, 376320ll * 65), false, "module without stream, 64 -> 65");
    check(direct_behind_on_branch_tail(4, 8, 448, false, 376320ll * 448), true, "float tail, 128 x 2 -> 448");
    check(direct_behind_on_branch_tail(4, 8, 448, false, 47040ll * 448), false, "float tail, 128 x 2 -> 448, cached");
    check(direct_behind_on_branch_tail(1, 8, 451, false, 188160ll * 451), false, "float tail, 32 x 8 -> 451");
    check(direct_behind_on_branch_tail(1, 9, 717, false, 188160ll * 717), false, "float tail, 3x3, 32 -> 717");
    check(direct_behind_on_branch_tail(7, 56, 717, false, 188160ll * 717), false, "float tail, 200 x 8 -> 717");
    check(direct_behind_on_branch_tail(2, 4, 451, true, 188160ll * 451), false, "half tail, 64 x 2 -> 451");
    check(direct_behind_on_branch_tail(1, 1, 448, true, 188160ll * 448), true, "half tail, 32 -> 448");
    check(direct_behind_on_branch_tail(2, 8, 448, true, 188160ll * 448), false, "half tail, 64 x 4 -> 448");
    printf("mismatches: %ld\n", bad);
    return bad ? 1 : 0;
}
