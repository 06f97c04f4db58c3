// Kernel arguments of the direct kernel's form with shared weights.
#pragma once
#include "conv_mfma_direct_kernel.h"
#include "shared_plan.h"

namespace bcnn {

inline DirectArgs shared_args(const ConvShape& s, int taps, const SharedWalk& walk)
{
    DirectArgs a{};
    a.s = s;
    a.taps = taps;
    a.n_words = taps * s.cw;
    a.per_tap = walk.per_tap;
    a.n_units = walk.groups;
    a.x_bytes = (int32_t)((int64_t)s.n * s.h * s.w * s.cw * 4);
    a.w_bytes = (int32_t)((int64_t)s.c_out * a.n_words * 4);
    a.pad_bytes = a.n_words * 4;
    a.row_jump = (s.w - s.ks) * s.cw;
    a.div_hw = DivBy::make(s.ho * s.wo);
    a.div_wo = DivBy::make(s.wo);
    a.div_tap = DivBy::make(a.per_tap);
    return a;
}

inline DirectBranch shared_extra(const ConvShape& s, const SharedWalk& walk)
{
    DirectBranch br{};
    const int c_in = s.k / (s.ks * s.ks);
    br.half = walk.half;
    br.last_bits = c_in % 32 ? (1u << (c_in % 32)) - 1u : ~0u;
    return br;
}

// tiles of cb x pb blocks a wave, four waves along the pixels
inline void set_tile(DirectArgs& a, int cb, int pb)
{
    a.n_ctiles = (a.s.c_out + 32 * cb - 1) / (32 * cb);
    a.n_ptiles = (a.s.m + 128 * pb - 1) / (128 * pb);
    a.div_ct = DivBy::make(a.n_ctiles);
}

}  // namespace bcnn
