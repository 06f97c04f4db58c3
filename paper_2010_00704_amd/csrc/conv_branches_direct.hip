// Branch mode of the matrix-core convolution without LDS staging (kernel: conv_mfma_direct_kernel.h).
#include "conv_mfma_direct.h"
#include "conv_mfma_direct_kernel.h"

namespace bcnn {
namespace {

template <int CB, int PB, int WC, int WP, int WK, int OUT>
hipError_t launch_pad(DirectArgs a, const BranchArgs& b, const DirectBranch& br, hipStream_t stream)
{
    a.n_ctiles = (a.s.c_out + 32 * CB * WC - 1) / (32 * CB * WC);
    a.n_ptiles = (a.s.m + 32 * PB * WP - 1) / (32 * PB * WP);
    a.div_ct = DivBy::make(a.n_ctiles);
    const dim3 blocks((unsigned)(a.n_ptiles * a.n_ctiles)), threads(64 * WC * WP * WK);
    const ModuleEp ep = b.tail ? *b.tail : ModuleEp{};
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, a, b.x, b.w, (const int32_t*)nullptr, b.out, ep, br);
    };
    if constexpr (WK > 1) {
        if (a.s.pad && b.zero_pad) go(conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, BRANCH + PAD_NOTHING>);
        else if (a.s.pad && b.pad_words) go(conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, BRANCH + PAD_OPERAND>);
        else go(conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, BRANCH + PAD_NONE>);
    } else {
        // (nine taps are more than this form is chosen for: shared_plan.h)
        if (a.s.pad) return hipErrorInvalidValue;
        go(conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, BRANCH + PAD_NONE>);
    }
    return hipGetLastError();
}

template <int CB, int PB, int WC, int WP, int WK>
hipError_t launch_out(const DirectArgs& a, const BranchArgs& b, const DirectBranch& br, hipStream_t stream)
{
    if (b.tail && b.tail->half) return launch_pad<CB, PB, WC, WP, WK, OUT_MODULE + REAL_F16>(a, b, br, stream);
    if (b.tail) {
        // (the 2 x 2 tile has no registers for the float stream's identity vectors: never chosen for it)
        if constexpr (CB * PB < 4) return launch_pad<CB, PB, WC, WP, WK, OUT_MODULE + REAL_F32>(a, b, br, stream);
        else return hipErrorInvalidValue;
    }
    if (b.fused) return launch_pad<CB, PB, WC, WP, WK, OUT_BITS>(a, b, br, stream);
    return launch_pad<CB, PB, WC, WP, WK, OUT_I32>(a, b, br, stream);
}

int64_t branch_x_bytes(const ConvShape& s, const BranchArgs& b)
{
    const int64_t one = (int64_t)s.n * s.h * s.w * s.cw * 4;
    return b.x_branch_stride ? (int64_t)(b.branches - 1) * b.x_branch_stride * 4 + one : one;
}

}  // namespace

bool conv_branches_direct_supported(const ConvShape& s, const BranchArgs& b)
{
    const int64_t w_bytes = (int64_t)s.c_out * b.branches * s.cw * 4;
    // a branch's sum (K padded to an even number of words) stays exact in fp32; 31-bit byte offsets
    return b.branches <= MAX_BRANCHES && s.c_out <= (1 << 20) && ((int64_t)s.cw + 1) * 32 < (1 << 22) && branch_x_bytes(s, b) < (1ll << 31) && w_bytes < (1ll << 31);
}

hipError_t launch_conv_branches_direct(const ConvShape& s, const BranchArgs& b, int tile, hipStream_t stream)
{
    DirectArgs a{};
    a.s = s;
    a.taps = b.branches;
    a.n_words = b.branches * s.cw;
    a.z = 64 * BranchWalk::make(s.cw).half_words - s.k / (s.ks * s.ks);   // of one branch
    a.x_bytes = (int32_t)branch_x_bytes(s, b);
    a.w_bytes = (int32_t)((int64_t)s.c_out * a.n_words * 4);
    a.pad_bytes = a.n_words * 4;
    a.row_jump = (s.w - s.ks) * s.cw;
    a.tap_step = (int32_t)b.x_branch_stride;
    a.div_hw = DivBy::make(s.ho * s.wo);
    a.div_wo = DivBy::make(s.wo);
    const DirectBranch br{b.scale, b.bias, b.pad_words, 0, 0u};
    switch (tile) {
        case DIRECT_1x1_K4: return b.branches <= APART_TAPS ? launch_out<1, 1, 1, 1, 4>(a, b, br, stream) : hipErrorInvalidValue;
        case DIRECT_1x1: return launch_out<1, 1, 1, 4, 1>(a, b, br, stream);
        case DIRECT_2x1: return launch_out<2, 1, 1, 4, 1>(a, b, br, stream);
        case DIRECT_2x2: return launch_out<2, 2, 1, 4, 1>(a, b, br, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bcnn
