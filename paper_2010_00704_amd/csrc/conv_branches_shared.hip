// Branch mode of the matrix-core convolution whose workgroups share expanded weights (kernel: conv_mfma_direct_kernel.h).
#include "conv_mfma_shared.h"
#include "conv_mfma_direct_kernel.h"
#include "shared_args.h"

namespace bcnn {
namespace {

template <int CB, int PB, int WIDE, int OUT>
hipError_t launch_pad(DirectArgs a, const BranchArgs& b, const DirectBranch& br, hipStream_t stream)
{
    set_tile(a, CB, PB);
    const dim3 blocks((unsigned)(a.n_ptiles * a.n_ctiles)), threads(256);
    const ModuleEp ep = b.tail ? *b.tail : ModuleEp{};
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, a, b.x, b.w, (const int32_t*)nullptr, b.out, ep, br);
    };
    // (without padding every tap is inside)
    if (a.s.pad && b.zero_pad) go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT, BRANCH + PAD_NOTHING, WIDE>);
    else if (a.s.pad && b.pad_words) go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT, BRANCH + PAD_OPERAND, WIDE>);
    else go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT, BRANCH + PAD_NONE, WIDE>);
    return hipGetLastError();
}

template <int CB, int PB, int WIDE>
hipError_t launch_out(const DirectArgs& a, const BranchArgs& b, const DirectBranch& br, hipStream_t stream)
{
    if (b.tail && b.tail->half) return launch_pad<CB, PB, WIDE, OUT_MODULE + REAL_F16>(a, b, br, stream);
    if (b.tail) return launch_pad<CB, PB, WIDE, OUT_MODULE + REAL_F32>(a, b, br, stream);
    if (b.fused) return launch_pad<CB, PB, WIDE, OUT_BITS>(a, b, br, stream);
    return launch_pad<CB, PB, WIDE, OUT_I32>(a, b, br, stream);
}

template <int CB, int PB>
hipError_t launch_wide(const DirectArgs& a, int wide, const BranchArgs& b, const DirectBranch& br, hipStream_t stream)
{
    switch (wide) {
        case 1: return launch_out<CB, PB, 1>(a, b, br, stream);
        case 2: return launch_out<CB, PB, 2>(a, b, br, stream);
        case 3: return launch_out<CB, PB, 3>(a, b, br, stream);
        case 5: return launch_out<CB, PB, 5>(a, b, br, stream);
        default: return launch_out<CB, PB, 4>(a, b, br, stream);
    }
}

}  // namespace

hipError_t launch_conv_branches_shared(const ConvShape& s, const BranchArgs& b, int tile, hipStream_t stream)
{
    const SharedWalk walk = SharedWalk::make(s.cw, b.branches);
    DirectArgs a = shared_args(s, b.branches, walk);
    const int64_t one = (int64_t)s.n * s.h * s.w * s.cw * 4;
    a.x_bytes = (int32_t)(b.x_branch_stride ? (int64_t)(b.branches - 1) * b.x_branch_stride * 4 + one : one);
    a.tap_step = (int32_t)b.x_branch_stride;
    DirectBranch br = shared_extra(s, walk);
    br.scale = b.scale;
    br.bias = b.bias;
    br.pad_words = b.pad_words;
    switch (tile) {
        case SHARED_1x1: return launch_wide<1, 1>(a, walk.wide, b, br, stream);
        case SHARED_2x1: return launch_wide<2, 1>(a, walk.wide, b, br, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bcnn
