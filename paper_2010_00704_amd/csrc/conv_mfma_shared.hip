// Launchers of the direct kernel's form with shared weights (kernel: conv_mfma_direct_kernel.h).
#include "conv_mfma_shared.h"
#include "conv_mfma_direct_kernel.h"
#include "shared_args.h"

namespace bcnn {
namespace {

template <int CB, int PB, int WIDE>
hipError_t launch_out(DirectArgs a, const DirectBranch& br, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out, const ModuleEp* ep,
                      hipStream_t stream)
{
    set_tile(a, CB, PB);
    const dim3 blocks((unsigned)(a.n_ptiles * a.n_ctiles)), threads(256);
    const ModuleEp e = ep ? *ep : ModuleEp{};
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, a, x, w, thr, out, e, br); };
    if (ep) {
        if constexpr (CB * PB < 4) {
            if (ep->half == REAL_BF16) go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT_MODULE + REAL_BF16, UNITS, WIDE>);
            else if (ep->half) go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT_MODULE + REAL_F16, UNITS, WIDE>);
            else go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT_MODULE + REAL_F32, UNITS, WIDE>);
        } else return hipErrorInvalidValue;
    } else if (thr) go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT_BITS, UNITS, WIDE>);
    else go(conv_mfma_direct_kernel<CB, PB, 1, 4, 1, OUT_I32, UNITS, WIDE>);
    return hipGetLastError();
}

template <int CB, int PB>
hipError_t launch_wide(const DirectArgs& a, const DirectBranch& br, int wide, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out, const ModuleEp* ep,
                       hipStream_t stream)
{
    switch (wide) {
        case 1: return launch_out<CB, PB, 1>(a, br, x, w, thr, out, ep, stream);
        case 2: return launch_out<CB, PB, 2>(a, br, x, w, thr, out, ep, stream);
        case 3: return launch_out<CB, PB, 3>(a, br, x, w, thr, out, ep, stream);
        case 5: return launch_out<CB, PB, 5>(a, br, x, w, thr, out, ep, stream);
        default: return launch_out<CB, PB, 4>(a, br, x, w, thr, out, ep, stream);
    }
}

}  // namespace

int conv_mfma_shared_choose(const ConvShape& s, int kind, const DirectChoice& other) { return shared_choose(s.m, s.c_out, s.cw, s.ks, s.stride, kind, other); }

hipError_t launch_conv_mfma_shared(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream)
{
    const SharedWalk walk = SharedWalk::make(s.cw, s.ks * s.ks);
    const DirectArgs a = shared_args(s, s.ks * s.ks, walk);
    const DirectBranch br = shared_extra(s, walk);
    switch (tile) {
        case SHARED_1x1: return launch_wide<1, 1>(a, br, walk.wide, x, w, thr, out, ep, stream);
        case SHARED_2x1: return launch_wide<2, 1>(a, br, walk.wide, x, w, thr, out, ep, stream);
        case SHARED_2x2: return launch_wide<2, 2>(a, br, walk.wide, x, w, thr, out, ep, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bcnn
