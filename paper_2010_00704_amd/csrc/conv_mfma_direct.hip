// Launchers of the matrix-core convolution without LDS staging (kernel: conv_mfma_direct_kernel.h).
#include "conv_mfma_direct.h"
#include "conv_mfma_direct_kernel.h"

namespace bcnn {
namespace {

template <int CB, int PB, int WC, int WP, int WK, int OUT>
hipError_t launch_mode(DirectArgs a, int mode, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                       const ModuleEp& ep, hipStream_t stream)
{
    a.n_ctiles = (a.s.c_out + 32 * CB * WC - 1) / (32 * CB * WC);
    a.n_ptiles = (a.s.m + 32 * PB * WP - 1) / (32 * PB * WP);
    a.div_ct = DivBy::make(a.n_ctiles);
    const dim3 blocks((unsigned)(a.n_ptiles * a.n_ctiles)), threads(64 * WC * WP * WK);
    const DirectBranch none{};
    if (mode == UNITS)
        hipLaunchKernelGGL((conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, UNITS>), blocks, threads, 0, stream, a, x, w, thr, out, ep, none);
    else if (mode == TAIL)
        hipLaunchKernelGGL((conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, TAIL>), blocks, threads, 0, stream, a, x, w, thr, out, ep, none);
    else
        hipLaunchKernelGGL((conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, WORDS>), blocks, threads, 0, stream, a, x, w, thr, out, ep, none);
    return hipGetLastError();
}

template <int CB, int PB, int WC, int WP, int WK>
hipError_t launch_out(const DirectArgs& a, int mode, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                      const ModuleEp* ep, hipStream_t stream)
{
    const ModuleEp none{};
    if (ep && ep->half == REAL_BF16) return launch_mode<CB, PB, WC, WP, WK, OUT_MODULE + REAL_BF16>(a, mode, x, w, thr, out, *ep, stream);
    if (ep && ep->half) return launch_mode<CB, PB, WC, WP, WK, OUT_MODULE + REAL_F16>(a, mode, x, w, thr, out, *ep, stream);
    if (ep) return launch_mode<CB, PB, WC, WP, WK, OUT_MODULE + REAL_F32>(a, mode, x, w, thr, out, *ep, stream);
    if (thr) return launch_mode<CB, PB, WC, WP, WK, OUT_BITS>(a, mode, x, w, thr, out, none, stream);
    return launch_mode<CB, PB, WC, WP, WK, OUT_I32>(a, mode, x, w, thr, out, none, stream);
}

}  // namespace

bool conv_mfma_direct_supported(const ConvShape& s)
{
    const int64_t n_words = (int64_t)s.ks * s.ks * s.cw;
    const int64_t x_bytes = (int64_t)s.n * s.h * s.w * s.cw * 4;
    const int64_t w_bytes = (int64_t)s.c_out * n_words * 4;
    // fp32 sums stay exact (the K axis is padded to at most four words per tap and a chunk); 31-bit byte offsets
    // (c_out bound: a wave's rows of an output tensor by 31-bit offsets)
    return s.c_out <= (1 << 20) && (n_words + 3 * s.ks * s.ks + 8) * 32 < (1 << 22) && x_bytes < (1ll << 31) && w_bytes < (1ll << 31);
}

DirectChoice conv_mfma_direct_choose(const ConvShape& s, int kind, bool staged) { return direct_estimate(s.m, s.c_out, s.cw, s.ks, kind, staged); }

hipError_t launch_conv_mfma_direct(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream)
{
    DirectArgs a{};
    a.s = s;
    a.n_ptiles = a.n_ctiles = 0;     // set with the tile
    const int mode = direct_mode(s.cw);
    a.n_words = s.ks * s.ks * s.cw;
    a.per_tap = mode == WORDS ? s.cw : (s.cw + 3) / 4;
    a.n_units = direct_units(s.cw, s.ks);
    a.n_chunks = (a.n_units + 1) / 2;
    a.z = 256 * a.n_chunks - s.k;
    a.x_bytes = (int32_t)((int64_t)s.n * s.h * s.w * s.cw * 4);
    a.w_bytes = (int32_t)((int64_t)s.c_out * a.n_words * 4);
    a.row_jump = (s.w - s.ks) * s.cw;
    a.div_hw = DivBy::make(s.ho * s.wo);
    a.div_wo = DivBy::make(s.wo);
    a.div_tap = DivBy::make(a.per_tap);
    switch (tile) {
        case DIRECT_1x1_K4: return launch_out<1, 1, 1, 1, 4>(a, mode, x, w, thr, out, ep, stream);
        case DIRECT_2x2_K4: return launch_out<2, 2, 1, 1, 4>(a, mode, x, w, thr, out, ep, stream);
        case DIRECT_2x1: return launch_out<2, 1, 1, 4, 1>(a, mode, x, w, thr, out, ep, stream);
        case DIRECT_1x1: return launch_out<1, 1, 1, 4, 1>(a, mode, x, w, thr, out, ep, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bcnn
