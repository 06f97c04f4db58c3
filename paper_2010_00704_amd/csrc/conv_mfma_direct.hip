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

// What a tile of this kernel costs, in microseconds: a launch with its latencies, a wave's chain of chunks, a
// wave's set-up and epilogue and its chunks where more waves than SIMDs (1024) share the issue slots.  The four
// numbers of each tile and kind of output are least-squares fits over 158 measured launches (graph replays, outputs on
// rotating buffers; 1x1 and 3x3, strides 1 and 2, 32 to 1024 channels on both sides, 25 to 430 000 pixels; rms error 8 to
// 15 %); choosing by them costs 1 % over the best of the tiles on average and 20 % at worst.
struct Cost { double fixed, chunk, wave, wave_chunk; };
struct TileCost { int tile, cb, pb, wc, wp, wk; Cost kind[3]; };     // kind: packed bits, int32 sums, module
static const TileCost TILES[] = {
    {DIRECT_1x1_K4, 1, 1, 1, 1, 4, {{2.49, 0.132, 0.050, 0.184}, {2.52, 0.144, 0.136, 0.151}, {2.77, 0.190, 0.267, 0.181}}},
    {DIRECT_2x2_K4, 2, 2, 1, 1, 4, {{2.89, 0.413, 0.587, 0.372}, {2.78, 0.500, 0.900, 0.306}, {3.80, 0.356, 1.403, 0.383}}},
    {DIRECT_2x1, 2, 1, 1, 4, 1, {{2.74, 0.299, 0.455, 0.215}, {2.83, 0.319, 1.039, 0.178}, {4.70, 0.289, 1.602, 0.215}}},
    {DIRECT_1x1, 1, 1, 1, 4, 1, {{2.63, 0.180, 0.238, 0.154}, {2.66, 0.209, 0.513, 0.130}, {3.68, 0.180, 0.790, 0.162}}},
};
// The same for the staged kernel's 2 x 4 tile (99 launches, C_in a multiple of 128, module calls in its plain form; rms 8,
// 20 and 10 %): workgroups of 128 channels x 256 pixels against 256 compute units.
static double staged_cost(const ConvShape& s, int kind)
{
    static const Cost KINDS[] = {{3.54, 0.594, 1.71, 0.191}, {6.00, 0.587, 5.08, 0.025}, {8.01, 0.575, 7.43, 0.165}};
    const Cost& c = KINDS[kind];
    const double chunks = (double)((s.ks * s.ks * (s.cw / 4) + 1) / 2);
    const double wgs = (double)((s.m + 255) / 256) * (double)((s.c_out + 127) / 128);
    return c.fixed + c.chunk * chunks + (c.wave + c.wave_chunk * chunks) * wgs / 256.0;
}

static int direct_mode(const ConvShape& s) { return s.cw < 4 ? WORDS : s.cw % 4 ? TAIL : UNITS; }
static int direct_units(const ConvShape& s)
{
    const int taps = s.ks * s.ks;
    return s.cw < 4 ? (taps * s.cw + 3) / 4 : taps * ((s.cw + 3) / 4);
}

int conv_mfma_direct_choose(const ConvShape& s, int kind, bool staged)
{
    const int chunks = (direct_units(s) + 1) / 2;
    int best = 0;
    double least = staged ? staged_cost(s, kind) : 1e30;
    for (const TileCost& t : TILES) {
        const double wgs = (double)((s.m + 32 * t.pb * t.wp - 1) / (32 * t.pb * t.wp)) *
                           (double)((s.c_out + 32 * t.cb * t.wc - 1) / (32 * t.cb * t.wc));
        const double waves = wgs * t.wc * t.wp * t.wk / 1024.0;
        const double mine = (double)((chunks + t.wk - 1) / t.wk);
        const Cost& c = t.kind[kind];
        const double cost = c.fixed + c.chunk * mine + (c.wave + c.wave_chunk * mine) * waves;
        if (cost < least) { least = cost; best = t.tile; }
    }
    return best;
}

hipError_t launch_conv_mfma_direct(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream)
{
    DirectArgs a{};
    a.s = s;
    a.n_ptiles = a.n_ctiles = 0;     // set with the tile
    const int mode = direct_mode(s);
    a.n_words = s.ks * s.ks * s.cw;
    a.per_tap = mode == WORDS ? s.cw : (s.cw + 3) / 4;
    a.n_units = direct_units(s);
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
