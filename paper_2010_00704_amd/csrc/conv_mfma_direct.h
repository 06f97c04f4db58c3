// The matrix-core convolution without LDS staging (kernel: conv_mfma_direct_kernel.h; launchers: conv_mfma_direct.hip,
// conv_branches_direct.hip; tiles and their choice: direct_plan.h).
#pragma once
#include "bcnn_common.h"
#include "direct_plan.h"

namespace bcnn {

bool conv_mfma_direct_supported(const ConvShape& s);
// A tile and its estimated time, or DIRECT_NONE: the staged kernel (direct_plan.h).
DirectChoice conv_mfma_direct_choose(const ConvShape& s, int kind, bool staged);
// thr == nullptr: int32 sums, else packed bits; ep != nullptr: module epilogue (thr and out are ignored)
hipError_t launch_conv_mfma_direct(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream);

// the same in branch mode (tiles DIRECT_1x1, DIRECT_2x1, DIRECT_2x2: four waves along the pixels; DIRECT_1x1_K4: four waves
// that take whole taps of up to APART_TAPS branches)
bool conv_branches_direct_supported(const ConvShape& s, const BranchArgs& b);
hipError_t launch_conv_branches_direct(const ConvShape& s, const BranchArgs& b, int tile, hipStream_t stream);

// 1x1 modules of at most eight words per pixel, plain case (conv_mfma_stream.hip)
bool conv_mfma_stream_supported(const ConvShape& s, const ModuleEp& ep);
hipError_t launch_conv_mfma_stream(const ConvShape& s, const uint32_t* x, const uint32_t* w, const ModuleEp& ep,
                                   hipStream_t stream);

}  // namespace bcnn
