// The matrix-core convolution without LDS staging (kernel and launcher: conv_mfma_direct.hip).
#pragma once
#include "bcnn_common.h"

namespace bcnn {

// Tiles: 32-channel x 32-pixel blocks of a wave; _K4: four waves split K, otherwise four waves side by side
// along the pixels.
enum { DIRECT_NONE = 0, DIRECT_1x1_K4, DIRECT_2x2_K4, DIRECT_2x1, DIRECT_1x1, DIRECT_2x2 };

bool conv_mfma_direct_supported(const ConvShape& s);
// The tile with the least estimated time for an output of that kind; DIRECT_NONE if `staged` (the staged matrix-core kernel covers the call)
// and that kernel is estimated to be faster.
enum { KIND_BITS_OUT = 0, KIND_SUMS_OUT = 1, KIND_MODULE_OUT = 2 };
int conv_mfma_direct_choose(const ConvShape& s, int kind, bool staged);
// thr == nullptr: int32 sums, else packed bits; ep != nullptr: module epilogue (thr and out are ignored)
hipError_t launch_conv_mfma_direct(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream);

// the same in branch mode (tiles DIRECT_1x1, DIRECT_2x1, DIRECT_2x2: four waves along the pixels)
bool conv_branches_direct_supported(const ConvShape& s, const BranchArgs& b);
int conv_branches_direct_choose(const ConvShape& s, const BranchArgs& b);
hipError_t launch_conv_branches_direct(const ConvShape& s, const BranchArgs& b, int tile, hipStream_t stream);

// 1x1 modules of at most eight words per pixel, plain case (conv_mfma_stream.hip)
bool conv_mfma_stream_supported(const ConvShape& s, const ModuleEp& ep);
hipError_t launch_conv_mfma_stream(const ConvShape& s, const uint32_t* x, const uint32_t* w, const ModuleEp& ep,
                                   hipStream_t stream);

}  // namespace bcnn
