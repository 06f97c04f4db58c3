// The direct kernel's form with shared weights (kernel: conv_mfma_direct_kernel.h, WIDE > 0; tiles and their choice:
// shared_plan.h).
#pragma once
#include "bcnn_common.h"
#include "shared_plan.h"

namespace bcnn {

// A tile of this form, or SHARED_NONE: `other`, the choice among the other kernels, is the better one.  The form covers
// what conv_mfma_direct_supported() covers.
int conv_mfma_shared_choose(const ConvShape& s, int kind, const DirectChoice& other);
// thr == nullptr: int32 sums, else packed bits; ep != nullptr: module epilogue (thr and out are ignored)
hipError_t launch_conv_mfma_shared(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream);


// the same in branch mode (tiles SHARED_1x1, SHARED_2x1)
hipError_t launch_conv_branches_shared(const ConvShape& s, const BranchArgs& b, int tile, hipStream_t stream);

}  // namespace bcnn
