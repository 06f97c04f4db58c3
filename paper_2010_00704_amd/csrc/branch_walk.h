// How the direct kernel's branch mode walks the packed words of one tap (kernel: conv_mfma_direct_kernel.h).  Plain C++ on
// purpose: the kernel reads its words through these functions, and a host-only test walks every word count with them.
//
// A tap's cw words are split between the two lane halves of a wave: half h walks the words h * half_words .., one K-step a
// word, in groups.  The first `full` groups are four words that BOTH halves have whole, one 16-byte load without a
// check; what is left, one to four K-steps, is a last group of single words, each with its check: of an odd count the
// second half is one word short, and the word after its last one belongs to the next tap, pixel or branch.
#pragma once
#include "div_by.h"

#if defined(__HIPCC__)
#define BCNN_WALK_INLINE __host__ __device__ __forceinline__
#else
#define BCNN_WALK_INLINE inline
#endif

namespace bcnn {

struct BranchWalk {
    int cw;
    int half_words;     // K-steps of a tap
    int full;           // groups of four whole words
    int rest;           // single words of the last group (0: there is none)
    static BCNN_WALK_INLINE BranchWalk make(int cw)
    {
        const int half = (cw + 1) / 2;
        const int full = cw >> 3;                                                  // (cw / 2) / 4: the shorter half's
        return BranchWalk{cw, half, full, half - 4 * full};
    }
    BCNN_WALK_INLINE int groups() const { return full + (rest != 0); }
    BCNN_WALK_INLINE int steps(int g) const { return g < full ? 4 : rest; }        // K-steps of a group
    BCNN_WALK_INLINE int first(int h, int g) const { return h * half_words + 4 * g; }   // a half's first word of a group
    BCNN_WALK_INLINE bool real(int word) const { return word < cw; }                // of a single word
};

}  // namespace bcnn
