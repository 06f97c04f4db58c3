// Where AUTO leaves the direct matrix-core kernel out: launches of few packed words per output that their output binds.
// Plain C++ on purpose: the entry points use these rules, and a host-only test checks measured calls.
// (`outputs` = pixels x output channels; times in us)
#pragma once
#include <stdint.h>

namespace bcnn {

// Packed bits, cw words per pixel.  With one or two words of a 1x1 filter the direct kernel's waves do little but their
// set-up, and a lane of the vector ALUs is through them in a few instructions.
// Measured (vector ALUs and direct): 64 -> 64 channels, 802 816 pixels 17.3 and 22.2, 200 704 pixels 7.9 and 7.8; 32 -> 128,
// 200 704 pixels 9.5 and 12.2, 50 176 pixels 5.1 and 5.3; 64 -> 512, 50 176 pixels 12.3 and 12.4.  Three words, and one word
// under a 3x3 filter, are ahead on the matrix cores or level at every size.
inline bool direct_behind_on_bits(int ks, int cw, int64_t outputs)
{
    return ks == 1 && ((cw == 1 && outputs >= 4000000) || (cw == 2 && outputs >= 15000000));
}

}  // namespace bcnn
