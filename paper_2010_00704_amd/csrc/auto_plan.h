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
// (up to 32 channels are one block of the direct kernel's tile whatever their number: 64 -> 16, 802 816 pixels 13.3 and 16.0)
inline bool direct_behind_on_bits(int ks, int cw, int c_out, int64_t outputs)
{
    if (ks != 1 || cw > 2) return false;
    return outputs >= (cw == 1 ? 4000000 : c_out <= 32 ? 6000000 : 15000000);
}

// Modules on a float stream that the streaming kernel does not take; has_*: which of the tensors the call has.  Rows leave the
// direct kernel in pieces of 128 bytes from many waves, which costs where there is little else (vector ALUs, or the
// staged kernel where it covers the call, and direct):
//   - without the stream or the bits out, 1x1 of up to two words: 64 -> 64 channels, 256 maps of 56 x 56 without the stream 44
//     and 50; 15 -> 64, 122 maps of 28 x 28 without the bits 13.3 and 16.0; 64 -> 320, 3000 pixels of it level;
//   - without identity, 1x1 of up to eight words, from 80 million outputs on: 64 -> 512, 240 maps of 56 x 56 345 and 443; 128 ->
//     512, 120 maps 181 and 222; 64 -> 256, 64 maps (51 million) 1.14 times ahead.
// Not where the rows are no whole 16-byte vectors, which the direct kernel reads and writes by unaligned vectors: 3x3, 64 -> 717, 30 maps of 56 x 56
// 267 and 157; 1x1, 64 -> 511 without identity, 240 maps 684 and 426; 64 -> 65 without the stream, 120 maps 47.5 and 40.2.
inline bool direct_behind_on_float_module(int ks, int cw, int c_out, bool has_id, bool has_r, bool has_x, int64_t outputs)
{
    if (ks != 1 || c_out % 4 != 0) return false;
    if (cw <= 2 && !(has_r && has_x)) return outputs >= 4000000;
    return cw <= 8 && !has_id && has_r && outputs >= 80000000;
}

// Branch sums that go on into a module's tail, `words` = branches x words per pixel: the same as for modules, and the vector ALUs
// walk all branches at once.  Streams that fit the last-level cache are ahead on the direct kernel (vector ALUs and direct):
// float, 128 channels x 2 -> 448, 120 maps of 56 x 56 266 and 317, 60 maps of 28 x 28 level; 320 x 2 1.2 times ahead; half, 32 -> 448 0.90
// times, 64 x 4 -> 448 1.1.  Rows that are no whole 16-byte vectors are ahead there too: 32 x 8 -> 451, 60 maps of 56 x 56, float 302 and 247,
// half 314 and 205.
inline bool direct_behind_on_branch_tail(int cw, int words, int c_out, bool half, int64_t outputs)
{
    if (cw % 8 == 0 || c_out % 4 != 0) return false;         // (whole units of eight words: not measured against the vector ALUs)
    return half ? outputs >= 80000000 && words <= 2 : outputs >= 40000000 && words <= 8;
}

}  // namespace bcnn
