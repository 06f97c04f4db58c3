// When a call takes the direct kernel's form with shared weights (conv_mfma_direct_kernel.h, WIDE > 0), with which tile, and how
// that form walks K.  Plain C++ on purpose: the launchers use these functions, and a host-only test walks every word count
// with them.
#pragma once
#include <initializer_list>
#include <limits.h>
#include <stdint.h>

#include "direct_plan.h"

namespace bcnn {

// Tiles: 32-channel x 32-pixel blocks of a wave; four waves along the pixels.
enum { SHARED_NONE = 0, SHARED_1x1, SHARED_2x1, SHARED_2x2 };

// How a tap's cw words are walked: lane half 0 takes the first `half` of them, half 1 the rest, one K-step a word of each, in
// groups of `wide` words a load.  Narrow taps (up to four words) go several to a group of four K-steps.  Words that do not
// exist are zeros on the weights' side.
struct SharedWalk {
    int half, wide, per_tap, groups;
    static SharedWalk make(int cw, int taps)
    {
        SharedWalk r;
        r.half = (cw + 1) / 2;
        r.wide = r.half < 3 ? r.half : 4;
        if (r.half >= 3)                                     // fewest K-steps; whole 16-byte loads where level
            for (int wide : {5, 3})
                if ((r.half + wide - 1) / wide * wide < (r.half + r.wide - 1) / r.wide * r.wide) r.wide = wide;
        r.per_tap = (r.half + r.wide - 1) / r.wide;
        r.groups = r.wide < 3 ? (taps * r.wide + 3) / 4 : taps * r.per_tap;
        return r;
    }
    int steps(int taps) const { return wide < 3 ? taps * wide : groups * wide; }       // K-steps that are multiplied
};

// Estimated times in microseconds, as for the tiles of direct_plan.h: a launch, its K-steps, and per workgroup and compute unit
// (256) its set-up with the epilogue and its K-steps.  Fits over 860 calls (500 to 440 000 pixels, 32 to 1024 channels on both
// sides, 1x1 and 3x3, strides 1 and 2; graph replays), rms 8 to 11 % for bits and sums, 11 to 14 % for modules.
enum { SHARED_BITS = 0, SHARED_SUMS = 1, SHARED_HALF = 2, SHARED_FLOAT = 3 };
struct SharedCost { double fixed, step, wg, wg_step; };
struct SharedTile { int tile, cb, pb; SharedCost kind[4]; };
static const SharedTile SHARED_TILES[] = {
    {SHARED_1x1, 1, 1, {{3.04, 0.0411, 0.341, 0.0302}, {3.55, 0.0424, 0.603, 0.0285}, {4.24, 0.0442, 1.27, 0.0236}, {4.50, 0.0420, 1.47, 0.0249}}},
    {SHARED_2x1, 2, 1, {{3.14, 0.0738, 0.349, 0.0421}, {3.79, 0.0785, 1.10, 0.0327}, {5.27, 0.0859, 2.30, 0.0189}, {6.11, 0.0748, 2.61, 0.0310}}},
    {SHARED_2x2, 2, 2, {{3.49, 0.1099, 0.498, 0.0618}, {4.53, 0.1208, 2.28, 0.0325}, {0, 0, 0, 0}, {0, 0, 0, 0}}},
};
inline double shared_cost(const SharedCost& c, int cb, int pb, int m, int c_out, int steps)
{
    const double wgs = (double)(((int64_t)m + 128 * pb - 1) / (128 * pb)) * (double)((c_out + 32 * cb - 1) / (32 * cb)) / 256.0;
    return c.fixed + c.step * steps + (c.wg + c.wg_step * steps) * wgs;
}

// Words a tap up to which this form is taken from the staged kernel and from the tiles that split K (us, other and this):
//   - 32 under a 3x3 filter, and under stride 2 against the staged kernel, where the fits end: 673 of 916 calls of 33 to 48 words were
//     behind, 9 % on average (half module, 1152 -> 512, stride 2, 32 585 pixels 83 and 130; sums, 1083 -> 800, 14 maps of 28 x 28
//     49 and 63; bits, 1x1, 1152 -> 896, stride 2, 16 611 pixels 11.5 and 16.5)
//   - fewer under stride 2, where no two rows share their taps' lines (half module, 562 -> 268, 9016 pixels 14.8 and 16.9; bits of 24
//     and 28 words 0.87 times the staged kernel)
//   - fewer where c_out fills the staged kernel's 128-channel tiles: half modules of 24 and 28 words 1.05
//     times that kernel on average, but 32 of 119 behind by up to 15 %, of 32 words 0.98, and under stride 2 of 24 and 28 0.95; sums of 16 and
//     20 words 0.95; all of them ahead below (1.1 to 1.2)
inline int shared_words(int c_out, int ks, int stride, int kind, int other)
{
    if (ks == 1) return other == DIRECT_NONE && stride > 1 ? 32 : INT_MAX;
    if (other != DIRECT_NONE) return stride > 1 && kind != SHARED_BITS ? 16 : 32;
    if (kind == SHARED_BITS) return stride > 1 ? 20 : 32;
    if (c_out % 128 != 0 || kind == SHARED_FLOAT) return 32;
    return kind == SHARED_SUMS ? 12 : 20;
}

// The tile, or SHARED_NONE where `other` is estimated to be as good.  Against the tiles that do not split K this form may be
// estimated a tenth behind: their estimates are that much too low on the calls that this one is ahead on.  Not so for sums,
// which their stores bind, and for modules whose taps are whole 16-byte units (a multiple of four words), which those tiles walk without masks
// (us, other and this: half module, 3x3, 110 -> 88, 73 maps of 41 x 41 20.8 and 23.0; 117 -> 224, 25 maps of 39 x 39 17.6 and 19.5;
// of 265 such calls 88 were more than 3 % behind, 1 is).
// Over 3000 calls that the estimates without this rule and that of shared_words() give to this form: bits 1.29 times the other choice on average,
// sums 1.26, half modules 1.12, float ones 1.13; 16 of them more than 5 % behind it, 13 % at worst (sums, 3x3, 32 -> 1007,
// 80 556 pixels 76 and 87), and 61 of 3500 more that the staged kernel covers, 14 % at worst (what is left of the estimates' errors).  (us, other and this: bits, 3x3, 320 -> 192, 39 maps of 38 x 38
// 27.9 and 16.3; 64 -> 64, 156 maps of 25 x 28 9.8 and 6.9; 1x1, 704 -> 704, 40 maps of 26 x 26 14.9 and 10.8; sums, 3x3, 468 -> 39,
// 191 maps of 37 x 36 52 and 38.)
inline int shared_choose(int m, int c_out, int cw, int ks, int stride, int kind, const DirectChoice& other)
{
    // sums of a 1x1 filter are bound by their store, which the other tiles keep busier (64 -> 672, 46 maps of 51 x 29 30.7 and 33.9)
    if (kind == SHARED_SUMS && ks == 1) return SHARED_NONE;
    const bool whole_k = other.tile == DIRECT_2x1 || other.tile == DIRECT_1x1;
    if (!whole_k && cw > shared_words(c_out, ks, stride, kind, other.tile)) return SHARED_NONE;
    const int taps = ks * ks, steps = SharedWalk::make(cw, taps).steps(taps);
    const bool too_low = whole_k && (kind == SHARED_BITS || (kind != SHARED_SUMS && cw % 4 != 0));
    double least = other.cost * (too_low ? 1.1 : 1.0);
    int best = SHARED_NONE;
    for (const SharedTile& t : SHARED_TILES) {
        const SharedCost& c = t.kind[kind];
        if (c.fixed == 0) continue;                          // (a 2 x 2 tile leaves a module no registers for its identity)
        const double cost = shared_cost(c, t.cb, t.pb, m, c_out, steps);
        if (cost < least) { least = cost; best = t.tile; }
    }
    return best;
}

// Branch calls (P shifted or parallel 1x1 branches, a real scale each).  Three forms of the direct kernel:
//   - taps apart: the four waves of a 32 x 32 block take whole taps and leave their sums in LDS, where they are scaled and added in
//     order: a quarter of the chain of K-steps.  Up to three blocks a compute unit; over 700 calls 2, 2.5, 3.5 and 4 are 0.3 to
//     2 % slower on average, none of them a call of more.  (us, the waves side by side and this: bits, 3x3, 384 -> 384, 2 maps
//     of 13 x 13 12.9 and 6.6; 128 -> 128, 8 maps of 10 x 10, float tail 10.5 and 5.0)
//   - every wave its own operands (direct_plan.h): at most eight words in all, of at most two a tap, or one branch of up to
//     four words, so that there is little expansion to share (64 x 3 -> 128, 29 376 pixels, float 7.1, with shared weights 8.7;
//     one branch, 96 -> 96, 242 452 pixels, bits 13.5 and 16.4; bits of such calls 11 % on average, sums 3 %, tails level)
//   - shared weights for the rest, 2 x 1 blocks a wave from twelve blocks a compute unit on (8, 10, 16 and 24 are 0.5 to
//     1.5 % slower on average; with a float tail, whose epilogue weighs more, direct_plan.h's estimates, and never for narrow taps:
//     96 x 3 -> 416, 286 117 pixels 199 with 1 x 1 blocks, 258 with 2 x 1) and where their second block does not idle too often: not for one or
//     three blocks of 32 channels, and five under a half tail (32 x 9 -> 81, 184 730 pixels, half tail 60.6, with 1 x 1 blocks 51)
// Together 1.33 to 1.40 times the second form alone over 700 calls of all kinds (32 to 1024 channels, 50 to 200 000 pixels, 2 to 9
// branches).  Of 3000 more calls above three blocks a compute unit, 14 are more than 5 % behind the second form, 10 % at worst (most of
// them tails of nine narrow taps with pad words, which have been faster since); 35 were before single branches, narrow taps and idle
// blocks had their rules, 24 % at worst.
enum { BRANCH_OWN = 0, BRANCH_APART, BRANCH_SHARED };
constexpr int APART_TAPS = 9;                                // sums of taps that fit LDS
struct BranchChoice { int form, tile; };
inline bool branches_apart(int m, int c_out, int branches)
{
    return branches <= APART_TAPS && (((int64_t)m + 31) / 32) * ((c_out + 31) / 32) <= 3 * 256;
}
inline BranchChoice branches_choose(int m, int c_out, int cw, int branches, bool tail, bool half)
{
    const int64_t blocks = (((int64_t)m + 31) / 32) * ((c_out + 31) / 32);
    if (branches_apart(m, c_out, branches)) return BranchChoice{BRANCH_APART, DIRECT_1x1_K4};
    const int own = branches_direct_choose(m, c_out, cw, branches, tail, half);
    if ((cw <= 2 && cw * branches <= 8) || (branches == 1 && cw <= 4)) return BranchChoice{BRANCH_OWN, own};
    const int across = (c_out + 31) / 32;
    const bool filled = across % 2 == 0 || across > (tail && half ? 5 : 3);
    const bool wide = filled && (tail && !half ? cw > 4 && own != DIRECT_1x1 : blocks >= 12 * 256);
    return BranchChoice{BRANCH_SHARED, wide ? SHARED_2x1 : SHARED_1x1};
}

}  // namespace bcnn
