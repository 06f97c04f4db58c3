// Which tile of the direct matrix-core kernel a call takes (kernel: conv_mfma_direct_kernel.h), or whether the staged kernel
// takes it.  Plain C++ on purpose: the launchers use these functions, and a host-only test checks which tiles and K
// walks the GPU tests' shapes reach.
#pragma once
#include <stdint.h>

#include "branch_walk.h"

namespace bcnn {

// Tiles: 32-channel x 32-pixel blocks of a wave; _K4: four waves split K, otherwise four waves side by side
// along the pixels.
enum { DIRECT_NONE = 0, DIRECT_1x1_K4, DIRECT_2x2_K4, DIRECT_2x1, DIRECT_1x1, DIRECT_2x2 };

// How K is walked: whole 16-byte units per tap; the same with a last unit that shares words with its neighbour; word by word.
enum { UNITS = 0, TAIL = 1, WORDS = 2 };
inline int direct_mode(int cw) { return cw < 4 ? WORDS : cw % 4 ? TAIL : UNITS; }
inline int direct_units(int cw, int ks)
{
    const int taps = ks * ks;
    return cw < 4 ? (taps * cw + 3) / 4 : taps * ((cw + 3) / 4);
}

// Kinds of output.  A module is plain where the staged kernel's epilogue has a fast form: whole 128-channel tiles, every
// part of the module present; else general.
enum { KIND_BITS_OUT = 0, KIND_SUMS_OUT = 1, KIND_MODULE_PLAIN = 2, KIND_MODULE_GENERAL = 3 };

// What a tile of this kernel costs, in microseconds: a launch with its latencies, a wave's chain of chunks, a
// wave's set-up and epilogue and its chunks where more waves than SIMDs (1024) share the issue slots.  The four
// numbers of each tile and kind of output are least-squares fits over 158 measured launches (graph replays, outputs on
// rotating buffers; 1x1 and 3x3, strides 1 and 2, 32 to 1024 channels on both sides, 25 to 430 000 pixels; rms error 8 to
// 15 %); choosing by them costs 1 % over the best of the tiles on average and 20 % at worst.  (To fit them again: time every
// tile, forced in the launcher, over such launches, and solve for the four numbers by non-negative least squares on the
// relative error.)
struct DirectCost { double fixed, chunk, wave, wave_chunk; };
struct DirectTile { int tile, cb, pb, wc, wp, wk; DirectCost kind[3]; };     // kind: packed bits, int32 sums, module
static const DirectTile DIRECT_TILES[] = {
    {DIRECT_1x1_K4, 1, 1, 1, 1, 4, {{2.49, 0.132, 0.050, 0.184}, {2.52, 0.144, 0.136, 0.151}, {2.77, 0.190, 0.267, 0.181}}},
    {DIRECT_2x2_K4, 2, 2, 1, 1, 4, {{2.89, 0.413, 0.587, 0.372}, {2.78, 0.500, 0.900, 0.306}, {3.80, 0.356, 1.403, 0.383}}},
    {DIRECT_2x1, 2, 1, 1, 4, 1, {{2.74, 0.299, 0.455, 0.215}, {2.83, 0.319, 1.039, 0.178}, {4.70, 0.289, 1.602, 0.215}}},
    {DIRECT_1x1, 1, 1, 1, 4, 1, {{2.63, 0.180, 0.238, 0.154}, {2.66, 0.209, 0.513, 0.130}, {3.68, 0.180, 0.790, 0.162}}},
};
// The same for the staged kernel's 2 x 4 tile (99 launches, C_in a multiple of 128; rms 8, 20, 10 and 18 %): workgroups of
// 128 channels x 256 pixels against 256 compute units.
static const DirectCost STAGED_COSTS[] = {{3.54, 0.594, 1.71, 0.191}, {6.00, 0.587, 5.08, 0.025}, {8.01, 0.575, 7.43, 0.165}, {15.5, 0.610, 7.10, 0.200}};
inline double staged_cost(int m, int c_out, int cw, int ks, int kind)
{
    const DirectCost& c = STAGED_COSTS[kind];
    const double chunks = (double)((ks * ks * (cw / 4) + 1) / 2);
    const double wgs = (double)(((int64_t)m + 255) / 256) * (double)((c_out + 127) / 128);
    return c.fixed + c.chunk * chunks + (c.wave + c.wave_chunk * chunks) * wgs / 256.0;
}

// The estimates are 8 to 20 % off, so the direct kernel has to be ahead by more than that in its estimate where the staged one
// is the established choice.  Over 413 bits and sums calls and 1500 modules, all timed on both kernels, these weights
// leave nothing more than 5 % behind the staged kernel but three general modules (11 % at worst; unweighted 26 %; us, staged
// and direct: bits 1x1, 256 -> 960, 17 maps of 56 x 56 under stride 2 5.8 and 7.9; plain float module, 1x1, 1024 -> 128, 64 maps
// of 28 x 28 17.3 and 22.8), and cost 1 % over the best choice on average.  General modules of few chunks are ahead on the
// direct kernel wherever measured.
static const double STAGED_BIAS[] = {0.85, 0.95, 0.71, 0.85};

// The tile with the least estimated time, and that time; DIRECT_NONE if `staged` (the staged matrix-core kernel covers the
// call) and that kernel is the better choice.
struct DirectChoice { int tile; double cost; };
inline DirectChoice direct_estimate(int m, int c_out, int cw, int ks, int kind, bool staged)
{
    const int chunks = (direct_units(cw, ks) + 1) / 2;
    int best = DIRECT_NONE;
    const bool weigh = staged && !(kind == KIND_MODULE_GENERAL && chunks < 9);
    const double rival = weigh ? staged_cost(m, c_out, cw, ks, kind) : 1e30;
    double least = weigh ? STAGED_BIAS[kind] * rival : 1e30;
    for (const DirectTile& t : DIRECT_TILES) {
        const double wgs = (double)(((int64_t)m + 32 * t.pb * t.wp - 1) / (32 * t.pb * t.wp)) *
                           (double)((c_out + 32 * t.cb * t.wc - 1) / (32 * t.cb * t.wc));
        const double waves = wgs * t.wc * t.wp * t.wk / 1024.0;
        const double mine = (double)((chunks + t.wk - 1) / t.wk);
        const DirectCost& c = t.kind[kind < KIND_MODULE_PLAIN ? kind : KIND_MODULE_PLAIN];
        const double cost = c.fixed + c.chunk * mine + (c.wave + c.wave_chunk * mine) * waves;
        if (cost < least) { least = cost; best = t.tile; }
    }
    return DirectChoice{best, best == DIRECT_NONE ? rival : least};
}

// Branch mode: estimated time of a tile as above, with a wave's chain of groups of four K-steps in place of chunks.
// Fits over 74 calls; rms error 14 to 19 %, the choice 1 to 2 % over the best tile on average, 24 % at worst.
struct BranchTile { int tile, cb, pb; DirectCost plain, tail; };
static const BranchTile BRANCH_TILES[] = {
    {DIRECT_1x1, 1, 1, {2.88, 0.421, 0.188, 0.165}, {3.97, 0.363, 0.984, 0.176}},
    {DIRECT_2x1, 2, 1, {3.76, 0.586, 0.696, 0.233}, {5.98, 0.461, 1.685, 0.311}},
    {DIRECT_2x2, 2, 2, {4.53, 0.722, 1.791, 0.311}, {7.20, 0.708, 3.077, 0.457}},
};
// (the 2 x 2 tile has no registers for a float tail's identity vectors)
inline int branches_direct_choose(int m, int c_out, int cw, int branches, bool tail, bool half)
{
    const double groups = (double)branches * (double)BranchWalk::make(cw).groups();
    int best = DIRECT_1x1;
    double least = 1e30;
    for (const BranchTile& t : BRANCH_TILES) {
        if (t.cb * t.pb == 4 && tail && !half) continue;
        const DirectCost& c = tail ? t.tail : t.plain;
        const double waves = 4.0 * (double)(((int64_t)m + 128 * t.pb - 1) / (128 * t.pb)) *
                             (double)((c_out + 32 * t.cb - 1) / (32 * t.cb)) / 1024.0;
        const double cost = c.fixed + c.chunk * groups + (c.wave + c.wave_chunk * groups) * waves;
        if (cost < least) { least = cost; best = t.tile; }
    }
    return best;
}

}  // namespace bcnn
