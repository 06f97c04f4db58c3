// The kernels whose weights stay in LDS (conv_mfma_resident.hip, in branch mode conv_branches_resident.hip): how a call is split over its workgroups and waves, and which calls
// take it.  Plain C++ on purpose: the launcher and the kernel use these functions, and a host-only test walks them.
#pragma once
#include <stdint.h>

#include "shared_plan.h"

#if defined(__HIPCC__)
#define BCNN_RESIDENT_INLINE __host__ __device__ __forceinline__
#else
#define BCNN_RESIDENT_INLINE inline
#endif

namespace bcnn {

constexpr int RESIDENT_WAVES = 8;                            // of a workgroup; one workgroup a compute unit
constexpr int RESIDENT_CHANNELS = 64;                        // of a workgroup, every wave takes all of them
constexpr int RESIDENT_STEPS = 72;                           // K-steps whose expanded weights fit LDS, 2 KB each
// Columns of 32 pixels whose places lie in LDS at a time: what the weights leave, in branch mode beside its scales and pad words.
constexpr int RESIDENT_COLUMNS = 52, RESIDENT_BRANCH_COLUMNS = 40;
constexpr int RESIDENT_PASS = 4;                             // columns of a wave at a time

// Part `part` of a number of columns in parts whose lengths differ by one at most, the longer ones (`rest` of them) first.
struct ResidentRun { int first, count; };
BCNN_RESIDENT_INLINE ResidentRun resident_run(int quotient, int rest, int part)
{
    return ResidentRun{part * quotient + (part < rest ? part : rest), quotient + (part < rest ? 1 : 0)};
}
// Columns of a wave's next pass when `left` are to do: as many as it takes, but the last two passes share theirs.
BCNN_RESIDENT_INLINE int resident_take(int left, int most) { return left <= most ? left : left >= 2 * most ? most : (left + 1) / 2; }

// Tiles of 64 channels, each with n_ranges workgroups that share out the columns.
struct ResidentSplit { int n_ctiles, n_ranges, columns; };
inline ResidentSplit resident_split(int m, int c_out)
{
    ResidentSplit r;
    r.columns = (int)(((int64_t)m + 31) / 32);
    r.n_ctiles = (c_out + RESIDENT_CHANNELS - 1) / RESIDENT_CHANNELS;
    r.n_ranges = r.n_ctiles < 256 ? 256 / r.n_ctiles : 1;
    if (r.n_ranges > r.columns) r.n_ranges = r.columns;
    return r;
}
// Whether the workgroups, one a compute unit, keep `percent` of the 256 busy in every round: 130 channel tiles have one range each and
// leave half of them idle, 290 take two rounds.  Below 2305 channels 90 % are always busy.
inline bool resident_fills(const ResidentSplit& s, int percent)
{
    const int64_t workgroups = (int64_t)s.n_ctiles * s.n_ranges, rounds = (workgroups + 255) / 256;
    return 100 * workgroups >= percent * 256 * rounds;
}

// Packed bits of 3x3 filters, 5 to 16 words a pixel, whose launch has two tiles of 64 channels x 32 pixels for every SIMD
// (1024) and more: below, the start with its expansion of all weights is what the launch takes.  Not where half of the only tile, or of every
// second one, is channels that do not exist (32 channels: 10 of 18 calls more than 5 % behind, 22 % at worst).  Over 420 calls (130 to 512 channels in, 64 to
// 2304 out, strides 1 and 2), timed on this kernel and on the one that ran them before, inputs from the last-level cache and from memory: 0.90 and 0.91 of
// the time from two tiles on, 13 and 26 of them more than 3 % behind, 15 % at worst (us, from memory: 62 maps of 12 x 12, 504 -> 832 15.4 and 17.3); between one and a half and two
// 0.98 and 0.99, 6 and 12 of 39 behind, 17 % at worst.  Of up to four words a pixel several taps share a group of K-steps: 0.95 to 1.03
// times, no better than level on average; 1x1 filters of up to 16 words 0.9 to 1.3.
// Workgroups that keep 85 % of the compute units busy: over 150 calls of 1025 to 20 000 channels out, 0.93 of the time at 85 to 90 %, 1.01 at 80 to 85 %,
// 1.35 at 50 to 60 % (54 x 54, stride 2, 256 -> 17 637 14.3 and 23.0; 344 maps of 9 x 9, 194 -> 9404 224 and 310).
inline bool resident_takes(int m, int c_out, int cw, int ks)
{
    if (ks != 3 || cw < 5) return false;
    const int across = (c_out + 31) / 32;
    if (across % 2 != 0 && across < 5) return false;
    const SharedWalk walk = SharedWalk::make(cw, 9);
    const ResidentSplit split = resident_split(m, c_out);
    return walk.steps(9) <= RESIDENT_STEPS && (int64_t)split.columns * split.n_ctiles >= 2 * 1024 && resident_fills(split, 85);
}

// Branch calls (P shifted or parallel 1x1 branches, a real scale each) without a module's tail and without taps that contribute
// nothing, 5 to 10 words a pixel (a tap is one group of K-steps).  Packed bits from 800 tiles of 64 channels x 32 pixels on, or of four and more
// taps from 400 on, and nowhere where waves take whole taps (an odd number of channel blocks: bits, nine taps, 256 -> 96, 3 maps of 49 x 49 5.2
// there and 6.2, sums, six, 245 -> 160 4.6 and 5.5); float sums of six and more taps on one tensor, whose stores weigh less (of one to three taps
// 0.94 to 1.16 times, of four and five 0.86 to 1.17).  Not float sums of branches that have tensors of their own: two taps ahead is not early enough for
// loads from memory that the stores delay.  Their inputs in the last-level cache 1.03 times on average over 104 calls, from memory 1.14 over 96, 1.49 at
// worst (492 maps of 24 x 24, four taps, 160 -> 192 45 and 66; 3x3, 37 maps of 40 x 40, 192 -> 512 42 and 59); bits of such calls 0.83, from memory too.
// Over 393 calls that the rule takes (time on shared weights and here, inputs from the last-level cache): bits 0.82 on average, of nine taps 0.88 at 400 to
// 800 tiles and 0.79 from 2048 on, of two taps 0.77, of one 0.90, two of 236 more than 3 % behind, 10 % at worst (three taps, 161 -> 76, 24 maps of 30 x 30 4.4
// and 4.8); sums 0.89, two of 157 behind, 4 % at worst.  Over 109 with inputs from memory: bits 0.81, none behind; sums 0.95, eleven of 81
// behind, 14 % at worst (seven taps, 192 -> 128, 10 maps of 47 x 47 6.8 and 7.8).
// Workgroups that keep 70 % of the compute units busy: over 90 calls of 1025 to 20 000 channels out, 0.93 of the time at 70 to 80 %, 1.05 at 60 to
// 70 %, 1.2 below (bits, 41 maps of 21 x 21, three taps, 192 -> 9172 89 and 120; sums, 4 maps of 28 x 28, nine taps, 218 -> 17 775 105 and 129).
// (an even number of taps of five words a load has no registers left)
constexpr int RESIDENT_TAPS = 16;
inline bool resident_takes_branches(int m, int c_out, int cw, int taps, bool bits, bool own, bool nothing_outside)
{
    if (cw < 5 || taps > RESIDENT_TAPS || nothing_outside || branches_apart(m, c_out, taps)) return false;
    const SharedWalk walk = SharedWalk::make(cw, taps);
    if (walk.per_tap != 1 || walk.steps(taps) > RESIDENT_STEPS || (taps % 2 == 0 && walk.wide > 4)) return false;
    const ResidentSplit split = resident_split(m, c_out);
    const int64_t tiles = (int64_t)split.columns * split.n_ctiles;
    if (!resident_fills(split, 70)) return false;
    if (!bits) return taps >= 6 && !own && tiles >= 400;
    return tiles >= (taps >= 4 ? 400 : 800);
}

}  // namespace bcnn
