// Which calls the ballot kernel of the pack takes, and how its workgroups cover them (kernel: pack.hip).  Plain C++ on
// purpose: launcher and kernel use these functions, and a host-only test walks the workgroups with them.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define BCNN_PACK_INLINE __host__ __device__ __forceinline__
#else
#define BCNN_PACK_INLINE inline
#endif

namespace bcnn {

// A launch of 256-thread workgroups holds fewer than 2^32 threads.
constexpr int64_t MAX_BLOCKS_256 = (1 << 24) - 1;

// nv: 16-byte vectors of a row per lane (0: the ballot kernel does not take the call).  A workgroup's four waves: 1 << tw_shift
// neighbouring tiles of a row x the rest along the groups of 64 channels.
struct BallotPlan { int nv, tw_shift, groups, tiles; int64_t blocks_per_image; };

// Timed on rotating buffers beyond the last-level cache: rows of up to 128 bytes (bfloat16, 1024 channels, 256 maps of 7 x 7
// 12.2 -> 9.5 us; float weights, 1024 x 1024 x 3 x 3 18.4 -> 9.5), launches that do not fill the chip (float, 64 channels, one
// 14 x 14 map 2.6 -> 2.3).  Longer rows of large launches stream better with the lanes along the positions (float, 256
// channels, 64 maps of 56 x 56 39 us against 48, although from cache this kernel is ahead there, 32 against 37).
inline BallotPlan plan_ballot(int esz, uintptr_t src, int64_t outer, int64_t channels, int64_t src_channels, int64_t inner)
{
    BallotPlan p{};
    const int64_t row = inner * esz;
    // images a whole number of dwords apart, addressable by 31-bit offsets
    if (inner < 2 || (src_channels * row) % 4 != 0 || (src & 3) != 0 || src_channels * row >= (1ll << 30) ||
        channels >= (1 << 24) || inner * ((channels + 31) / 32) >= (1 << 28))
        return p;
    const int per = 16 / esz;                                // elements of a vector
    const int64_t fit = (inner + per - 1) / per;             // vectors of a row
    p.groups = (int)((channels + 63) / 64);
    auto tiles = [&](int nv) { return (inner + nv * per - 1) / (nv * per); };
    const bool whole_rows = fit <= (esz == 1 ? 4 : 8);
    // a wave takes whole rows (of at most 64 positions), or a few vectors of them where the launch is small
    p.nv = !whole_rows ? 4 : fit <= 1 ? 1 : fit <= 2 ? 2 : fit <= 4 ? 4 : 8;
    if (!whole_rows && outer * p.groups * tiles(4) >= 2048) { p.nv = 0; return p; }
    while (p.nv > 1 && outer * p.groups * tiles(p.nv) < 2048) p.nv /= 2;
    p.tiles = (int)tiles(p.nv);
    p.tw_shift = p.tiles < 2 ? 0 : p.tiles < 3 ? 1 : 2;     // neighbouring tiles share cache lines
    const int gw = 4 >> p.tw_shift;
    p.blocks_per_image = (int64_t)((p.tiles + (1 << p.tw_shift) - 1) >> p.tw_shift) * ((p.groups + gw - 1) / gw);
    if (p.blocks_per_image * outer > MAX_BLOCKS_256) p.nv = 0;
    return p;
}

// Wave `wave` of the image's workgroup `at` -> its tile of the rows and its group of 64 channels; false: it has neither.
BCNN_PACK_INLINE bool ballot_place(int at, int wave, int tw_shift, int groups, int tiles, int& tile, int& g)
{
    const int tw = 1 << tw_shift, gw = 4 >> tw_shift;
    const int gblocks = (groups + gw - 1) >> (2 - tw_shift);
    const int tb = at / gblocks;
    tile = tb * tw + (wave & (tw - 1));
    g = (at - tb * gblocks) * gw + (wave >> tw_shift);
    return tile < tiles && g < groups;
}

}  // namespace bcnn
