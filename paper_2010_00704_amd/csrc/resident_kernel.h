// What the kernels whose weights stay in LDS have in common: the plain one (conv_mfma_resident.hip) and branch mode
// (conv_branches_resident.hip).
#pragma once
#include "bcnn_common.h"
#include "div_by.h"
#include "resident_plan.h"

#include <type_traits>

namespace bcnn {

struct ResidentArgs {
    ConvShape s;
    int32_t taps;                // filter taps, or branches
    int32_t n_ctiles, n_ranges;
    int32_t quotient, rest;      // columns of a range: quotient, one more in the first `rest`
    int32_t n_words;             // of a weight row
    int32_t half, per_tap;       // words of a tap's longer lane half; groups a tap
    int32_t n_groups;            // per_tap a tap; a group is one load: WIDE words of each half
    int32_t whole;               // every word of every group exists and has 32 channels
    uint32_t last_bits;          // channels of a pixel's last word
    int32_t low_bits;            // positions 4 i + 0 .. 2 of a channel's words that exist (plain kernel)
    int32_t x_bytes, w_bytes;
    int32_t tap_words, row_jump; // words from a tap to the next one, and more from a filter row's last to the next one's first
    DivBy div_ct, div_hw, div_wo, div_tap;
};

// (launches `taps` of cw words each; tap_words: 3x3, the next pixel; branches with tensors of their own, the stride between those)
inline ResidentArgs resident_args(const ConvShape& s, int taps, const SharedWalk& walk)
{
    const ResidentSplit split = resident_split(s.m, s.c_out);
    const int c_in = s.k / (s.ks * s.ks);
    ResidentArgs a;
    a.s = s;
    a.taps = taps;
    a.n_ctiles = split.n_ctiles;
    a.n_ranges = split.n_ranges;
    a.quotient = split.columns / split.n_ranges;
    a.rest = split.columns % split.n_ranges;
    a.n_words = taps * s.cw;
    a.half = walk.half;
    a.per_tap = walk.per_tap;
    a.n_groups = walk.groups;
    a.last_bits = c_in % 32 ? (1u << (c_in % 32)) - 1u : ~0u;
    a.whole = c_in % 32 == 0 && s.cw == 2 * walk.half && walk.half == walk.per_tap * walk.wide;
    // 24 of a whole word's 32 channels, of the last word's those of its bits
    a.low_bits = taps * (24 * (c_in / 32) + (c_in % 32 ? __builtin_popcount(a.last_bits & 0x77777777u) : 0));
    a.x_bytes = (int32_t)((int64_t)s.n * s.h * s.w * s.cw * 4);
    a.w_bytes = (int32_t)((int64_t)s.c_out * a.n_words * 4);
    a.tap_words = s.ks == 3 ? s.cw : 0;
    a.row_jump = s.ks == 3 ? (s.w - 3) * s.cw : 0;
    a.div_ct = DivBy::make(a.n_ctiles);
    a.div_hw = DivBy::make(s.ho * s.wo);
    a.div_wo = DivBy::make(s.wo);
    a.div_tap = DivBy::make(a.per_tap);
    return a;
}

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v3i __attribute__((ext_vector_type(3)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// MFMA row i of a 32-row block carries this row (channel, or pixel) of the block, so that a lane ends up holding 16
// consecutive ones (lane half h, register r <-> row 16h + r).
__device__ __forceinline__ int row_to_channel(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// only LDS is shared: loads in flight stay in flight
__device__ __forceinline__ void meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// the workgroup's place: each XCD takes a contiguous range of them, channel tile fastest
struct ResidentPlace { int range, o0; };
__device__ __forceinline__ ResidentPlace resident_place(const ResidentArgs& a)
{
    int tile = blockIdx.x;
    const int per_xcd = (a.n_ranges * a.n_ctiles) >> 3;
    if (tile < per_xcd * 8) tile = (tile & 7) * per_xcd + (tile >> 3);
    const int range = a.div_ct(tile);
    return ResidentPlace{range, (tile - range * a.n_ctiles) * RESIDENT_CHANNELS};
}

// WIDE words from a byte offset on (4-byte alignment; what lies past the tensor's end reads as zero, so no part of the offset is in the
// scalar one, which the bounds check leaves out)
template <int WIDE>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t res, int off, int (&v)[WIDE])
{
    if constexpr (WIDE >= 4) {
        const v4i q = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(res, off, 0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = q[i];
        if constexpr (WIDE == 5) v[4] = (int)__builtin_amdgcn_raw_buffer_load_b32(res, (int)((uint32_t)off + 16u), 0, 0);
    } else {
        const v3i q = __builtin_bit_cast(v3i, __builtin_amdgcn_raw_buffer_load_b96(res, off, 0, 0));
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = q[i];
    }
}

// Where the pixels of `count` columns lie and which taps of theirs are inside the image, once for all waves: byte offset of the window's
// top-left tap, one validity bit per tap.
__device__ __forceinline__ void resident_places(const ResidentArgs& a, v2i* pixel, int first, int count)
{
    const ConvShape& s = a.s;
    for (int i = threadIdx.x; i < 32 * count; i += 64 * RESIDENT_WAVES) {
        int m = 32 * first + i;
        m = m < s.m ? m : s.m - 1;
        const int n = a.div_hw(m);
        const int r = m - n * s.ho * s.wo;
        const int oh = a.div_wo(r);
        const int ph = oh * s.stride - s.pad;
        const int pw = (r - oh * s.wo) * s.stride - s.pad;
        uint32_t cols = 0, taps = 0;
#pragma unroll
        for (int v = 0; v < 3; ++v) cols |= (uint32_t)((uint32_t)(pw + v) < (uint32_t)s.w) << v;
#pragma unroll
        for (int u = 0; u < 3; ++u) taps |= ((uint32_t)(ph + u) < (uint32_t)s.h) ? cols << (3 * u) : 0u;
        pixel[i] = v2i{((n * s.h + ph) * s.w + pw) * s.cw * 4, s.ks == 1 ? 0xFFFF : (int)taps};   // 1x1: no padding, every branch is inside
    }
}

// Every column of the workgroup in passes of one to MOST columns: pass(std::integral_constant<int, columns>, column, its place in `pixel`).
// TABLE: columns that `pixel` holds; the first places have been put there.
template <int MOST, int TABLE, class Pass>
__device__ __forceinline__ void resident_columns(const ResidentArgs& a, const ResidentRun& columns, v2i* pixel, int wave, Pass&& pass)
{
    for (int done = 0;;) {
        const int here = columns.count - done < TABLE ? columns.count - done : TABLE;
        const ResidentRun mine = resident_run(here / RESIDENT_WAVES, here % RESIDENT_WAVES, wave);
#pragma unroll 1
        for (int place = mine.first, left = mine.count; left > 0;) {
            const int take = resident_take(left, MOST), col = columns.first + done + place;
            if (MOST >= 4 && take == 4) pass(std::integral_constant<int, MOST >= 4 ? 4 : 1>{}, col, place);
            else if (MOST >= 3 && take == 3) pass(std::integral_constant<int, MOST >= 3 ? 3 : 1>{}, col, place);
            else if (take == 2) pass(std::integral_constant<int, 2>{}, col, place);
            else pass(std::integral_constant<int, 1>{}, col, place);
            place += take;
            left -= take;
        }
        done += here;
        if (done >= columns.count) break;
        meet();
        resident_places(a, pixel, columns.first + done, columns.count - done < TABLE ? columns.count - done : TABLE);
        meet();
    }
}

}  // namespace
}  // namespace bcnn
