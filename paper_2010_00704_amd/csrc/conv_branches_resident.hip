// Branch mode of the matrix-core convolution with all of a workgroup's weights expanded in LDS (conv_mfma_resident.hip): F x F
// convolution as F*F shifted 1x1 branches, or P parallel ones, each with a real scale per output channel (BCNN paper, Section 4.2.1, last
// paragraph; Figure 2, bottom); bits or float sums.
//
// Plain codes on both sides (conv_mfma_direct_kernel.h); the pixels are the instruction's rows, so that a tap's scale is one register a
// channel block and its sums start from an inline zero.  A wave has two columns of 32 pixels x two blocks of 32 channels, in turn: the
// fold of one column's completed tap, tot = fma(scale, y_t, tot), is dealt out behind the matrix instructions of the other column, with the
// expansion of the next input fragment: eight vector instructions behind each, pinned there by scheduling barriers.
// Bound: the vector ALUs' issue, 8.1 instructions (8.8 with pad words) per matrix instruction of 35 cycles: 43 to 48 cycles each;
// the start, 4500 cycles of 35 000 (3x3, 256 -> 256, 64 maps of 28 x 28); and a wave's odd column, whose pass works on a second one of nothing: that call
// has 24 or 25 columns a workgroup, three a wave in passes of two and one, so that 77 % of its matrix instructions are wanted.  With the fold in one piece in
// front of a tap's products it was 58 cycles.
// Measured (us, graph replays on one card, shared weights and this): that call as bits, pad words 22.6 and 17.4, -1 outside 21.2 and 16.8, float sums, pad words
// 23.6 and 20.5 (inputs from memory 22.9 and 22.0); 40 maps of 27 x 27, 320 -> 200, bits, pad words 18.5 and 12.7; 1x1, three branches with tensors of
// their own, 256 -> 256, 64 maps of 28 x 28, bits 11.0 and 8.8.
// Not for taps that contribute nothing outside (their lane masks need registers that the interleaved fold has not), taps of two groups (the fold
// at some of them only: forms of a column under branches spill) and module tails.
#include "conv_mfma_resident.h"
#include "resident_kernel.h"

namespace bcnn {
namespace {

struct ResidentBranch {
    const float* scale;          // [taps][c_out]
    const float* bias;           // [c_out] or nullptr
    const uint32_t* pad_words;   // [taps][cw] (PAD_OPERAND)
};
enum { PAD_NONE = 0, PAD_OPERAND = 1 };                      // outside the image: -1, the branch's pad words
constexpr int MAX_TAPS = RESIDENT_TAPS;

// 32 x 32 bits, a row of them in every lane of a half: bit c of lane r and bit r of lane c change places, in five steps of halves.
__device__ __forceinline__ uint32_t transpose_bits(uint32_t v, int j)
{
    auto step = [&](uint32_t from, int size, uint32_t low) __attribute__((always_inline)) {
        const bool upper = (j & size) != 0;
        const uint32_t turned = __builtin_amdgcn_alignbit(from, from, upper ? size : 32 - size);   // right, or left, by size
        const uint32_t keep = upper ? ~low : low;
        v = (v & keep) | (turned & ~keep);
    };
    step((uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F), 16, 0x0000FFFFu);                                     // lane ^ 16
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true), 8, 0x00FF00FFu);                    // row_ror 8: lane ^ 8
    step((uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x101F), 4, 0x0F0F0F0Fu);                                      // lane ^ 4
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true), 2, 0x33333333u);                     // quad_perm: lane ^ 2
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true), 1, 0x55555555u);                     // quad_perm: lane ^ 1
    return v;
}

template <int WIDE, bool BITS, int PAD, bool ODD>
__global__ __launch_bounds__(64 * RESIDENT_WAVES, 2) void conv_branches_resident_kernel(
    ResidentArgs a, const uint32_t* __restrict__ x, const uint32_t* __restrict__ w, void* __restrict__ out, ResidentBranch br)
{
    constexpr int CB = RESIDENT_CHANNELS / 32;
    constexpr int UNIT = WIDE > 4 ? 8 : 4;                   // words of a group's pad words, 16-byte aligned
    __shared__ struct {
        // [channel block][K-step][unit of 16 bytes = a row's words' codes]: lane half h finds row i at unit 32 h + (i ^ 8 h)
        __align__(16) char weights[CB * RESIDENT_STEPS * 1024];
        v2i pixel[RESIDENT_BRANCH_COLUMNS * 32];
        float scale[MAX_TAPS + 1][RESIDENT_CHANNELS];        // the last row: the bias
        __align__(16) int pad[PAD == PAD_OPERAND ? MAX_TAPS + 1 : 1][2][UNIT];   // [tap][lane half]
    } lds;
    const ConvShape& s = a.s;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int hsel = lane >> 5, j = lane & 31;

    const ResidentPlace at = resident_place(a);
    const int o0 = at.o0;
    const ResidentRun columns = resident_run(a.quotient, a.rest, at.range);
    const int n_groups = a.n_groups;

    const auto xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(x), 0, a.x_bytes, 0x00020000);
    const auto wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w), 0, a.w_bytes, 0x00020000);
    uint32_t m8, c2;                                         // held in registers: v_and_or_b32 takes no literals
    asm volatile("v_mov_b32 %0, 0x88888888" : "=v"(m8));
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));
    auto expand = [&](uint32_t word) __attribute__((always_inline)) -> v4i {
        return v4i{(int)(((word << 3) & m8) | c2), (int)(((word << 2) & m8) | c2), (int)(((word << 1) & m8) | c2), (int)((word & m8) | c2)};
    };

    // ---- weights -> LDS, as in the plain kernel, with plain codes; a row of a block is its channel
    const int g0 = wave >> 1, wb = wave & 1;
    const int urow = lane >> 1, uhalf = lane & 1;
    const int uwords = uhalf ? s.cw - a.half : a.half;
    const int uchannel = o0 + 32 * wb + urow;
    const int urow_at = ((uchannel < s.c_out ? uchannel : s.c_out - 1) * a.n_words + uhalf * a.half) * 4;
    char* put_at = lds.weights + (wb * n_groups + g0) * WIDE * 1024 + (uhalf * 32 + (urow ^ (uhalf * 8))) * 16;
    auto fetch_w = [&](int gi, int (&v)[WIDE]) __attribute__((always_inline)) {
        const int tap = a.div_tap(gi);
        load_words(wres, urow_at + (tap * s.cw + WIDE * (gi - tap * a.per_tap)) * 4, v);
    };
    auto put = [&](int gi, const int (&v)[WIDE]) __attribute__((always_inline)) {
        if (a.whole) {
#pragma unroll
            for (int i = 0; i < WIDE; ++i) *reinterpret_cast<v4i*>(put_at + i * 1024) = expand((uint32_t)v[i]);
            return;
        }
        const int k0 = WIDE * (gi - a.div_tap(gi) * a.per_tap);
#pragma unroll
        for (int i = 0; i < WIDE; ++i) {
            const uint32_t bits = k0 + i < uwords ? (uhalf * a.half + k0 + i == s.cw - 1 ? a.last_bits : ~0u) : 0u;
            const uint32_t word = (uint32_t)v[i];
            v4i code;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const uint32_t sign = (bits << (3 - jj)) & m8;
                code[jj] = (int)(((word << (3 - jj)) & sign) | (sign >> 2));
            }
            *reinterpret_cast<v4i*>(put_at + i * 1024) = code;
        }
    };
    {
        int v0[WIDE], v1[WIDE];
        fetch_w(g0, v0);
        fetch_w(g0 + 4, v1);
        // scales, bias and pad words are on their way while the places are computed
        constexpr int SHARE = ((MAX_TAPS + 1) * RESIDENT_CHANNELS + 64 * RESIDENT_WAVES - 1) / (64 * RESIDENT_WAVES);
        const auto scale_res = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(br.scale), 0, a.taps * s.c_out * 4, 0x00020000);
        const auto bias_res = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(br.bias), 0, br.bias ? s.c_out * 4 : 0, 0x00020000);
        const int cl = t % RESIDENT_CHANNELS, row0 = t / RESIDENT_CHANNELS;      // (channels past c_out read what nobody looks at)
        uint32_t scales[SHARE];
#pragma unroll
        for (int i = 0; i < SHARE; ++i)
            scales[i] = __builtin_amdgcn_raw_buffer_load_b32(scale_res, ((row0 + i * RESIDENT_WAVES) * s.c_out + o0 + cl) * 4, 0, 0);
        const uint32_t bias = __builtin_amdgcn_raw_buffer_load_b32(bias_res, (o0 + cl) * 4, 0, 0);
        uint32_t pad = 0;
        if constexpr (PAD == PAD_OPERAND) {
            static_assert(2 * UNIT * MAX_TAPS <= 64 * RESIDENT_WAVES, "a pad word a thread");
            const auto pres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(br.pad_words), 0, a.n_words * 4, 0x00020000);
            const int k = t % UNIT, word = ((t / UNIT) & 1) * a.half + k;
            pad = __builtin_amdgcn_raw_buffer_load_b32(pres, k < WIDE && word < s.cw ? (t / (2 * UNIT) * s.cw + word) * 4 : -4, 0, 0);
        }
        resident_places(a, lds.pixel, columns.first, columns.count < RESIDENT_BRANCH_COLUMNS ? columns.count : RESIDENT_BRANCH_COLUMNS);
#pragma unroll
        for (int i = 0; i < SHARE; ++i)
            if (row0 + i * RESIDENT_WAVES < MAX_TAPS) lds.scale[row0 + i * RESIDENT_WAVES][cl] = __uint_as_float(scales[i]);
        if (row0 == 0) lds.scale[MAX_TAPS][cl] = __uint_as_float(bias);
        if constexpr (PAD == PAD_OPERAND) {
            if (t < 2 * UNIT * MAX_TAPS) (&lds.pad[0][0][0])[t] = (int)pad;
        }
#pragma unroll 1
        for (int gi = g0; gi < n_groups; gi += 4) {
            int v[WIDE];
#pragma unroll
            for (int i = 0; i < WIDE; ++i) { v[i] = v0[i]; v0[i] = v1[i]; }
            fetch_w(gi + 8, v1);
            put(gi, v);
            put_at += 4 * WIDE * 1024;
        }
        meet();
    }

    const char* const my_weights = lds.weights + (hsel * 32 + (j ^ (hsel * 8))) * 16;
    const int block_bytes = n_groups * WIDE * 1024;

    // P columns from `col` on; two columns are worked on, whatever P
    auto pass = [&](auto pc, int col, int place) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value, Q = 2;
        int base[Q], taps[Q];
#pragma unroll
        for (int pb = 0; pb < Q; ++pb) {
            const v2i q = lds.pixel[32 * (place + (pb < P ? pb : 0)) + row_to_channel(j)];
            base[pb] = q[0] + hsel * a.half * 4;
            taps[pb] = pb < P ? q[1] : 0;
        }
        struct Inputs { int x[Q][WIDE]; } ring[2];
        int f_tap = 0;
        auto fetch_x = [&](Inputs& c) __attribute__((always_inline)) {
            const int bit = f_tap < a.taps ? f_tap : 31;
            const int xo = (f_tap * a.tap_words + ((f_tap * 11) >> 5) * a.row_jump) * 4;
#pragma unroll
            for (int pb = 0; pb < Q; ++pb) {
                const int in = __builtin_amdgcn_sbfe(taps[pb], (uint32_t)bit, 1u);
                load_words(xres, ((base[pb] + xo) & in) | (~in & PAST_ALL), c.x[pb]);
            }
            ++f_tap;
        };
        if constexpr (ODD) fetch_x(ring[1]);                 // of an odd number of taps the first stands alone, of an even one the first two
        fetch_x(ring[0]);
        if constexpr (!ODD) fetch_x(ring[1]);

        v16f acc[Q][CB], tot[Q][CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const float bias = lds.scale[MAX_TAPS][32 * cb + j] + (BITS ? 0.0f : -0.0f);   // (bits: no -0)
#pragma unroll
            for (int pb = 0; pb < Q; ++pb)
#pragma unroll
                for (int r = 0; r < 16; ++r) tot[pb][cb][r] = bias;
        }
        v4i fw[WIDE][CB];
        const char* from = my_weights;
        auto read_w = [&](int k) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) fw[k][cb] = *reinterpret_cast<const v4i*>(from + cb * block_bytes + k * 1024);
        };
#pragma unroll
        for (int k = 0; k < WIDE; ++k) read_w(k);
        int tap = 0;
        float sc[CB], sc_before[CB] = {0.0f, 0.0f};          // of its tap and of the one before
        auto word = [&](const Inputs& c, int pb, int k) __attribute__((always_inline)) -> uint32_t { return (uint32_t)c.x[pb][k]; };
        // the branch's pad words take the place of the zeros that a tap outside has read
        auto set_pad = [&](Inputs& c, int t_tap) __attribute__((always_inline)) {
            if constexpr (PAD == PAD_OPERAND) {
                int pad[UNIT];
                const int* const p = lds.pad[t_tap][hsel];
                *reinterpret_cast<v4i*>(pad) = *reinterpret_cast<const v4i*>(p);
                if constexpr (WIDE > 4) pad[4] = p[4];
#pragma unroll
                for (int pb = 0; pb < Q; ++pb) {
                    const uint32_t in = (uint32_t)__builtin_amdgcn_sbfe(taps[pb], (uint32_t)t_tap, 1u);
#pragma unroll
                    for (int k = 0; k < WIDE; ++k) c.x[pb][k] = (int)(((uint32_t)c.x[pb][k] & in) | ((uint32_t)pad[k] & ~in));
                }
            }
        };
        // tot = fma(scale, y_t, tot) in the order t = 0, 1, ...
        auto fold_one = [&](int e, int pb, const float (&sv)[CB]) __attribute__((always_inline)) {
            const int cb = e >> 4, r = e & 15;
            tot[pb][cb][r] = __builtin_fmaf(sv[cb], acc[pb][cb][r], tot[pb][cb][r]);
        };
        v4i next;                                            // the next matrix instructions' input fragment
        // One column's K-steps of a group.  Behind every matrix instruction: a share of the fold of the other column's completed tap, half
        // of the next input fragment and, in the last column, the next group's weights of the K-step just done.
        auto column = [&](auto pbc, auto folds, const float (&sv)[CB], uint32_t after, const Inputs& c) __attribute__((always_inline)) {
            constexpr int pb = decltype(pbc)::value, SLOTS = WIDE * CB;
#pragma unroll
            for (int k = 0; k < WIDE; ++k) {
                const v8i fx = {next[0], next[1], next[2], next[3], 0, 0, 0, 0};
                uint32_t wd = k + 1 < WIDE ? word(c, pb, k + 1) : after;
                v4i e;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const v8i w8 = {fw[k][cb][0], fw[k][cb][1], fw[k][cb][2], fw[k][cb][3], 0, 0, 0, 0};
                    const v16f zero = {};
                    acc[pb][cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fx, w8, k == 0 ? zero : acc[pb][cb], 4, 4, 0, 0, 0, 0);
                    if constexpr (decltype(folds)::value) {
                        const int i = k * CB + cb;
#pragma unroll
                        for (int q = i * 32 / SLOTS; q < (i + 1) * 32 / SLOTS; ++q) fold_one(q, 1 - pb, sv);
                    }
                    if (cb == 0) {
                        e[0] = (int)(((wd << 3) & m8) | c2);
                        e[1] = (int)(((wd << 2) & m8) | c2);
                    } else {
                        e[2] = (int)(((wd << 1) & m8) | c2);
                        e[3] = (int)((wd & m8) | c2);
                        if (pb == Q - 1) read_w(k);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                next = e;
            }
        };
        using C0 = std::integral_constant<int, 0>;
        using C1 = std::integral_constant<int, 1>;
        // a tap: column 0 beside the fold of column 1's tap before, column 1 beside the fold of column 0's
        auto one_tap = [&](auto folds, Inputs& c, Inputs& then) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) sc[cb] = lds.scale[tap][32 * cb + j];
            column(C0{}, folds, sc_before, word(c, 1, 0), c);
            from += WIDE * 1024;
            set_pad(then, tap + 1);
            column(C1{}, std::true_type{}, sc, word(then, 0, 0), c);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) sc_before[cb] = sc[cb];
            ++tap;
        };
        constexpr int FIRST = ODD ? 1 : 0;
        set_pad(ring[FIRST], 0);
        next = expand(word(ring[FIRST], 0, 0));
        one_tap(std::false_type{}, ring[FIRST], ring[1 - FIRST]);
        fetch_x(ring[FIRST]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!ODD) {
            one_tap(std::true_type{}, ring[1], ring[0]);
            fetch_x(ring[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll 1
        for (int left = a.taps - (ODD ? 1 : 2); left > 0; left -= 2) {
            one_tap(std::true_type{}, ring[0], ring[1]);
            fetch_x(ring[0]);
            __builtin_amdgcn_sched_barrier(0);
            one_tap(std::true_type{}, ring[1], ring[0]);
            fetch_x(ring[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < 32; ++q) fold_one(q, 1, sc_before);

        // ---- a lane holds 16 pixels of one channel; rows past the end are past the buffer's size and store nothing
        const int rows = s.m - 32 * col;
        const int row_bytes = (BITS ? s.cwo : s.c_out) * 4;
        const uint64_t row = reinterpret_cast<uint64_t>(out) + (uint64_t)col * (uint64_t)(32 * row_bytes);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)row);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(row >> 32));
        const auto res = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>((hi << 32) | lo), 0,
                                                           __builtin_amdgcn_readfirstlane((rows < 32 * P ? rows : 32 * P) * row_bytes), 0x00020000);
        constexpr uint32_t NOWHERE = 0x7FFFFF00u;
        if constexpr (BITS) {
            // sums are never -0 (they start from +0 or a bias that is no -0), and the maximum turns NaN negative
            const int left = s.c_out - (o0 + 32 * hsel);
            const uint32_t valid = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
#pragma unroll
            for (int pb = 0; pb < P; ++pb) {
                uint32_t negative[CB] = {0u, 0u};            // of the lane's 16 pixels
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int r = 15; r >= 0; --r)
                        negative[cb] = __builtin_amdgcn_alignbit(negative[cb], __float_as_uint(__builtin_fmaxf(tot[pb][cb][r], -3.402823466e38f)), 31);
                // lane half h: channel block h, 32 pixels of one channel a lane
                const auto both = __builtin_amdgcn_permlane32_swap(negative[0], negative[1], false, false);
                const uint32_t word = transpose_bits(both[0] | (both[1] << 16), j);
                const uint32_t to = (uint32_t)((32 * pb + j) * s.cwo + (o0 >> 5) + hsel) * 4u;
                __builtin_amdgcn_raw_buffer_store_b32((int)(~word & valid), res, (int)(left > 0 ? to : NOWHERE), 0, 0);
            }
        } else {
            // (The row in the vector offset: the scalar one is left out of the bounds check, which drops the rows past the end.  Computed
            // here: they are the same for every pass, and kept in registers they spill.)
#pragma unroll
            for (int pb = 0; pb < P; ++pb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const int ch = o0 + 32 * cb + j;
                    uint32_t to = ch < s.c_out ? (uint32_t)((32 * pb + 16 * hsel) * row_bytes + ch * 4) : NOWHERE;
                    asm volatile("" : "+v"(to));
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(tot[pb][cb][r]), res, (int)(to + (uint32_t)(r * row_bytes)), 0, 0);
                }
        }
    };
    resident_columns<2, RESIDENT_BRANCH_COLUMNS>(a, columns, lds.pixel, wave, pass);
}

template <int WIDE>
hipError_t launch_wide(const ResidentArgs& a, const BranchArgs& b, hipStream_t stream)
{
    const dim3 blocks((unsigned)(a.n_ranges * a.n_ctiles)), threads(64 * RESIDENT_WAVES);
    const ResidentBranch br{b.scale, b.bias, b.pad_words};
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, a, b.x, b.w, b.out, br); };
    // (without padding every tap is inside)
    auto of_pad = [&](auto bits, auto odd) {
        if (a.s.pad && b.pad_words) go(conv_branches_resident_kernel<WIDE, decltype(bits)::value, PAD_OPERAND, decltype(odd)::value>);
        else go(conv_branches_resident_kernel<WIDE, decltype(bits)::value, PAD_NONE, decltype(odd)::value>);
    };
    auto of_taps = [&](auto bits) {
        if (a.taps % 2) of_pad(bits, std::true_type{});
        else if constexpr (WIDE < 5) go(conv_branches_resident_kernel<WIDE, decltype(bits)::value, PAD_NONE, false>);   // (3x3 filters have nine)
    };
    if (b.fused) of_taps(std::true_type{});
    else of_taps(std::false_type{});
    return hipGetLastError();
}

}  // namespace

hipError_t launch_conv_branches_resident(const ConvShape& s, const BranchArgs& b, hipStream_t stream)
{
    const SharedWalk walk = SharedWalk::make(s.cw, b.branches);
    if (b.branches % 2 == 0 && walk.wide > 4) return hipErrorInvalidValue;
    if (walk.wide < 3 || walk.per_tap != 1 || walk.steps(b.branches) > RESIDENT_STEPS || b.branches > MAX_TAPS || b.tail || (s.pad && b.zero_pad))
        return hipErrorInvalidValue;
    ResidentArgs a = resident_args(s, b.branches, walk);
    const int64_t one = (int64_t)s.n * s.h * s.w * s.cw * 4;
    a.x_bytes = (int32_t)(b.x_branch_stride ? (int64_t)(b.branches - 1) * b.x_branch_stride * 4 + one : one);
    a.tap_words += (int32_t)b.x_branch_stride;
    switch (walk.wide) {
        case 3: return launch_wide<3>(a, b, stream);
        case 5: return launch_wide<5>(a, b, stream);
        default: return launch_wide<4>(a, b, stream);
    }
}

}  // namespace bcnn
