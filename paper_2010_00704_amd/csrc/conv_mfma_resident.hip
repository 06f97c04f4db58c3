// Binary convolution on the matrix cores with all of a workgroup's weights expanded in LDS: packed bits of the larger 3x3 launches.
//
// Arithmetic and codes as in conv_mfma_fp4_kernel.h (+-1 as 4-bit floats, exact fp32 sums; inputs are the bit alone in three
// registers of a fragment, four instructions; the weights carry the signs and, here, the opposite one, so that a sum's sign is
// the output bit).  BCNN paper, Section 1: the operator is a matrix product; Section 4.2.1: operands are +-1, padding is -1.
//
// What this kernel is for.  The staged kernel expands both operands in every wave, for every tile, between the matrix instructions of
// one wave per SIMD, and nothing covers a tile's first loads and its epilogue; with K walks of nine chunks that was half of the time, and 784 of
// its workgroups ran as 512 and 272.  Here 256 workgroups, one a compute unit, each expand 64 channels x all of K once (2 KB a
// K-step, up to 144 KB), and then their eight waves, two per SIMD, walk all of K for 64 channels x up to four columns of 32 pixels at a time
// without a barrier: a wave's epilogue and first loads hide behind its neighbour's matrix instructions.  A weight fragment is one
// conflict-free 16-byte LDS read; a column's words come straight from memory, two groups of K-steps ahead.  Columns are dealt out to within one:
// passes of four or three per wave, no tile left over.
// Bound: the K loop by the matrix cores: 32 to 35 cycles per instruction and SIMD (its own rate), and by the board's power limit when it runs
// for long (16.7 ns per instruction; constant operands 15.7); a launch of one or two passes by its start, 8000 cycles until
// the first product of 27 000 (3x3, 256 -> 256, 64 maps of 28 x 28): arguments 900, places of the pixels 1700, weights' loads and expansion
// 3700, first inputs 1500.
// Measured (us, graph replays on one card, the staged kernel before and this): that call 14.1 and 13.5, 64 maps of 56 x 56 under stride 2, 256 -> 512
// 27.3 and 23.5, 512 maps of 28 x 28, 256 -> 256 82.7 and 76.3; inputs from memory 13.9 and 13.4, 28.8 and 24.7, 83.7 and 79.5.  Tried, where this one took
// 12.6, 21.9 and 72.5 in kernel times: 1 x 7 blocks a wave (half as many LDS reads, twice the expansion: 13.3, 24.3 and 79.7), 128
// channels a workgroup (twice the weights to expand at the start: 13.9 on the first), the first inputs asked for in front of the expansion
// (its loads then wait for them, loads complete in order: 13.4), the start's code unrolled (instructions come from
// memory once per launch: 1500 more of them cost 1 us), the expansion spread over the first pass's K loop (15.7: a barrier per round).
#include "conv_mfma_resident.h"
#include "resident_kernel.h"

namespace bcnn {
namespace {

template <int WIDE>
__global__ __launch_bounds__(64 * RESIDENT_WAVES, 2) void conv_mfma_resident_kernel(
    ResidentArgs a, const uint32_t* __restrict__ x, const uint32_t* __restrict__ w, const int32_t* __restrict__ thr, uint32_t* __restrict__ out)
{
    constexpr int CB = RESIDENT_CHANNELS / 32;               // channel blocks
    __shared__ struct {
        // [channel block][K-step][unit of 16 bytes = a row's words' codes]: lane half h finds row i at unit 32 h + (i ^ 8 h)
        __align__(16) char weights[CB * RESIDENT_STEPS * 1024];
        v2i pixel[RESIDENT_COLUMNS * 32];                    // byte offset of the window's top-left tap, one validity bit per tap
        __align__(16) float start[RESIDENT_CHANNELS];        // what a channel's sums start from
    } lds;
    const ConvShape& s = a.s;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int hsel = lane >> 5, j = lane & 31;

    const ResidentPlace at = resident_place(a);
    const int o0 = at.o0;
    const ResidentRun columns = resident_run(a.quotient, a.rest, at.range);
    const int n_groups = a.n_groups, odd = n_groups & 1;

    const auto xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(x), 0, a.x_bytes, 0x00020000);
    const auto wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w), 0, a.w_bytes, 0x00020000);
    uint32_t m8, c2;                                         // held in registers: v_and_or_b32 takes no literals
    asm volatile("v_mov_b32 %0, 0x88888888" : "=v"(m8));
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));
    const uint32_t c4 = c2 << 1, c6 = c2 | c4;

    // ---- weights -> LDS.  Four waves a channel block, groups in turn; lane 2 r + h expands half h of row r (neighbouring lanes
    // read neighbouring 16 bytes, and neither the writes nor the readers' reads of a row's units meet in a bank)
    const int g0 = wave >> 1, wb = wave & 1;
    const int urow = lane >> 1, uhalf = lane & 1;
    const int uwords = uhalf ? s.cw - a.half : a.half;       // words of a tap that the half has
    const int uchannel = 32 * wb + row_to_channel(urow);
    const int urow_at = ((o0 + uchannel < s.c_out ? o0 + uchannel : s.c_out - 1) * a.n_words + uhalf * a.half) * 4;
    char* put_at = lds.weights + (wb * n_groups + g0) * WIDE * 1024 + (uhalf * 32 + (urow ^ (uhalf * 8))) * 16;
    auto fetch_w = [&](int gi, int (&v)[WIDE]) __attribute__((always_inline)) {
        const int tap = a.div_tap(gi);
        load_words(wres, urow_at + (tap * s.cw + WIDE * (gi - tap * a.per_tap)) * 4, v);
    };
    int pop = 0;                                             // the row's set bits at positions 4 i + 0 .. 2
    auto put_whole = [&](const int (&v)[WIDE]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < WIDE; ++i) {
            const uint32_t word = (uint32_t)v[i];
            pop += __builtin_popcount(word & 0x77777777u);
            *reinterpret_cast<v4i*>(put_at + i * 1024) =
                v4i{(int)(((word << 3) & m8) | c6), (int)(((word << 2) & m8) | c4), (int)(((word << 1) & m8) | c2), (int)((~word & m8) | c2)};
        }
    };
    // words that do not exist (past a half's end) and channels past c_in become 0.0, whatever the inputs hold there
    auto put_part = [&](int gi, const int (&v)[WIDE]) __attribute__((always_inline)) {
        const int k0 = WIDE * (gi - a.div_tap(gi) * a.per_tap);
#pragma unroll
        for (int i = 0; i < WIDE; ++i) {
            const uint32_t bits = k0 + i < uwords ? (uhalf * a.half + k0 + i == s.cw - 1 ? a.last_bits : ~0u) : 0u;
            const uint32_t word = (uint32_t)v[i];
            pop += __builtin_popcount(word & bits & 0x77777777u);
            const uint32_t s0 = (bits << 3) & m8, s1 = (bits << 2) & m8, s2 = (bits << 1) & m8, s3 = bits & m8;
            *reinterpret_cast<v4i*>(put_at + i * 1024) =
                v4i{(int)(((word << 3) & s0) | (s0 >> 1) | (s0 >> 2)), (int)(((word << 2) & s1) | (s1 >> 1)),
                    (int)(((word << 1) & s2) | (s2 >> 2)), (int)((~word & s3) | (s3 >> 2))};
        }
    };

    int threshold = 0;
    if (t < RESIDENT_CHANNELS) threshold = thr[o0 + t < s.c_out ? o0 + t : s.c_out - 1];
    {
        int v0[WIDE], v1[WIDE];
        fetch_w(g0, v0);
        fetch_w(g0 + 4, v1);
        // The weights' codes make a sum -(y + correction): the correction, sum of the channel's +-1 at positions 4 i + 0 .. 2, is
        // 2 popcount - positions.  |y| <= K, so thresholds beyond +-(K + 1) decide nothing new and are clamped.
        if (t < RESIDENT_CHANNELS) lds.start[t] = (float)(min(max(threshold, -s.k), s.k + 1) - a.low_bits) - 0.5f;
        meet();
        resident_places(a, lds.pixel, columns.first, columns.count < RESIDENT_COLUMNS ? columns.count : RESIDENT_COLUMNS);
#pragma unroll 1
        for (int gi = g0; gi < n_groups; gi += 4) {
            int v[WIDE];
#pragma unroll
            for (int i = 0; i < WIDE; ++i) { v[i] = v0[i]; v0[i] = v1[i]; }
            fetch_w(gi + 8, v1);
            if (a.whole) put_whole(v);
            else put_part(gi, v);
            put_at += 4 * WIDE * 1024;
        }
        atomicAdd(&lds.start[uchannel], (float)(2 * pop));   // (whole numbers and a half: exact in any order)
        meet();
    }

    auto expand_x = [&](uint32_t word) __attribute__((always_inline)) -> v8i {
        return v8i{(int)(word & 0x11111111u), (int)(word & 0x22222222u), (int)(word & 0x44444444u), (int)((word & m8) | c2), 0, 0, 0, 0};
    };
    const char* const my_weights = lds.weights + (hsel * 32 + (j ^ (hsel * 8))) * 16;
    const int block_bytes = n_groups * WIDE * 1024;

    // ---- P columns from column `col` on, whose places are in LDS from `place` on
    auto pass = [&](auto pc, int col, int place) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        int base[P], taps[P];
#pragma unroll
        for (int pb = 0; pb < P; ++pb) {
            const v2i q = lds.pixel[32 * (place + pb) + j];
            base[pb] = q[0] + hsel * a.half * 4;
            taps[pb] = q[1];
        }
        struct Inputs { int x[P][WIDE]; } ring[2];
        int f_tap = 0, f_g = 0;                              // next group to fetch
        auto fetch_x = [&](Inputs& c) __attribute__((always_inline)) {
            const int bit = f_tap < a.taps ? f_tap : 31;        // (bit 31 is never set: groups past the end read nothing)
            const int xo = (f_tap * a.tap_words + ((f_tap * 11) >> 5) * a.row_jump + WIDE * f_g) * 4;   // (11 tap) >> 5 is tap / 3 up to 8
#pragma unroll
            for (int pb = 0; pb < P; ++pb) {
                const int in = __builtin_amdgcn_sbfe(taps[pb], (uint32_t)bit, 1u);               // all bits or none
                load_words(xres, ((base[pb] + xo) & in) | (~in & PAST_ALL), c.x[pb]);
            }
            const bool done = f_g + 1 == a.per_tap;
            f_g = done ? 0 : f_g + 1;
            f_tap += done;
        };
        // (of an odd number of groups the first stands alone, in ring[1])
        if (odd) fetch_x(ring[1]);
        fetch_x(ring[0]);
        if (!odd) fetch_x(ring[1]);

        v16f acc[CB][P];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < 16; q += 4) {
                const v4f v = *reinterpret_cast<const v4f*>(&lds.start[32 * cb + 16 * hsel + q]);
#pragma unroll
                for (int pb = 0; pb < P; ++pb)
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc[cb][pb][q + k] = v[k];
            }
        struct Fragments { v4i f[CB]; } fw[2];
        const char* from = my_weights;
        auto read_w = [&](int ks, Fragments& f) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) f.f[cb] = *reinterpret_cast<const v4i*>(from + cb * block_bytes + ks * 1024);
        };
        read_w(0, fw[0]);
        // One input fragment ahead is expanded behind a matrix instruction, the next K-step's weights are read behind the first
        // (the last K-step's read ahead ends inside `lds` and is never multiplied).
        auto group = [&](const Inputs& c) __attribute__((always_inline)) {
            v8i next = expand_x((uint32_t)c.x[0][0]);
#pragma unroll
            for (int k = 0; k < WIDE; ++k) {
                read_w(k + 1, fw[(k + 1) & 1]);
                const v4i* const f = fw[k & 1].f;
#pragma unroll
                for (int pb = 0; pb < P; ++pb) {
                    const v8i fx = next;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const v8i w8 = {f[cb][0], f[cb][1], f[cb][2], f[cb][3], 0, 0, 0, 0};
                        acc[cb][pb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8, fx, acc[cb][pb], 4, 4, 0, 0, 0, 0);
                        if (cb == 0) {
                            if (pb + 1 < P) next = expand_x((uint32_t)c.x[pb + 1][k]);
                            else if (k + 1 < WIDE) next = expand_x((uint32_t)c.x[0][k + 1]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if constexpr (WIDE % 2) fw[0] = fw[1];
            from += WIDE * 1024;
        };
        if (odd) {
            group(ring[1]);
            fetch_x(ring[1]);
        }
#pragma unroll 1
        for (int gi = odd; gi < n_groups; gi += 2) {
            group(ring[0]);
            fetch_x(ring[0]);
            __builtin_amdgcn_sched_barrier(0);
            group(ring[1]);
            fetch_x(ring[1]);
            __builtin_amdgcn_sched_barrier(0);
        }

        // ---- signs -> words.  Rows past the end are past the buffer's size and store nothing.
        const int rows = s.m - 32 * col;
        const uint64_t row = reinterpret_cast<uint64_t>(out) + (uint64_t)col * (uint64_t)(32 * s.cwo * 4);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)row);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(row >> 32));
        const auto bits_res = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>((hi << 32) | lo), 0,
                                                                __builtin_amdgcn_readfirstlane((rows < 32 * P ? rows : 32 * P) * s.cwo * 4), 0x00020000);
        constexpr uint32_t NOWHERE = 0x7FFFFF00u;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int left = s.c_out - (o0 + 32 * cb);       // channels of the word
            const uint32_t valid = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
#pragma unroll
            for (int pb = 0; pb < P; pb += 2) {              // lanes of the lower half end up with column pb, those of the upper half with the next
                uint32_t half_word[2] = {0u, 0u};
#pragma unroll
                for (int e = 0; e < 2 && pb + e < P; ++e)
#pragma unroll
                    for (int r = 15; r >= 0; --r) half_word[e] = __builtin_amdgcn_alignbit(half_word[e], __float_as_uint(acc[cb][pb + e][r]), 31);
                const auto both = __builtin_amdgcn_permlane32_swap(half_word[0], half_word[1], false, false);
                const uint32_t to = (uint32_t)((32 * (pb + hsel) + j) * s.cwo + (o0 >> 5) + cb) * 4u;
                const bool ok = left > 0 && (pb + 1 < P || hsel == 0);
                __builtin_amdgcn_raw_buffer_store_b32((int)((both[0] | (both[1] << 16)) & valid), bits_res, (int)(ok ? to : NOWHERE), 0, 0);
            }
        }
    };
    resident_columns<RESIDENT_PASS, RESIDENT_COLUMNS>(a, columns, lds.pixel, wave, pass);
}

}  // namespace

hipError_t launch_conv_mfma_resident(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, uint32_t* out, hipStream_t stream)
{
    const SharedWalk walk = SharedWalk::make(s.cw, 9);
    if (s.ks != 3 || walk.steps(9) > RESIDENT_STEPS) return hipErrorInvalidValue;
    const ResidentArgs a = resident_args(s, 9, walk);
    const dim3 blocks((unsigned)(a.n_ranges * a.n_ctiles)), threads(64 * RESIDENT_WAVES);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, a, x, w, thr, out); };
    if (walk.wide == 3) go(conv_mfma_resident_kernel<3>);
    else if (walk.wide == 4) go(conv_mfma_resident_kernel<4>);
    else if (walk.wide == 5) go(conv_mfma_resident_kernel<5>);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace bcnn
