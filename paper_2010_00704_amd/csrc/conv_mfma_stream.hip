// 1x1 convolution modules of few words per pixel (C_in up to 256): the paper's building block (Section 4.2.1, first
// paragraph) on the matrix cores as a streaming kernel.
//
// At these sizes a module is its real stream: 2 bytes read and 2 written per element in half precision against
// C_in / 16 bits of packed operands, so HBM bounds it and everything else has to stay out of its way.
//   - A wave owns 32 pixels x 32 * CB channels: NKS matrix K-steps per 32 channels (lane half h takes the words
//     h * half_words .. of a row; words past the end are zero on both sides), operands straight from memory.
//   - The accumulators start at minus the count of positions that are zero on both sides, so the matrix result is the
//     integer sum itself.
//   - The sums turn from the matrix layout (lane = pixel, 16 channels) to rows of channels through a wave's own LDS
//     region: a lane then holds the 16 bytes of a row that one vector load and one vector store move, 8 channels of a
//     16-bit stream or 4 of a float one, and whole cache lines leave at once.
//   - The identity vectors are requested first of all; the stream may be updated in place (a wave reads and writes
//     its own elements only, and reads them first).  They are ordinary loads: the call before has usually just written
//     them, and non-temporal ones gave away what the last-level cache still held (22.9 against 20.7 us).
//   - Parameters are vector loads through buffers (a missing one is a buffer of no bytes): scalar loads under branches
//     cost more than the rest of a wave (28.6 against 22.9 us).
//   - One block per wave: walking two or four with the next one's operands in flight was slower at 55 of 64 shapes.
//   - Real-valued chain: the interface's order, one rounding per step.  It is most of a wave's instructions, and on few resident
//     waves their issue is not hidden: 12.3 us where the same loads and stores alone take 9.5 (half, 128 channels, 32 maps of 56 x
//     56), 9.7 and 6.7 (256 channels, 28 x 28).  Conversions inside the additions, one rounding per pair of elements, signs without
//     lane masks and no division where the identity is not replicated took 588 vector instructions to 489 (half; float 503,
//     bfloat16 553): 12.3 -> 12.1, 9.7 -> 8.7, 128 maps of 28 x 28 26.4 -> 24.2, 96 channels, 32 maps of 56 x 56 11.5 -> 10.9.
//     Tried: the parameters through LDS (28 registers fewer; 256 channels 24.2 -> 26.2, float 41 -> 45), and on top of it half of the
//     pixels at a time for a fifth wave on every SIMD (spills; 9.7, 29).
// The plain case only (every part of the module present, rows of whole 16-byte vectors); everything else takes the
// direct kernel.
// Measured (graph replays of one call, so partly from the last-level cache; us, against the kernel that ran the call before):
// half, 32 images: 64 channels, 112 x 112 31 -> 20 (22.6 from memory, 4.8 TB/s); 128 channels, 56 x 56 16.9 -> 12.4; 256
// channels, 28 x 28 10.6 -> 8.7; 32 channels, 224 x 224 50 -> 34; float, 256 channels, 56 x 56 43 -> 36.  On buffers that
// rotate through memory it is ahead of the kernels before it or within 4 % at all of 1098 sizes, types and channel counts, but for
// float, 256 -> 128 on 50 000 pixels and 256 -> 512 on 12 544 (0.92 and 0.93 times the staged kernel).
#include "bcnn_common.h"
#include "conv_mfma_direct.h"
#include "div_by.h"
#include "sign_bits.h"

#include <type_traits>

namespace bcnn {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct StreamArgs {
    ConvShape s;
    int32_t n_ctiles;        // workgroups along the channels
    int32_t half_words;      // ceil(cw / 2)
    int32_t z;               // positions that are zero on both sides
    int32_t x_bytes, w_bytes;
    DivBy div_ct, div_hw, div_wo;
};

__device__ __forceinline__ int row_to_channel(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// v + t in float.  Half: one instruction that converts on its way (fma with a factor of one that the compiler does not see; the
// product is exact, so there is one rounding, as in an addition).
template <int REAL>
__device__ __forceinline__ float plus(typename real_type<REAL>::type v, float t, float one)
{
    if constexpr (REAL == REAL_F16) return __builtin_fmaf((float)v, one, t);
    else return (float)v + t;
}

template <int NKS, int CB, int WC, int REAL>
__global__ __launch_bounds__(256, CB == 1 ? 4 : (REAL == REAL_F32 || NKS == 4) ? 2 : 3) void conv_mfma_stream_kernel(
    StreamArgs a, const uint32_t* __restrict__ x, const uint32_t* __restrict__ w, ModuleEp ep)
{
    using real_t = typename real_type<REAL>::type;
    constexpr int ESZ = REAL == REAL_F32 ? 4 : 2;
    constexpr int PER = 16 / ESZ;                            // channels of a 16-byte vector
    typedef real_t realv __attribute__((ext_vector_type(PER)));
    typedef real_t real2 __attribute__((ext_vector_type(2)));
    constexpr int TCH = 32 * CB;
    constexpr int CG = TCH / PER;                            // lanes per pixel
    constexpr int PX_STEP = 64 / CG;                         // pixels per vector instruction
    constexpr int GROUPS = 32 / PX_STEP;
    constexpr int ROW = TCH + 4;                             // floats; rows stay 16-byte aligned, banks skewed by 4
    __shared__ __align__(16) float lds[4 * 32 * ROW];

    const ConvShape& s = a.s;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wc = wave % WC, wp = wave / WC;
    const int hsel = lane >> 5, j = lane & 31;
    const int pt = a.div_ct((int)blockIdx.x);
    const int o0 = (((int)blockIdx.x - pt * a.n_ctiles) * WC + wc) * TCH;
    if (o0 >= s.c_out) return;                               // (no barrier in this kernel)
    constexpr int WP = 4 / WC;
    const int b = pt * WP + wp;                              // the wave's block of 32 pixels
    if (32 * b >= s.m) return;
    float* tile = lds + wave * (32 * ROW);

    uint32_t m8, c2;                                         // held in registers: v_and_or_b32 takes no literals
    asm volatile("v_mov_b32 %0, 0x88888888" : "=v"(m8));
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));
    float one;
    asm volatile("v_mov_b32 %0, 1.0" : "=v"(one));
    auto expand = [&](uint32_t word) -> v4i {
        return v4i{(int)(((word << 3) & m8) | c2), (int)(((word << 2) & m8) | c2), (int)(((word << 1) & m8) | c2),
                   (int)((word & m8) | c2)};
    };
    const auto xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(x), 0, a.x_bytes, 0x00020000);
    const auto wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w), 0, a.w_bytes, 0x00020000);
    const int half0 = hsel * a.half_words;
    // NKS words of a row from word offset `at`, zero past the row's end
    auto load_words = [&](const __amdgpu_buffer_rsrc_t& res, int at, bool row, int (&v)[NKS]) {
        if (s.cw == 2 * NKS) {
            const int off = row ? (at + half0) * 4 : -16;
            if constexpr (NKS == 1) {
                v[0] = (int)__builtin_amdgcn_raw_buffer_load_b32(res, off, 0, 0);
            } else if constexpr (NKS == 2) {
                const v2i q = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(res, off, 0, 0));
                v[0] = q[0]; v[1] = q[1];
            } else {
                const v4i q = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(res, off, 0, 0));
                v[0] = q[0]; v[1] = q[1]; v[2] = q[2]; v[3] = q[3];
            }
        } else {
#pragma unroll
            for (int i = 0; i < NKS; ++i) {
                const bool real = row && i < a.half_words && half0 + i < s.cw;
                v[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(res, real ? (at + half0 + i) * 4 : -4, 0, 0);
            }
        }
    };

    // ---- the lane's part of a pixel row
    const int cl = PER * (lane % CG);                        // channel within the wave's tile
    const int c0 = o0 + cl;
    const int px0 = lane / CG;
    const bool chan_ok = c0 < s.c_out;                       // c_out is a multiple of PER
    const int id_row = ep.id_channels * ESZ, r_row = s.c_out * ESZ, xn_row = s.cwo * 4;
    const uint32_t NOWHERE = 0x7FFFFFF0u;                    // past every buffer
    int id0 = c0;
    if (ep.id_channels != s.c_out) id0 = c0 % ep.id_channels;   // (uniform: a division is twenty instructions)
    const uint32_t id_off = chan_ok ? __umul24((uint32_t)px0, (uint32_t)id_row) + (uint32_t)(id0 * ESZ) : NOWHERE;
    const uint32_t r_off = chan_ok ? __umul24((uint32_t)px0, (uint32_t)r_row) + (uint32_t)(c0 * ESZ) : NOWHERE;
    const uint32_t xn_off = chan_ok && (cl & 31) == 0 ? __umul24((uint32_t)px0, (uint32_t)xn_row) + (uint32_t)((c0 >> 5) * 4) : NOWHERE;
    // the block's rows of a tensor: base and the bytes that exist
    auto rows_of = [&](const void* base, int row_bytes) {
        const int m = 32 * b;
        const int rows = s.m - m > 32 ? 32 : s.m - m;
        const uint64_t at = reinterpret_cast<uint64_t>(base) + (uint64_t)m * (uint64_t)row_bytes;
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>((hi << 32) | lo), 0,
                                                 __builtin_amdgcn_readfirstlane(rows * row_bytes), 0x00020000);
    };
    realv id[GROUPS];
    {
        const auto res = rows_of(ep.identity, id_row);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
            id[g] = __builtin_bit_cast(realv, __builtin_amdgcn_raw_buffer_load_b128(res, (int)(id_off + (uint32_t)(g * PX_STEP * id_row)), 0, 0));
    }
    int xw[NKS];
    {
        const int m = 32 * b + j;
        const bool row = m < s.m;
        int at = m;
        if (s.stride != 1) {
            const int hw = s.ho * s.wo, n = a.div_hw(row ? m : 0), r = (row ? m : 0) - n * hw, oh = a.div_wo(r);
            at = (n * s.h + oh * s.stride) * s.w + (r - oh * s.wo) * s.stride;
        }
        load_words(xres, at * s.cw, row, xw);
    }
    v4i fw[CB][NKS];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int ch = o0 + 32 * cb + row_to_channel(j);
        int v[NKS];
        load_words(wres, (int)__umul24((uint32_t)(ch < s.c_out ? ch : s.c_out - 1), (uint32_t)s.cw), true, v);
#pragma unroll
        for (int i = 0; i < NKS; ++i) fw[cb][i] = expand((uint32_t)v[i]);
    }
    // the lane's per-channel parameters; a missing slope is the slope 1 (1 * t is t), a missing next bias 0
    float pg[PER], pb[PER], pa[PER], pc[PER];
    auto load_params = [&](const float* p, float (&v)[PER]) {
        const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, p ? s.c_out * 4 : 0, 0x00020000);
#pragma unroll
        for (int k = 0; k < PER; k += 4) {
            const v4f q = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(res, chan_ok ? (c0 + k) * 4 : -16, 0, 0));
            v[k] = q[0]; v[k + 1] = q[1]; v[k + 2] = q[2]; v[k + 3] = q[3];
        }
    };
    load_params(ep.scale, pg);
    load_params(ep.bias, pb);
    load_params(ep.slope, pa);
    load_params(ep.next_bias, pc);
#pragma unroll
    for (int k = 0; k < PER; ++k) pc[k] = pc[k] + 0.0f;      // -0 becomes +0: no sum with it is -0
    if (!ep.slope) {
#pragma unroll
        for (int k = 0; k < PER; ++k) pa[k] = 1.0f;
    }
    v16f start;
#pragma unroll
    for (int r = 0; r < 16; ++r) start[r] = (float)-a.z;

    v16f acc[CB];
#pragma unroll
    for (int i = 0; i < NKS; ++i) {
        const v4i q = expand((uint32_t)xw[i]);
        const v8i fx = {q[0], q[1], q[2], q[3], 0, 0, 0, 0};
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const v4i p = fw[cb][i];
            const v8i fwv = {p[0], p[1], p[2], p[3], 0, 0, 0, 0};
            acc[cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fwv, fx, i ? acc[cb] : start, 4, 4, 0, 0, 0, 0);
        }
    }
    // same wave writes and reads: LDS operations of a wave complete in order
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int r = 0; r < 16; r += 4)
            *reinterpret_cast<v4f*>(tile + j * ROW + 32 * cb + 16 * hsel + r) =
                v4f{acc[cb][r], acc[cb][r + 1], acc[cb][r + 2], acc[cb][r + 3]};
    __builtin_amdgcn_wave_barrier();
    const auto r_res = rows_of(ep.r, r_row);
    const auto xn_res = rows_of(ep.x_next, xn_row);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const float* from = tile + (g * PX_STEP + px0) * ROW + cl;
        float y[PER];
#pragma unroll
        for (int q = 0; q < PER; q += 4) {
            const v4f v = *reinterpret_cast<const v4f*>(from + q);
            y[q] = v[0]; y[q + 1] = v[1]; y[q + 2] = v[2]; y[q + 3] = v[3];
        }
        float t[PER], stored[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            t[k] = plus<REAL>(id[g][k], __builtin_fmaf(pg[k], y[k], pb[k]), one);
            const float neg = pa[k] * t[k];
            t[k] = t[k] >= 0.0f ? t[k] : neg;
        }
        v4i st;
#pragma unroll
        for (int k = 0; k < PER; k += PER / 4) {
            if constexpr (REAL == REAL_F32) {
                st[k] = __float_as_int(t[k]);
                stored[k] = t[k] + pc[k];
            } else {
                // rounded two at a time; what the stream stores is read back from the packed pair (which the asm hides: the
                // compiler would round every element a second time)
                int pair = __builtin_bit_cast(int, real2{(real_t)t[k], (real_t)t[k + 1]});
                asm("" : "+v"(pair));
                const real2 two = __builtin_bit_cast(real2, pair);
                stored[k] = plus<REAL>(two[0], pc[k], one);
                stored[k + 1] = plus<REAL>(two[1], pc[k + 1], one);
                st[k / 2] = pair;
            }
        }
        const uint32_t bits = sign_bits_of_sums(stored);
        __builtin_amdgcn_raw_buffer_store_b128(st, r_res, (int)(r_off + (uint32_t)(g * PX_STEP * r_row)), 0, 0);
        // 32 / PER neighbouring lanes hold the 32 channels of one packed word
        uint32_t wd = (chan_ok ? bits : 0u) << (cl & 31);
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0xB1, 0xF, 0xF, true);       // quad_perm [1,0,3,2]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x4E, 0xF, 0xF, true);       // quad_perm [2,3,0,1]
        if constexpr (PER == 4)
            wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x141, 0xF, 0xF, true);  // row_half_mirror
        __builtin_amdgcn_raw_buffer_store_b32((int)wd, xn_res, (int)(xn_off + (uint32_t)(g * PX_STEP * xn_row)), 0, 0);
    }
}

}  // namespace

bool conv_mfma_stream_supported(const ConvShape& s, const ModuleEp& ep)
{
    const int per = ep.half == REAL_F32 ? 4 : 8;
    const uintptr_t both = reinterpret_cast<uintptr_t>(ep.r) | reinterpret_cast<uintptr_t>(ep.identity);
    const int64_t x_bytes = (int64_t)s.n * s.h * s.w * s.cw * 4, w_bytes = (int64_t)s.c_out * s.cw * 4;
    // (c_out bound: 32 rows of any of the three streams stay below 2^31 bytes)
    return s.ks == 1 && s.cw <= 8 && ep.identity && ep.r && ep.x_next && s.c_out % per == 0 && ep.id_channels % per == 0 &&
           (both & 15) == 0 && s.c_out <= (1 << 20) && x_bytes < (1ll << 31) && w_bytes < (1ll << 31);
}

hipError_t launch_conv_mfma_stream(const ConvShape& s, const uint32_t* x, const uint32_t* w, const ModuleEp& ep, hipStream_t stream)
{
    StreamArgs a;
    a.s = s;
    a.half_words = (s.cw + 1) / 2;
    const int nks = a.half_words <= 1 ? 1 : a.half_words <= 2 ? 2 : 4;
    a.z = 64 * nks - s.k;
    a.x_bytes = (int32_t)((int64_t)s.n * s.h * s.w * s.cw * 4);
    a.w_bytes = (int32_t)((int64_t)s.c_out * s.cw * 4);
    a.div_hw = DivBy::make(s.ho * s.wo);
    a.div_wo = DivBy::make(s.wo);
    // 64 channels a wave unless that leaves SIMDs idle (up to 1024 waves: 32 channels, 64 channels on 20 480 pixels
    // 4.4 -> 4.1 us, on 228 096 pixels 13.3 against 16.1) or there are no more than 32; two waves side by side
    // along the channels where they fill 128 (128 channels, 410 874 pixels 37.9 -> 34.7 us) and not where half of
    // the second would idle (192 channels, 139 638 pixels 34.4 against 27.2 us).
    const int64_t blocks = ((int64_t)s.m + 31) / 32, c64 = (s.c_out + 63) / 64;
    const bool narrow = s.c_out <= 32 || blocks * c64 <= 1024;
    const bool pair = !narrow && c64 % 2 == 0;
    a.n_ctiles = narrow ? (s.c_out + 31) / 32 : (int)(pair ? c64 / 2 : c64);
    a.div_ct = DivBy::make(a.n_ctiles);
    const int wp = pair ? 2 : 4;
    const dim3 grid((unsigned)((blocks + wp - 1) / wp * a.n_ctiles));
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, a, x, w, ep); };
    auto tile = [&](auto n, auto real) {
        constexpr int N = decltype(n)::value, R = decltype(real)::value;
        if (narrow) go(conv_mfma_stream_kernel<N, 1, 1, R>);
        else if (pair) go(conv_mfma_stream_kernel<N, 2, 2, R>);
        else go(conv_mfma_stream_kernel<N, 2, 1, R>);
    };
    auto type = [&](auto n) {
        if (ep.half == REAL_BF16) tile(n, std::integral_constant<int, REAL_BF16>{});
        else if (ep.half) tile(n, std::integral_constant<int, REAL_F16>{});
        else tile(n, std::integral_constant<int, REAL_F32>{});
    };
    if (nks == 1) type(std::integral_constant<int, 1>{});
    else if (nks == 2) type(std::integral_constant<int, 2>{});
    else type(std::integral_constant<int, 4>{});
    return hipGetLastError();
}

}  // namespace bcnn
