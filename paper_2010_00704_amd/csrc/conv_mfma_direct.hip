// Binary convolution on the matrix cores without LDS staging of the operands, for every channel count.
//
// Arithmetic as in conv_mfma_fp4_kernel.h (+-1 as 4-bit floats, exact fp32 sums; BCNN paper, Section 1: the
// operator is a matrix product; Section 4.2.1: operands are +-1, padding is -1), with the plain codes on both
// sides: bit b of a word becomes the nibble 0b1010 (-1.0) or 0b0010 (+1.0), seven vector instructions a
// fragment, and positions that are zero in both operands count +1 each, one constant for the whole call.
//
// What this kernel is for.  The staged kernel wants long launches of wide tiles: 128 channels x 256 pixels a
// workgroup, three LDS stages, 16-byte units that never straddle a tap (C_in a multiple of 128).  A small
// launch leaves it with a few workgroups on 256 compute units, each walking all of K alone, and a ragged channel
// count does not fit it at all.  Here a wave fetches its operands from global memory straight into the
// registers the matrix instruction's lanes need (lane = row of the tile, 16 bytes = four K-words of one row), so
// a tile needs no barrier until its sums are complete, and
//   - WK waves of a workgroup can split K between them and add their exact partial sums in LDS at the end;
//   - K is walked in 16-byte units per tap; a tap whose words are no multiple of four ends in a unit that starts
//     four words before the tap's end, and the words it shares with its neighbour are masked to zero on both
//     sides (TAIL); taps of fewer than four words are walked word by word over the flattened K axis (WORDS).
// Bound: latency for the small launches, vector-ALU issue (expansion, about seven instructions per MFMA with
// 2 x 2 blocks a wave) and the loads' latency for the large ones, HBM and the epilogue for module outputs of small K.
// Measured (graph replays, us, against the kernel that ran the call before): 3x3, 1024 -> 1024, one 7 x 7 image
// 25.2 -> 5.1; 3x3, 320 -> 200, 13 maps of 27 x 27 47.7 -> 11.3; 3x3, 64 -> 64, one 14 x 14 image 6.3 -> 4.4 (sums)
// and 10.3 -> 4.5 (bits); 3x3, 832 -> 224, 22 maps of 30 x 30 232 -> 27; 1x1 module, 1024 channels, 32 maps of
// 7 x 7 11.5 -> 7.5.
#include "bcnn_common.h"
#include "conv_mfma_direct.h"
#include "div_by.h"

#include <type_traits>

namespace bcnn {

struct DirectArgs {
    ConvShape s;
    int32_t n_ptiles, n_ctiles;
    int32_t per_tap;         // units per tap (WORDS: words per tap)
    int32_t n_units;         // units along K (WORDS: of the flattened word axis, the last one may be partial)
    int32_t n_words;         // taps * cw
    int32_t n_chunks;        // ceil(n_units / 2): a chunk is one unit per lane half = four K-steps
    int32_t z;               // 256 * n_chunks - K: positions that are zero on both sides and count +1 each
    int32_t x_bytes, w_bytes;
    int32_t row_jump;        // words added to the input offset per completed filter row
    DivBy div_ct, div_hw, div_wo, div_tap;
};

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

enum { OUT_I32 = 0, OUT_BITS = 1, OUT_MODULE = 2 };          // OUT_MODULE + REAL_*
enum { UNITS = 0, TAIL = 1, WORDS = 2 };

// MFMA row i of a 32-row block carries this channel of the block, so that a lane ends up holding 16
// consecutive channels of one pixel (lane half h, register r <-> channel 16h + r).
__device__ __forceinline__ int row_to_channel(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// A wave owns CB x PB blocks of 32 channels x 32 pixels; a workgroup WC x WP such tiles, each shared by WK
// waves that split K.
template <int CB, int PB, int WC, int WP, int WK, int OUT, int MODE>
__global__ __launch_bounds__(64 * WC * WP * WK) void conv_mfma_direct_kernel(
    DirectArgs a, const uint32_t* __restrict__ x, const uint32_t* __restrict__ w,
    const int32_t* __restrict__ thr, void* __restrict__ out, ModuleEp ep)
{
    constexpr bool MODULE = OUT >= OUT_MODULE;
    constexpr int REAL = MODULE ? OUT - OUT_MODULE : REAL_F32;
    constexpr bool HALF = REAL != REAL_F32;
    using real_t = typename real_type<REAL>::type;
    typedef real_t real4 __attribute__((ext_vector_type(4)));
    constexpr int TCH = 32 * CB, TPX = 32 * PB;              // a wave's tile
    // Partial (WK > 1) or complete sums on their way from the matrix layout to rows of channels.  WK = 1:
    // every wave turns one pixel block at a time around in a region of its own.
    constexpr int ROW = TCH + 4;                             // floats; rows stay 16-byte aligned, banks skewed by 4
    constexpr int REGION = (WK > 1 ? TPX : 32) * ROW;
    __shared__ __align__(16) float lds[WC * WP * WK * REGION];

    const ConvShape& s = a.s;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wk = wave % WK, wc = (wave / WK) % WC, wp = wave / (WK * WC);
    const int hsel = lane >> 5, j = lane & 31;

    // workgroup -> tile: each XCD takes a contiguous range, channel tile fastest
    int tile = blockIdx.x;
    {
        const int per_xcd = (a.n_ptiles * a.n_ctiles) >> 3;
        if (tile < per_xcd * 8) tile = (tile & 7) * per_xcd + (tile >> 3);
    }
    const int ptile = a.div_ct(tile);
    const int o0 = (tile - ptile * a.n_ctiles) * (TCH * WC) + TCH * wc;   // first channel and pixel of the wave's tile
    const int m0 = ptile * (TPX * WP) + TPX * wp;

    // ---- the lane's rows
    int wrow[CB];                                            // word offset of the weight row
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int ch = o0 + 32 * cb + row_to_channel(j);
        wrow[cb] = (ch < s.c_out ? ch : s.c_out - 1) * a.n_words;
    }
    int rbase[PB];                                           // word offset of the window's top-left tap
    uint32_t vmask[PB];                                      // one validity bit per tap
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        int m = m0 + 32 * pb + j;
        m = m < s.m ? m : s.m - 1;
        if (s.ks == 1 && s.stride == 1) {
            rbase[pb] = m * s.cw;
            vmask[pb] = 1u;
        } else {
            const int hw = s.ho * s.wo;
            const int n = a.div_hw(m);
            const int r = m - n * hw;
            const int oh = a.div_wo(r);
            const int ph = oh * s.stride - s.pad;
            const int pw = (r - oh * s.wo) * s.stride - s.pad;
            rbase[pb] = ((n * s.h + ph) * s.w + pw) * s.cw;
            uint32_t vm = 1u;                                // 1x1: no padding, always inside
            if (s.ks == 3) {
                uint32_t cols = 0;
                vm = 0;
#pragma unroll
                for (int v = 0; v < 3; ++v) cols |= (uint32_t)((uint32_t)(pw + v) < (uint32_t)s.w) << v;
#pragma unroll
                for (int u = 0; u < 3; ++u) vm |= ((uint32_t)(ph + u) < (uint32_t)s.h) ? cols << (3 * u) : 0u;
            }
            vmask[pb] = vm;
        }
    }

    // ---- identity vectors of the module's plain case are requested before the K loop.  After the transpose a
    // lane holds four consecutive channels, eight lanes a packed word; G such groups per lane.
    constexpr int CG = TCH / 4;                              // groups per pixel of the wave's tile
    constexpr int GROUPS = WK > 1 ? (TPX * CG + 64 * WK - 1) / (64 * WK) : TPX * CG / 64;
    const int lt = WK > 1 ? wk * 64 + lane : lane;           // place among the threads that share the tile
    const int c0 = o0 + 4 * (lt % CG);
    constexpr int PX_STEP = (WK > 1 ? 64 * WK : 64) / CG;    // pixels between a lane's groups
    const int px0 = lt / CG;
    const bool some = WK == 1 || (64 * WK <= TPX * CG) || px0 < TPX;
    bool vec = false;
    real4 ids[MODULE ? GROUPS : 1];
    const int id0 = MODULE ? c0 % (ep.id_channels > 0 ? ep.id_channels : 1) : 0;
    if constexpr (MODULE) {
        const uintptr_t both = reinterpret_cast<uintptr_t>(ep.r) | reinterpret_cast<uintptr_t>(ep.identity);
        vec = ep.identity && ep.r && ep.x_next && s.c_out % 4 == 0 && ep.id_channels % 4 == 0 && (both & (HALF ? 7 : 15)) == 0;
        if (vec) {
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                const int m = m0 + px0 + g * PX_STEP;
                ids[g] = real4{(real_t)0, (real_t)0, (real_t)0, (real_t)0};
                if (some && m < s.m && c0 < s.c_out)
                    ids[g] = __builtin_nontemporal_load(reinterpret_cast<const real4*>(
                        static_cast<const real_t*>(ep.identity) + (size_t)m * ep.id_channels + id0));
            }
        }
    }

    // ---- operands of one chunk: a unit (four words) of every row of the tile, straight into registers.  Offsets
    // past the buffers (taps outside the image, K padding) read as zero.
    const auto xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(x), 0, a.x_bytes, 0x00020000);
    const auto wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w), 0, a.w_bytes, 0x00020000);
    struct Chunk { v4i w[CB], x[PB]; };
    auto fetch = [&](int chunk, Chunk& c) {
        const int u = 2 * chunk + hsel;
        if constexpr (MODE != WORDS) {
            const int tap = a.div_tap(u);
            const int q = u - tap * a.per_tap;
            const bool real = u < a.n_units;
            int k = tap * s.cw + 4 * q;
            const bool last = MODE == TAIL && q == a.per_tap - 1;
            if constexpr (MODE == TAIL) {
                if (last) k = tap * s.cw + s.cw - 4;
            }
            const int xo = k + ((tap >= 3) + (tap >= 6)) * a.row_jump;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                c.w[cb] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                    wres, real ? (wrow[cb] + k) * 4 : -16, 0, 0));
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                const bool in = real && ((vmask[pb] >> (tap & 31)) & 1u);
                c.x[pb] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                    xres, in ? (rbase[pb] + xo) * 4 : -16, 0, 0));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 4 * u + i;
                const int tap = a.div_tap(k);
                const bool real = k < a.n_words;
                const int xo = k + ((tap >= 3) + (tap >= 6)) * a.row_jump;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    c.w[cb][i] = __builtin_bit_cast(int, __builtin_amdgcn_raw_buffer_load_b32(
                        wres, real ? (wrow[cb] + k) * 4 : -4, 0, 0));
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const bool in = real && ((vmask[pb] >> (tap & 31)) & 1u);
                    c.x[pb][i] = __builtin_bit_cast(int, __builtin_amdgcn_raw_buffer_load_b32(
                        xres, in ? (rbase[pb] + xo) * 4 : -4, 0, 0));
                }
            }
        }
    };
    // words that a tap's last unit shares with its neighbour count as zero on both sides
    const int shared = MODE == TAIL ? 4 * a.per_tap - s.cw : 0;   // 1 .. 3
    auto mask_tail = [&](int chunk, Chunk& c) {
        if constexpr (MODE == TAIL) {
            const int u = 2 * chunk + hsel;
            const int q = u - a.div_tap(u) * a.per_tap;
            const bool last = q == a.per_tap - 1;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int keep = last && i < shared ? 0 : -1;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) c.w[cb][i] &= keep;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) c.x[pb][i] &= keep;
            }
        }
    };
    uint32_t m8, c2;                                         // held in registers: v_and_or_b32 takes no literals
    asm volatile("v_mov_b32 %0, 0x88888888" : "=v"(m8));
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));
    auto expand = [&](uint32_t word) -> v8i {
        return v8i{(int)(((word << 3) & m8) | c2), (int)(((word << 2) & m8) | c2), (int)(((word << 1) & m8) | c2),
                   (int)((word & m8) | c2), 0, 0, 0, 0};
    };

    v16f acc[CB][PB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][pb][r] = 0.0f;

    auto multiply = [&](const Chunk& c) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            v8i fw[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) fw[cb] = expand((uint32_t)c.w[cb][ks]);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                const v8i fx = expand((uint32_t)c.x[pb][ks]);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    acc[cb][pb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw[cb], fx, acc[cb][pb], 4, 4, 0, 0, 0, 0);
            }
        }
    };
    // A wave takes the chunks wk, wk + WK, ...; AHEAD of them are in flight while one is multiplied.
    constexpr int AHEAD = (CB * PB == 1) ? 4 : 2;
    Chunk ring[AHEAD];
    const int mine = (a.n_chunks - wk + WK - 1) / WK;        // may be zero or negative
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (i < mine) fetch(wk + WK * i, ring[i]);
    for (int i = 0; i < mine; i += AHEAD) {
#pragma unroll
        for (int b = 0; b < AHEAD; ++b) {
            if (i + b < mine) {
                mask_tail(wk + WK * (i + b), ring[b]);
                multiply(ring[b]);
                if (i + b + AHEAD < mine) fetch(wk + WK * (i + b + AHEAD), ring[b]);
            }
        }
    }

    // ---- epilogue.  A pixel's channels through LDS: lane (pixel j, half h) holds channels 16h .. 16h+15 of a block.
    float* region = lds + (wp * WC + wc) * WK * REGION;
    auto park = [&](float* dst, int pb, int row0) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
                *reinterpret_cast<v4f*>(dst + (row0 + j) * ROW + 32 * cb + 16 * hsel + r) =
                    v4f{acc[cb][pb][r], acc[cb][pb][r + 1], acc[cb][pb][r + 2], acc[cb][pb][r + 3]};
    };
    const float zf = (float)a.z;
    // per-channel parameters of the lane's four channels (clamped loads for a ragged c_out)
    int th[4];
    float pg[4], pbi[4], pa[4], pc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int ch = c0 + k < s.c_out ? c0 + k : s.c_out - 1;
        if constexpr (OUT == OUT_BITS) th[k] = thr[ch];
        if constexpr (MODULE) {
            pg[k] = ep.scale[ch];
            pbi[k] = ep.bias[ch];
            pa[k] = ep.slope ? ep.slope[ch] : 1.0f;
            pc[k] = ep.next_bias ? ep.next_bias[ch] : 0.0f;
        }
    }
    const bool out_vec = OUT == OUT_I32 && s.c_out % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    // four sums (still with the constant z) of pixel m, channels c0 ..; every lane of the wave calls it
    auto emit = [&](v4f v, int m, bool ok, int g) {
        const int nch = s.c_out - c0;                        // real channels from c0 on (may be <= 0)
        uint32_t nib = 0;
        if constexpr (OUT == OUT_I32) {
            int32_t* y = static_cast<int32_t*>(out) + (size_t)m * s.c_out + c0;
            const v4i q = {(int)(v[0] - zf), (int)(v[1] - zf), (int)(v[2] - zf), (int)(v[3] - zf)};
            if (ok && nch > 0) {
                if (out_vec) {
                    __builtin_nontemporal_store(q, reinterpret_cast<v4i*>(y));
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (k < nch) y[k] = q[k];
                }
            }
            return;
        } else if constexpr (OUT == OUT_BITS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nib |= (uint32_t)(k < nch && (int)(v[k] - zf) >= th[k]) << k;
        } else {
            real_t* rp = static_cast<real_t*>(ep.r) + (size_t)m * s.c_out + c0;
            real4 id = ids[g];
            if (!vec) {
                const real_t* idrow = static_cast<const real_t*>(ep.identity) + (size_t)m * ep.id_channels;
#pragma unroll
                for (int k = 0; k < 4; ++k) id[k] = (ok && ep.identity && k < nch) ? idrow[(id0 + k) % ep.id_channels] : (real_t)0;
            }
            real4 st;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // a missing slope is the slope 1 (1 * t is t)
                const float val = module_value<REAL>(v[k] - zf, pg[k], pbi[k], vec || ep.identity != nullptr, (float)id[k], true, pa[k]);
                nib |= (uint32_t)(k < nch && val + pc[k] >= 0.0f) << k;
                st[k] = (real_t)val;
            }
            if (ok && nch > 0) {
                if (vec) {
                    *reinterpret_cast<real4*>(rp) = st;
                } else if (ep.r) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (k < nch) rp[k] = st[k];
                }
            }
        }
        // eight neighbouring lanes hold the 32 channels of one packed word
        uint32_t wd = nib << (4 * (lane & 7));
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x141, 0xF, 0xF, true);  // row_half_mirror
        uint32_t* yp = MODULE ? ep.x_next : static_cast<uint32_t*>(out);
        if (ok && nch > 0 && (lane & 7) == 0 && (!MODULE || yp)) yp[(size_t)m * s.cwo + (c0 >> 5)] = wd;
    };
    if constexpr (WK > 1) {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) park(region + wk * REGION, pb, 32 * pb);
        __syncthreads();
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int px = px0 + g * PX_STEP;
            v4f sum = {0.0f, 0.0f, 0.0f, 0.0f};
            if (some) {
#pragma unroll
                for (int k = 0; k < WK; ++k)
                    sum += *reinterpret_cast<const v4f*>(region + k * REGION + px * ROW + 4 * (lt % CG));
            }
            emit(sum, m0 + px, some && m0 + px < s.m, g);
        }
    } else {
        // same wave wrote and reads: LDS operations of a wave complete in order
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            park(region, pb, 0);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int g = 0; g < GROUPS / PB; ++g) {
                const int px = px0 + g * PX_STEP;
                const v4f sum = *reinterpret_cast<const v4f*>(region + px * ROW + 4 * (lt % CG));
                const int m = m0 + 32 * pb + px;
                emit(sum, m, m < s.m, pb * (GROUPS / PB) + g);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

template <int CB, int PB, int WC, int WP, int WK, int OUT>
hipError_t launch_mode(DirectArgs a, int mode, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                       const ModuleEp& ep, hipStream_t stream)
{
    a.n_ctiles = (a.s.c_out + 32 * CB * WC - 1) / (32 * CB * WC);
    a.n_ptiles = (a.s.m + 32 * PB * WP - 1) / (32 * PB * WP);
    a.div_ct = DivBy::make(a.n_ctiles);
    const dim3 blocks((unsigned)(a.n_ptiles * a.n_ctiles)), threads(64 * WC * WP * WK);
    if (mode == UNITS)
        hipLaunchKernelGGL((conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, UNITS>), blocks, threads, 0, stream, a, x, w, thr, out, ep);
    else if (mode == TAIL)
        hipLaunchKernelGGL((conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, TAIL>), blocks, threads, 0, stream, a, x, w, thr, out, ep);
    else
        hipLaunchKernelGGL((conv_mfma_direct_kernel<CB, PB, WC, WP, WK, OUT, WORDS>), blocks, threads, 0, stream, a, x, w, thr, out, ep);
    return hipGetLastError();
}

template <int CB, int PB, int WC, int WP, int WK>
hipError_t launch_out(const DirectArgs& a, int mode, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                      const ModuleEp* ep, hipStream_t stream)
{
    const ModuleEp none{};
    if (ep && ep->half == REAL_BF16) return launch_mode<CB, PB, WC, WP, WK, OUT_MODULE + REAL_BF16>(a, mode, x, w, thr, out, *ep, stream);
    if (ep && ep->half) return launch_mode<CB, PB, WC, WP, WK, OUT_MODULE + REAL_F16>(a, mode, x, w, thr, out, *ep, stream);
    if (ep) return launch_mode<CB, PB, WC, WP, WK, OUT_MODULE + REAL_F32>(a, mode, x, w, thr, out, *ep, stream);
    if (thr) return launch_mode<CB, PB, WC, WP, WK, OUT_BITS>(a, mode, x, w, thr, out, none, stream);
    return launch_mode<CB, PB, WC, WP, WK, OUT_I32>(a, mode, x, w, thr, out, none, stream);
}

}  // namespace

bool conv_mfma_direct_supported(const ConvShape& s)
{
    const int64_t n_words = (int64_t)s.ks * s.ks * s.cw;
    const int64_t x_bytes = (int64_t)s.n * s.h * s.w * s.cw * 4;
    const int64_t w_bytes = (int64_t)s.c_out * n_words * 4;
    // fp32 sums stay exact (the K axis is padded to at most four words per tap and a chunk); 31-bit byte offsets
    return (n_words + 3 * s.ks * s.ks + 8) * 32 < (1 << 22) && x_bytes < (1ll << 31) && w_bytes < (1ll << 31);
}

// What a tile of this kernel costs, in microseconds: a launch with its latencies, a wave's chain of chunks, a
// wave's set-up and epilogue and its chunks where more waves than SIMDs (1024) share the issue slots.  The four
// numbers of each tile are least-squares fits over 163 measured launches (graph replays; 1x1 and 3x3, strides 1 and
// 2, 7 to 1024 input and 32 to 1024 output channels, 25 to 430 000 pixels, sums and bits; rms error 11 to 16 %);
// choosing by them costs 1 % over the best of the tiles on average and 20 % at worst.
struct Cost { double fixed, chunk, wave, wave_chunk; };
struct TileCost { int tile, cb, pb, wc, wp, wk; Cost plain, module; };
// (module calls: 63 launches of 1x1 and 3x3 modules, 32 to 845 channels, all three stream types; rms 13 to 17 %,
// the choice 0.5 % over the best)
static const TileCost TILES[] = {
    {DIRECT_1x1_K4, 1, 1, 1, 1, 4, {2.55, 0.182, 0.129, 0.166}, {2.98, 0.000, 0.643, 0.133}},
    {DIRECT_2x2_K4, 2, 2, 1, 1, 4, {3.45, 0.450, 0.974, 0.330}, {4.08, 0.243, 2.080, 0.373}},
    {DIRECT_2x1, 2, 1, 1, 4, 1, {3.48, 0.308, 0.697, 0.205}, {5.30, 0.229, 2.360, 0.256}},
    {DIRECT_1x1, 1, 1, 1, 4, 1, {2.97, 0.199, 0.404, 0.144}, {3.88, 0.147, 1.350, 0.155}},
};
// The same for the staged kernel's 2 x 4 tile (83 launches, C_in a multiple of 128, rms 16 %; module calls: its plain
// form, 18 launches, rms 13 %): workgroups of 128 channels x 256 pixels against 256 compute units.
static double staged_cost(const ConvShape& s, bool module)
{
    const Cost c = module ? Cost{7.13, 0.772, 7.54, 0.279} : Cost{3.97, 0.597, 2.12, 0.227};
    const double chunks = (double)((s.ks * s.ks * (s.cw / 4) + 1) / 2);
    const double wgs = (double)((s.m + 255) / 256) * (double)((s.c_out + 127) / 128);
    return c.fixed + c.chunk * chunks + (c.wave + c.wave_chunk * chunks) * wgs / 256.0;
}

static int direct_mode(const ConvShape& s) { return s.cw < 4 ? WORDS : s.cw % 4 ? TAIL : UNITS; }
static int direct_units(const ConvShape& s)
{
    const int taps = s.ks * s.ks;
    return s.cw < 4 ? (taps * s.cw + 3) / 4 : taps * ((s.cw + 3) / 4);
}

int conv_mfma_direct_choose(const ConvShape& s, bool module, bool staged)
{
    const int chunks = (direct_units(s) + 1) / 2;
    int best = 0;
    double least = staged ? staged_cost(s, module) : 1e30;
    for (const TileCost& t : TILES) {
        const double wgs = (double)((s.m + 32 * t.pb * t.wp - 1) / (32 * t.pb * t.wp)) *
                           (double)((s.c_out + 32 * t.cb * t.wc - 1) / (32 * t.cb * t.wc));
        const double waves = wgs * t.wc * t.wp * t.wk / 1024.0;
        const double mine = (double)((chunks + t.wk - 1) / t.wk);
        const Cost& c = module ? t.module : t.plain;
        const double cost = c.fixed + c.chunk * mine + (c.wave + c.wave_chunk * mine) * waves;
        if (cost < least) { least = cost; best = t.tile; }
    }
    return best;
}

hipError_t launch_conv_mfma_direct(const ConvShape& s, const uint32_t* x, const uint32_t* w, const int32_t* thr, void* out,
                                   const ModuleEp* ep, int tile, hipStream_t stream)
{
    DirectArgs a;
    a.s = s;
    a.n_ptiles = a.n_ctiles = 0;     // set with the tile
    const int mode = direct_mode(s);
    a.n_words = s.ks * s.ks * s.cw;
    a.per_tap = mode == WORDS ? s.cw : (s.cw + 3) / 4;
    a.n_units = direct_units(s);
    a.n_chunks = (a.n_units + 1) / 2;
    a.z = 256 * a.n_chunks - s.k;
    a.x_bytes = (int32_t)((int64_t)s.n * s.h * s.w * s.cw * 4);
    a.w_bytes = (int32_t)((int64_t)s.c_out * a.n_words * 4);
    a.row_jump = (s.w - s.ks) * s.cw;
    a.div_hw = DivBy::make(s.ho * s.wo);
    a.div_wo = DivBy::make(s.wo);
    a.div_tap = DivBy::make(a.per_tap);
    switch (tile) {
        case DIRECT_1x1_K4: return launch_out<1, 1, 1, 1, 4>(a, mode, x, w, thr, out, ep, stream);
        case DIRECT_2x2_K4: return launch_out<2, 2, 1, 1, 4>(a, mode, x, w, thr, out, ep, stream);
        case DIRECT_2x1: return launch_out<2, 1, 1, 4, 1>(a, mode, x, w, thr, out, ep, stream);
        case DIRECT_1x1: return launch_out<1, 1, 1, 4, 1>(a, mode, x, w, thr, out, ep, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bcnn
