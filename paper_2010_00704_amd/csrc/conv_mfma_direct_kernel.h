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
// 25.2 -> 5.1; 3x3, 320 -> 200, 13 maps of 27 x 27 47.7 -> 10.1 (8.9 among other calls); 3x3, 64 -> 64, one 14 x 14 image 6.3 -> 4.4 (sums)
// and 10.3 -> 4.5 (bits); 3x3, 832 -> 224, 22 maps of 30 x 30 232 -> 27; 1x1 module, 1024 channels, 32 maps of
// 7 x 7 11.5 -> 7.5.  At least two workgroups of a SIMD are asked for in the launch bounds: without that the compiler
// keeps the accumulators in the accumulation registers and copies them (2 x 1 blocks: 84 registers a lane instead of
// 96; the second call above took 11.3 before that, the third takes 2.9 since).
// Buffer accesses in the epilogue instead of predicated ones: float module, 1x1, 256 channels, 32 maps of 56 x 56 (1 x 1
// blocks) 39.3 -> 33.2, half, 64 channels, 112 x 112 30.9 -> 24.8; sums, 1x1, 256 -> 256, 32 maps of 56 x 56 19.3 (staged 22.5).
// Shared weights (WIDE > 0): the larger launches of those.  There every wave expanded both operands for itself, seven
// instructions a fragment, and read its weight rows 16 bytes to a cache line: vector issue and L1 look-ups bound it at three
// to six times the matrix cores' time.  Now a workgroup expands a stage of weights once, into LDS, for its four waves, which
// lie along the pixels: a fragment is one 16-byte LDS read, and what is left of the expansion is the inputs'.  Two stages
// in turn, one barrier each (LDS only: loads stay in flight across it); a 2 x 2 tile keeps LDS reads at half of their rate
// (2 x 1: all of it, and still level, because its launches balance better).  Weights of words that do not exist are 0.0, so the
// walk needs no masks on the inputs and no constant afterwards; bits start their sums at 1/2 - threshold and leave as signs,
// without a turn through LDS.  Phase clocks of 3x3, 256 -> 256, 784 workgroups: set-up 3400 cycles, the loop 36 to 40 cycles per
// MFMA and SIMD with two to four workgroups a compute unit (the instruction's own rate is 35.4), end 30: the launch is
// bound by what the dispatcher leaves uneven (two to four workgroups a compute unit where three would do).
// Measured (us, before and after): bits, 3x3, 320 -> 192, 39 maps of 38 x 38 27.9 -> 16.3; 220 -> 64, 440 000 pixels 45 -> 27; 1x1,
// 704 -> 704, 40 maps of 26 x 26 14.9 -> 10.8; sums, 3x3, 468 -> 39, 191 maps of 37 x 36 52 -> 38; half module, 3x3, 131 -> 256,
// 97 500 pixels 49 -> 41.  Tried: 4 x 2 and 2 x 4 blocks a wave (one wave per SIMD takes 67 cycles per MFMA, waiting for LDS
// and barriers; nowhere ahead), halves of a tap side by side in 32-byte pieces (wide rows no faster, all rows 3 % slower).
// Branch mode has three forms (shared_plan.h): every wave its own operands, shared weights, and for small launches waves that
// take whole taps of a block and scale and add their sums in order at the end (a wave's chain is a quarter as long).  With
// shared weights the pixels are the instruction's rows, so that a tap's scale is one register a block: 16-byte scale reads
// took as much LDS time as the weights (24.7 us against 26.7 on the first call below), and zeros as an inline start
// operand replace a move per element and tap.  Measured in graphs, us: 3x3, 256 -> 256, 64 maps of 28 x 28, bits, pad words 34.9 every
// wave for itself and 23.4 shared (a pass 33.6 and 22.2 to 23.4, by box; the staged kernel 64), -1 outside 30.7 and 22.9, nothing
// outside 33.4 and 24.7; 512 -> 512, 10 maps of 14 x 14 12.3 and 9.4; 160 -> 160, 49 maps of 41 x 41, float 44.6 and 24.8; 64 -> 64, 213 maps of
// 39 x 42, half tail 57 and 39; 384 -> 384, 2 maps of 13 x 13, bits 13.2 and, taps apart, 5.4.  Counters of the first of these: vector units
// busy for 40 % of the time, matrix cores 19, LDS 24; its 1568 workgroups are one and a half rounds of four a compute unit.  2 x 2 blocks a wave (two waves per SIMD) 28.8 on the first of these, 1 x 2 36.8.
#pragma once
#include "bcnn_common.h"
#include "branch_walk.h"
#include "direct_plan.h"
#include "div_by.h"
#include "shared_plan.h"

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
    // branch mode
    int32_t taps;            // branches
    int32_t tap_step;        // words between the branches' input tensors
    int32_t pad_bytes;
};

// What only some forms of the kernel read.  Branch mode: per-branch scales, bias, what a tap outside the image stands for;
// shared weights: how a tap's words are split (shared_plan.h).
struct DirectBranch {
    const float* scale;         // [taps][c_out]
    const float* bias;          // [c_out] or nullptr
    const uint32_t* pad_words;  // [taps][cw] (PAD_OPERAND)
    int32_t half;               // words of the longer lane half
    uint32_t last_bits;         // channels of a pixel's last word
};

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v3i __attribute__((ext_vector_type(3)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

enum { OUT_I32 = 0, OUT_BITS = 1, OUT_MODULE = 2 };          // OUT_MODULE + REAL_*
// Branch mode (F x F convolution as F*F shifted 1x1 branches, or P parallel ones, each with a real scale per output
// channel: Section 4.2.1, last paragraph; Figure 2, bottom).  OUT_I32 then stores float sums, OUT_BITS z >= 0.
enum { PAD_NONE = 0, PAD_OPERAND = 1, PAD_NOTHING = 2 };     // outside the image: -1, the branch's pad words, no contribution
constexpr int BRANCH = 4;                                    // MODE = BRANCH + PAD_*
constexpr int MAX_BRANCHES = 16;                             // scales kept in LDS

// MFMA row i of a 32-row block carries this channel of the block, so that a lane ends up holding 16
// consecutive channels of one pixel (lane half h, register r <-> channel 16h + r).
__device__ __forceinline__ int row_to_channel(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// A wave owns CB x PB blocks of 32 channels x 32 pixels; a workgroup WC x WP such tiles, each shared by WK
// waves that split K.
template <int CB, int PB, int WC, int WP, int WK, int OUT, int MODE, int WIDE = 0>
__global__ __launch_bounds__(64 * WC * WP * WK, (WIDE > 0 && MODE < BRANCH && OUT != OUT_MODULE) ? 3 : 2) void conv_mfma_direct_kernel(
    DirectArgs a, const uint32_t* __restrict__ x, const uint32_t* __restrict__ w,
    const int32_t* __restrict__ thr, void* __restrict__ out, ModuleEp ep, DirectBranch br)
{
    constexpr bool BR = MODE >= BRANCH;
    constexpr int PAD = BR ? MODE - BRANCH : PAD_NONE;
    constexpr bool TAPS_APART = BR && WK > 1;                // the waves of a tile take whole taps
    static_assert(!TAPS_APART || (CB == 1 && PB == 1), "one block of 32 x 32 shared by the waves");
    constexpr bool MODULE = OUT >= OUT_MODULE;
    constexpr int REAL = MODULE ? OUT - OUT_MODULE : REAL_F32;
    constexpr bool HALF = REAL != REAL_F32;
    using real_t = typename real_type<REAL>::type;
    typedef real_t real4 __attribute__((ext_vector_type(4)));
    typedef real_t real4_any __attribute__((ext_vector_type(4), aligned(sizeof(real_t))));
    constexpr int TCH = 32 * CB, TPX = 32 * PB;              // a wave's tile
    // Partial (WK > 1) or complete sums on their way from the matrix layout to rows of channels.  WK = 1:
    // every wave turns one pixel block at a time around in a region of its own.
    constexpr int ROW = TCH + 4;                             // floats; rows stay 16-byte aligned, banks skewed by 4
    constexpr int REGION = (WK > 1 ? TPX : 32) * ROW;
    constexpr bool SHARED = WIDE > 0;
    // Branch mode with shared weights has the pixels as the instruction's rows: a lane holds 16 pixels of one channel, and a
    // tap's scale is one register a block.  Everywhere else a lane holds 16 channels of one pixel.
    constexpr bool LANE_CHANNEL = SHARED && BR;
    static_assert(!SHARED || (WC == 1 && WK == 1), "shared weights: the workgroup's waves lie along the pixels");
    constexpr int SG = SHARED ? WP / CB : 1;                 // groups of a stage: every thread expands one unit of it
    constexpr int STEPS = WIDE < 3 ? 4 : WIDE;               // K-steps of a group
    constexpr int STAGE = SG * STEPS * CB * 1024;            // bytes
    constexpr bool SIGN_OUT = SHARED && OUT == OUT_BITS && !BR;
    constexpr int EP_FLOATS = SIGN_OUT ? 0 : TAPS_APART ? APART_TAPS * REGION : WC * WP * WK * REGION;
    __shared__ __align__(16) float lds[EP_FLOATS > 2 * STAGE / 4 || !SHARED ? EP_FLOATS : 2 * STAGE / 4];

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

    // shared weights: what a channel's sums start from is asked for first (see below)
    int start = 0;
    if constexpr (SHARED && (BR || SIGN_OUT)) {
        const void* from = BR ? static_cast<const void*>(br.bias) : thr;
        const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(from), 0, from ? s.c_out * 4 : 0, 0x00020000);
        start = (int)__builtin_amdgcn_raw_buffer_load_b32(res, (o0 + t) * 4, 0, 0);
    }

    // ---- the lane's rows
    int wrow[CB];                                            // word offset of the weight row
#pragma unroll
    for (int cb = 0; cb < CB && !SHARED; ++cb) {
        const int ch = o0 + 32 * cb + row_to_channel(j);
        wrow[cb] = (ch < s.c_out ? ch : s.c_out - 1) * a.n_words;
    }
    int rbase[PB];                                           // word offset of the window's top-left tap
    uint32_t vmask[PB];                                      // one validity bit per tap
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        int m = m0 + 32 * pb + (LANE_CHANNEL ? row_to_channel(j) : j);
        m = m < s.m ? m : s.m - 1;
        if (s.ks == 1 && s.stride == 1) {
            rbase[pb] = m * s.cw;
            vmask[pb] = 0xFFFFu;
        } else {
            const int hw = s.ho * s.wo;
            const int n = a.div_hw(m);
            const int r = m - n * hw;
            const int oh = a.div_wo(r);
            const int ph = oh * s.stride - s.pad;
            const int pw = (r - oh * s.wo) * s.stride - s.pad;
            rbase[pb] = ((n * s.h + ph) * s.w + pw) * s.cw;
            uint32_t vm = 0xFFFFu;                           // 1x1: no padding, every branch is inside
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
    auto first_id = [&](int c) { return c % (ep.id_channels > 0 ? ep.id_channels : 1); };
    auto turn_of = [&](int id) { return id > ep.id_channels - 4 ? id + 4 - ep.id_channels : 0; };
    // Output tensors (and the identity) are raw buffers per wave tile: base = the row of the tile's first pixel, size =
    // its rows that exist.  Rows past the end read zeros and store nothing, and so does a lane without channels, whose
    // offset is past every size: no predicates between the accesses.
    constexpr uint32_t NOWHERE = 0x7FFFFF00u;
    const bool chan_ok = some && c0 < s.c_out;
    auto rows_of = [&](const void* base, int row_bytes) {
        int rows = s.m - m0;
        rows = rows < 0 ? 0 : (rows > TPX ? TPX : rows);
        const uint64_t at = reinterpret_cast<uint64_t>(base) + (uint64_t)m0 * (uint64_t)row_bytes;
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>((hi << 32) | lo), 0,
                                                 __builtin_amdgcn_readfirstlane(base ? rows * row_bytes : 0), 0x00020000);
    };
    constexpr int ESZ = (int)sizeof(real_t);
    if constexpr (MODULE) {
        const uintptr_t both = reinterpret_cast<uintptr_t>(ep.r) | reinterpret_cast<uintptr_t>(ep.identity);
        // (a missing identity, real stream or next packing is a buffer of no bytes)
        const int id0 = first_id(c0);
        vec = s.c_out % 4 == 0 && ep.id_channels % 4 == 0 && (both & 3) == 0;
        if (vec) {
            const int row_bytes = ep.id_channels * ESZ;
            const auto res = rows_of(ep.identity, row_bytes);
            const uint32_t off = chan_ok ? (uint32_t)(px0 * row_bytes + id0 * ESZ) : NOWHERE;
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                const int at = (int)(off + (uint32_t)(g * PX_STEP * row_bytes));
                if constexpr (HALF) ids[g] = __builtin_bit_cast(real4, __builtin_amdgcn_raw_buffer_load_b64(res, at, 0, 0));
                else ids[g] = __builtin_bit_cast(real4, __builtin_amdgcn_raw_buffer_load_b128(res, at, 0, 0));
            }
        } else if (ep.identity && ep.id_channels >= 4) {
            // rows off a vector's grid: the same at the elements' own alignment, without branches.  Rows past the end read the
            // last one, a lane whose four channels reach past the row its last four, `turn` back.
            // (Kernel times, us, against an element a load after the K loop and an element a store: 1x1, half, 711 channels, 5 maps of
            // 102 x 102 76 -> 50; 105 channels, 16 of 56 x 56 15.0 -> 11.1, float 18.6 -> 11.8; 3x3, float, 700 -> 701, 16 of 56 x 56
            // 196 -> 151; 6 of 18 x 18, 1x1, 318 channels 4.9 -> 4.4.)
            const real_t* const from = static_cast<const real_t*>(ep.identity) + (chan_ok ? id0 - turn_of(id0) : 0);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                const int m = m0 + px0 + g * PX_STEP;
                ids[g] = *reinterpret_cast<const real4_any*>(from + (int64_t)(m < s.m ? m : s.m - 1) * ep.id_channels);
            }
        } else {
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) ids[g] = real4{};
        }
    }

    // ---- operands of one chunk: a unit (four words) of every row of the tile, straight into registers.  Offsets
    // past the buffers (taps outside the image, K padding) read as zero.
    const auto xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(x), 0, a.x_bytes, 0x00020000);
    const auto wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w), 0, a.w_bytes, 0x00020000);
    // (pad words are a second load, added when the chunk is multiplied: added at once it would wait for both loads)
    struct Chunk { v4i w[CB], x[PB], pad[PAD == PAD_OPERAND ? PB : 1]; };
    auto fetch = [&](int chunk, Chunk& c) {
        const int u = 2 * chunk + hsel;
        if constexpr (MODE == UNITS || MODE == TAIL) {
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
        } else if constexpr (MODE == WORDS) {
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
    v16f tot[BR && !TAPS_APART ? CB : 1][BR && !TAPS_APART ? PB : 1];   // branch mode: the scaled sum so far
    __shared__ __align__(16) float apart_scale[TAPS_APART ? APART_TAPS : 1][TCH];
    __shared__ uint32_t apart_mask[32];                      // validity bits of the tile's pixels

    auto multiply = [&](const Chunk& c, int steps) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (BR && ks >= steps) break;
            v8i fw[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) fw[cb] = expand((uint32_t)c.w[cb][ks]);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                const v8i fx = expand((uint32_t)(PAD == PAD_OPERAND ? c.x[pb][ks] | c.pad[pb][ks] : c.x[pb][ks]));
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    acc[cb][pb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw[cb], fx, acc[cb][pb], 4, 4, 0, 0, 0, 0);
            }
        }
    };
    if constexpr (SHARED) {
        // Weights: a stage of SG groups of four K-steps is expanded once for all waves, in LDS, double buffered; thread t
        // expands four words of row t % (32 CB), fetched a stage ahead.  Inputs: every wave's own rows, a group in
        // registers two groups ahead.  Words that do not exist (the shorter half's last one, groups past the end,
        // channels past c_in) are 0.0 on the weights' side, whatever the input's words are: no constant is left to correct.
        constexpr bool NARROW = WIDE < 3;                    // several taps a group
        constexpr int ROWS = 32 * CB, TPG = NARROW ? 4 / WIDE : 1;
        char* const stage = reinterpret_cast<char*>(lds);
        const int urow = t % ROWS, unit = ROWS >= 64 ? wave / (ROWS / 64) : t / ROWS;
        const int ugroup = unit >> 1, uhalf = unit & 1;
        int urow_words;
        {
            const int ch = o0 + (LANE_CHANNEL ? urow : (urow & ~31) + row_to_channel(urow & 31));
            urow_words = (ch < s.c_out ? ch : s.c_out - 1) * a.n_words;
        }
        const int n_groups = a.n_units;
        const int tap_words = a.tap_step + (s.ks == 3 ? s.cw : 0), row_words = s.ks == 3 ? a.row_jump : 0;
        // word offset of a tap in the input, from the window's top-left one; (11 tap) >> 5 is tap / 3 up to 8
        auto tap_at = [&](int tap) __attribute__((always_inline)) { return tap * tap_words + ((tap * 11) >> 5) * row_words; };
        int rb[PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) rb[pb] = (rbase[pb] + hsel * br.half) * 4;
        const auto pres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(br.pad_words), 0, PAD == PAD_OPERAND ? a.pad_bytes : 0, 0x00020000);
        // (no part of the offset in the scalar one, which the bounds check leaves out)
        auto load_words = [&](auto res, int off, auto& v, int at) __attribute__((always_inline)) {
            if constexpr (WIDE >= 4) {
                const v4i q = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(res, off, 0, 0));
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = q[i];
                if constexpr (WIDE == 5) v[4] = (int)__builtin_amdgcn_raw_buffer_load_b32(res, (int)((uint32_t)off + 16u), 0, 0);
            } else if constexpr (WIDE == 3) {
                const v3i q = __builtin_bit_cast(v3i, __builtin_amdgcn_raw_buffer_load_b96(res, off, 0, 0));
#pragma unroll
                for (int i = 0; i < 3; ++i) v[i] = q[i];
            } else if constexpr (WIDE == 2) {
                const v2i q = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(res, off, 0, 0));
                v[at] = q[0];
                v[at + 1] = q[1];
            } else v[at] = (int)__builtin_amdgcn_raw_buffer_load_b32(res, off, 0, 0);
        };
        // Pad words are a second load, added when the group is multiplied: added where it is fetched it waits for both loads.  A
        // module's tail of 2 x 1 blocks, and a float one of two or four words, have no registers for that: a wave less on every SIMD can
        // cost more than the wait (64 -> 64, 80 maps of 39 x 39, half 18.0 us and 19.3 added later; 200 -> 200, 20 maps of 27 x 27, float
        // 17.0 and 18.3).  The other tails of 1 x 1 blocks: one word a load 1.12 times faster over 480 calls, half ones of two words 1.10, the
        // rest level; before, 27 of those 480 were up to 12 % slower than with a wave's own operands, one is.
        constexpr bool PAD_LATER = PAD == PAD_OPERAND && (!MODULE || (CB == 1 && !(REAL == REAL_F32 && WIDE % 2 == 0)));
        struct Inputs { int x[PB][STEPS], pad[PAD_LATER ? PB : 1][STEPS]; };
        auto fetch_x = [&](int gi, Inputs& c) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < TPG; ++i) {
                const int tap = NARROW ? gi * TPG + i : a.div_tap(gi);
                const int k = NARROW ? 0 : WIDE * (gi - tap * a.per_tap);
                const int bit = tap < a.taps ? tap : 31;     // (bit 31 is never set)
                const int xo = (tap_at(tap) + k) * 4;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const int in = __builtin_amdgcn_sbfe((int)vmask[pb], (uint32_t)bit, 1u);     // all bits or none
                    load_words(xres, ((rb[pb] + xo) & in) | (~in & PAST_ALL), c.x[pb], i * WIDE);
                    if constexpr (PAD == PAD_OPERAND) {
                        const int at = (((tap * s.cw + hsel * br.half + k) * 4) & ~in) | (in & PAST_ALL);
                        if constexpr (PAD_LATER) load_words(pres, at, c.pad[pb], i * WIDE);
                        else if (!NARROW || s.ks == 3) {     // (always: the branch keeps the loads of a narrow group's taps apart, else again too many registers)
                            int p[STEPS];
                            load_words(pres, at, p, i * WIDE);
#pragma unroll
                            for (int q = i * WIDE; q < (i + 1) * WIDE; ++q) c.x[pb][q] |= p[q];
                        }
                    }
                }
            }
        };
        auto fetch_w = [&](int st, int (&v)[STEPS]) __attribute__((always_inline)) {
            const int gi = st * SG + ugroup;
#pragma unroll
            for (int i = 0; i < TPG; ++i) {
                const int tap = NARROW ? gi * TPG + i : a.div_tap(gi);
                const int k = tap * s.cw + uhalf * br.half + (NARROW ? 0 : WIDE * (gi - tap * a.per_tap));
                load_words(wres, (urow_words + k) * 4, v, i * WIDE);
            }
        };
        const int uwords = uhalf ? s.cw - br.half : br.half;   // words of a tap that this thread's half has
        auto put_w = [&](int st, const int (&v)[STEPS]) __attribute__((always_inline)) {
            const int gi = st * SG + ugroup;
            char* const to = stage + (st & 1) * STAGE + ugroup * (STEPS * CB * 1024) + (urow >> 5) * 1024 + (uhalf * 32 + (urow & 31)) * 16;
            const int tap0 = NARROW ? gi * TPG : a.div_tap(gi), k0 = NARROW ? 0 : WIDE * (gi - tap0 * a.per_tap);
            const int last = NARROW ? tap0 + TPG - 1 : tap0;
            // the common case in front: every word exists and is whole
            const bool whole = (last < a.taps) & (NARROW ? uwords == WIDE : k0 + WIDE <= uwords) & ((br.last_bits == ~0u) | (uhalf * br.half + k0 + WIDE < s.cw));
            if (whole) {
#pragma unroll
                for (int i = 0; i < STEPS; ++i) {
                    const v8i c = expand((uint32_t)v[i]);
                    *reinterpret_cast<v4i*>(to + i * (CB * 1024)) = v4i{c[0], c[1], c[2], c[3]};
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const int tap = NARROW ? tap0 + i / WIDE : tap0;
                const int k = k0 + (NARROW ? i % WIDE : i);  // within the half
                const bool real = tap < a.taps && k < uwords;
                const uint32_t bits = real ? (uhalf * br.half + k == s.cw - 1 ? br.last_bits : ~0u) : 0u;
                const uint32_t word = (uint32_t)v[i];
                v4i code;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const uint32_t sign = (bits << (3 - jj)) & 0x88888888u;
                    code[jj] = (int)(((word << (3 - jj)) & sign) | (sign >> 2));
                }
                *reinterpret_cast<v4i*>(to + i * (CB * 1024)) = code;
            }
        };
        // weight fragments of a K-step, read one step ahead
        struct Fragments { v4i f[CB]; };
        auto read_w = [&](const char* from, int ks, Fragments& fw) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) fw.f[cb] = *reinterpret_cast<const v4i*>(from + (ks * CB + cb) * 1024 + lane * 16);
        };
        auto step = [&](const Fragments& fw, const Inputs& c, int ks, bool first) __attribute__((always_inline)) {
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                const v8i fx = expand((uint32_t)(PAD_LATER ? c.x[pb][ks] | c.pad[pb][ks] : c.x[pb][ks]));
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const v8i w8 = {fw.f[cb][0], fw.f[cb][1], fw.f[cb][2], fw.f[cb][3], 0, 0, 0, 0};
                    const v16f from_zero = {};
                    acc[cb][pb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(LANE_CHANNEL ? fx : w8, LANE_CHANNEL ? w8 : fx, first ? from_zero : acc[cb][pb], 4, 4, 0, 0, 0, 0);
                }
            }
        };
        // branch mode: a completed tap's sums join the total, tot = fma(scale, y_t, tot) in the order t = 0, 1, ...
        __shared__ __align__(16) float scale_lds[BR ? MAX_BRANCHES : 1][TCH];
        auto fold = [&](int tap) __attribute__((always_inline)) {
            float sc[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) sc[cb] = scale_lds[tap][32 * cb + j];
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                if constexpr (PAD == PAD_NOTHING) {
                    // Lane i of a half holds the validity of pixel row_to_channel(i): of a lane's r-th one in bit 8 (r / 4) + r % 4, of
                    // the upper half's four bits further.  Both become a lane mask on the scalar unit (us, bit tests per lane and
                    // this: 3x3, 256 -> 256, 64 maps of 28 x 28, bits 27.6 and 25.5; 160 -> 160, 49 maps
                    // of 41 x 41, float 28.2 and 25.2; 96 -> 96, 30 maps of 30 x 30 8.9 and 8.0).
                    const int inside = (int)(uint32_t)__ballot((vmask[pb] >> tap) & 1u);
                    if (inside != -1) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int bit = 8 * (r >> 2) + (r & 3);
                            const uint64_t lo = (uint32_t)((inside << (31 - bit)) >> 31), hi = (uint32_t)((inside << (27 - bit)) >> 31);
                            const bool in = __builtin_amdgcn_inverse_ballot_w64(lo | hi << 32);
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) {
                                const float zn = __builtin_fmaf(sc[cb], acc[cb][pb][r], tot[cb][pb][r]);
                                tot[cb][pb][r] = in ? zn : tot[cb][pb][r];
                            }
                        }
                        continue;
                    }
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) tot[cb][pb][r] = __builtin_fmaf(sc[cb], acc[cb][pb][r], tot[cb][pb][r]);
            }
        };
        auto group = [&](int gi, const char* from, const Inputs& c) __attribute__((always_inline)) {
            Fragments fw[2];
            read_w(from, 0, fw[0]);
            const int tap0 = NARROW ? gi * TPG : a.div_tap(gi), g = NARROW ? 0 : gi - tap0 * a.per_tap;
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                const int tap = NARROW ? tap0 + k / WIDE : tap0;
                if (k + 1 < STEPS) read_w(from, k + 1, fw[(k + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                if (!NARROW || k < WIDE || tap < a.taps) {   // (a group of narrow taps may reach past the last one)
                    if (BR && (NARROW ? k % WIDE == 0 : k == 0 && g == 0)) step(fw[k & 1], c, k, true);
                    else step(fw[k & 1], c, k, false);
                    if constexpr (BR) {
                        if (NARROW ? k % WIDE == WIDE - 1 : k == STEPS - 1 && g == a.per_tap - 1) fold(tap);
                    }
                }
            }
        };
        int uw[STEPS];
        Inputs ring[2];
        fetch_w(0, uw);
        fetch_x(0, ring[0]);
        if constexpr (BR) {
            for (int i = t; i < a.taps * TCH; i += 64 * WP) {
                const int tp = i / TCH, cl = i - tp * TCH;
                scale_lds[tp][cl] = br.scale[(size_t)tp * s.c_out + (o0 + cl < s.c_out ? o0 + cl : s.c_out - 1)];
            }
        }
        // what a channel's sums start from: the bias, or what makes the sums' sign the output bit: sum - thr + 1/2
        __shared__ __align__(16) float start_lds[BR || SIGN_OUT ? TCH : 1];
        if constexpr (BR || SIGN_OUT) {
            if (t < TCH) {
                if constexpr (BR) start_lds[t] = __int_as_float(start);
                else start_lds[t] = 0.5f - (float)min(max(start, -s.k), s.k + 1);
            }
        }
        put_w(0, uw);
        fetch_w(1, uw);
        fetch_x(1, ring[1]);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                if constexpr (BR) {
                    const float bias = start_lds[32 * cb + j];
#pragma unroll
                    for (int r = 0; r < 16; ++r) tot[cb][pb][r] = bias;
                } else if constexpr (SIGN_OUT) {
#pragma unroll
                    for (int q = 0; q < 16; q += 4) {
                        const v4f v = *reinterpret_cast<const v4f*>(&start_lds[32 * cb + 16 * hsel + q]);
#pragma unroll
                        for (int k = 0; k < 4; ++k) acc[cb][pb][q + k] = v[k];
                    }
                }
            }
        static_assert(SG == 2 || SG == 4, "the input ring's two places in turn");
        // `part` groups of a stage; the first one's inputs lie in ring[0]
        auto walk = [&](int st, auto part) __attribute__((always_inline)) {
            const char* from = stage + (st & 1) * STAGE;
#pragma unroll
            for (int i = 0; i < decltype(part)::value; ++i) {
                const int gi = st * SG + i;
                group(gi, from + i * (STEPS * CB * 1024), ring[i & 1]);
                if constexpr (decltype(part)::value == SG) {
                    fetch_x(gi + 2, ring[i & 1]);
                    if (i == 0) {
                        put_w(st + 1, uw);
                        fetch_w(st + 2, uw);
                    }
                }
            }
            // only LDS is shared: loads in flight stay in flight
            if constexpr (decltype(part)::value == SG) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        };
        using C1 = std::integral_constant<int, 1>;
        using ALL = std::integral_constant<int, SG>;
        const int n_full = n_groups / SG;
        for (int st = 0; st < n_full; ++st) walk(st, ALL{});
        const int left = n_groups - n_full * SG;
        if (left == 1) walk(n_full, C1{});
        if constexpr (SG == 4) {
            using C2 = std::integral_constant<int, 2>;
            if (left == 2) walk(n_full, C2{});
            if (left == 3) {
                walk(n_full, C2{});
                fetch_x(n_full * SG + 2, ring[0]);
                group(n_full * SG + 2, stage + (n_full & 1) * STAGE + 2 * (STEPS * CB * 1024), ring[0]);
            }
        }
        if (left && !SIGN_OUT) __syncthreads();              // the epilogue's rows lie where the weights were
    } else if constexpr (!BR) {
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
                    multiply(ring[b], 4);
                    if (i + b + AHEAD < mine) fetch(wk + WK * (i + b + AHEAD), ring[b]);
                }
            }
        }
    } else {
        // (a wave of TAPS_APART takes the taps wk, wk + WK, ... and leaves their sums in LDS)
        // A tap's words are split between the lane halves and walked in groups of four words = four K-steps with one
        // 16-byte load per row; the last group is single words (branch_walk.h).  Every load is wave-uniform but for the
        // rows' offsets and their validity.
        // Positions that are zero on both sides count +1 each, a.z a tap.  Own operands: the accumulators start a tap at minus
        // that, so a completed tap costs one fma per element, tot = fma(scale, y_t, tot) in the order t = 0, 1, ... (the
        // chain is part of the interface), and one move to restart.  Taps apart: it is taken off where a tap's sums go to LDS.
        const BranchWalk walk = BranchWalk::make(s.cw);
        const int per_tap = walk.groups();
        const float start = (float)-a.z;                     // a.z: of one tap
        const auto pres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(br.pad_words), 0, PAD == PAD_OPERAND ? a.pad_bytes : 0, 0x00020000);
        auto fetch_group = [&](int tap, int g, Chunk& c) {
            const int k = walk.first(hsel, g);               // first word within the tap
            const int wo = tap * s.cw + k;
            const int xo = k + tap * a.tap_step + (s.ks == 3 ? tap * s.cw + ((tap >= 3) + (tap >= 6)) * a.row_jump : 0);
            if (g < walk.full) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    c.w[cb] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wres, (wrow[cb] + wo) * 4, 0, 0));
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const bool in = s.ks == 1 || ((vmask[pb] >> tap) & 1u);
                    c.x[pb] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xres, in ? (rbase[pb] + xo) * 4 : -16, 0, 0));
                    if constexpr (PAD == PAD_OPERAND) c.pad[pb] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(pres, in ? -16 : wo * 4, 0, 0));
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i >= walk.rest) break;
                    const bool real = walk.real(k + i);      // an odd count leaves the second half one word short
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
                        c.w[cb][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(wres, real ? (wrow[cb] + wo + i) * 4 : -4, 0, 0);
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) {
                        const bool in = s.ks == 1 || ((vmask[pb] >> tap) & 1u);
                        c.x[pb][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(xres, real && in ? (rbase[pb] + xo + i) * 4 : -4, 0, 0);
                        if constexpr (PAD == PAD_OPERAND) c.pad[pb][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(pres, real && !in ? (wo + i) * 4 : -4, 0, 0);
                    }
                }
            }
        };
        if constexpr (TAPS_APART) {
            for (int i = t; i < a.taps * TCH; i += 64 * WK) {
                const int tp = i / TCH, cl = i - tp * TCH;
                apart_scale[tp][cl] = br.scale[(size_t)tp * s.c_out + (o0 + cl < s.c_out ? o0 + cl : s.c_out - 1)];
            }
            if (t < 32) apart_mask[t] = vmask[0];
            constexpr int AHEAD = 4;
            Chunk ring[AHEAD];
            const int mine = (a.taps - wk + WK - 1) / WK * per_tap;     // groups of the wave's taps
            int f_tap = wk, f_g = 0, tap = wk, g = 0;                   // next to fetch, next to multiply
            auto fetch_next = [&](Chunk& c) {
                fetch_group(f_tap, f_g, c);
                const bool done = ++f_g == per_tap;
                f_g = done ? 0 : f_g;
                f_tap += done ? WK : 0;
            };
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
                if (i < mine) fetch_next(ring[i]);
            for (int i = 0; i < mine; i += AHEAD) {
#pragma unroll
                for (int b = 0; b < AHEAD; ++b) {
                    if (i + b < mine) {
                        multiply(ring[b], walk.steps(g));
                        if (i + b + AHEAD < mine) fetch_next(ring[b]);
                        if (++g == per_tap) {
#pragma unroll
                            for (int r = 0; r < 16; r += 4)
                                *reinterpret_cast<v4f*>(lds + tap * REGION + j * ROW + 16 * hsel + r) =
                                    v4f{acc[0][0][r] + start, acc[0][0][r + 1] + start, acc[0][0][r + 2] + start, acc[0][0][r + 3] + start};
#pragma unroll
                            for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;
                            g = 0;
                            tap += WK;
                        }
                    }
                }
            }
        } else {
            __shared__ __align__(16) float scale_lds[MAX_BRANCHES][TCH * WC];
            for (int i = t; i < a.taps * (TCH * WC); i += 64 * WC * WP) {
                const int tp = i / (TCH * WC), cl = i - tp * (TCH * WC);
                const int ch = o0 - TCH * wc + cl;
                scale_lds[tp][cl] = br.scale[(size_t)tp * s.c_out + (ch < s.c_out ? ch : s.c_out - 1)];
            }
            static_assert(!BR || WK > 1 || PAD == PAD_NONE, "calls whose taps leave the image take the other forms");
            Chunk cur, nxt;
            fetch_group(0, 0, cur);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                float b[16];
                const int ch = o0 + 32 * cb + 16 * hsel;         // the lane's 16 channels of the block
#pragma unroll
                for (int r = 0; r < 16; ++r) b[r] = br.bias ? br.bias[ch + r < s.c_out ? ch + r : s.c_out - 1] : 0.0f;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) { tot[cb][pb][r] = b[r]; acc[cb][pb][r] = start; }
            }
            __syncthreads();
            // (the groups' walk although this form is chosen for single words, one group a tap: without it the compiler takes four to ten
            // registers more, and a float tail's 106 instead of 96 leave a wave less on every SIMD: up to 14 % slower)
            for (int tap = 0; tap < a.taps; ++tap) {
                for (int g = 0; g < per_tap; ++g) {
                    const bool more = g + 1 < per_tap;
                    if (more || tap + 1 < a.taps) fetch_group(more ? tap : tap + 1, more ? g + 1 : 0, nxt);
                    multiply(cur, walk.steps(g));
                    cur = nxt;
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v4f sc = *reinterpret_cast<const v4f*>(&scale_lds[tap][TCH * wc + 32 * cb + 16 * hsel + 4 * q]);
#pragma unroll
                        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                tot[cb][pb][4 * q + k] = __builtin_fmaf(sc[k], acc[cb][pb][4 * q + k], tot[cb][pb][4 * q + k]);
                                acc[cb][pb][4 * q + k] = start;
                            }
                    }
            }
        }
    }

    // ---- epilogue.  A pixel's channels through LDS: lane (pixel j, half h) holds channels 16h .. 16h+15 of a block.
    float* region = lds + (wp * WC + wc) * WK * REGION;
    auto park = [&](float* dst, int pb, int row0) {
        if constexpr (LANE_CHANNEL) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) dst[(row0 + 16 * hsel + r) * ROW + 32 * cb + j] = tot[cb][pb][r];
            return;
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
            {
                const v16f& v = [&]() -> const v16f& { if constexpr (BR && !TAPS_APART) return tot[cb][pb]; else return acc[cb][pb]; }();
                *reinterpret_cast<v4f*>(dst + (row0 + j) * ROW + 32 * cb + 16 * hsel + r) = v4f{v[r], v[r + 1], v[r + 2], v[r + 3]};
            }
    };
    if constexpr (SIGN_OUT) {
        const auto bits_res = rows_of(out, s.cwo * 4);
        uint32_t half_word[CB][PB];                          // complements of the lane's 16 channels of a block
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                uint32_t wd = 0;
#pragma unroll
                for (int r = 15; r >= 0; --r) wd = __builtin_amdgcn_alignbit(wd, __float_as_uint(acc[cb][pb][r]), 31);
                half_word[cb][pb] = wd;
            }
        // lanes of the lower half end up with pixel block 0 (PB = 1: channel block 0), those of the upper half with 1
        auto put_word = [&](uint32_t lo, uint32_t hi, int px, int cb, bool mine) {
            const auto both = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
            const int left = s.c_out - (o0 + 32 * cb);       // channels of the word
            const uint32_t valid = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
            const uint32_t wd = ~(both[0] | (both[1] << 16)) & valid;
            const uint32_t at = (uint32_t)(px * s.cwo + (o0 >> 5) + cb) * 4u;
            __builtin_amdgcn_raw_buffer_store_b32((int)wd, bits_res, (int)(mine && left > 0 ? at : NOWHERE), 0, 0);
        };
        if constexpr (PB % 2 == 0) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int pb = 0; pb < PB; pb += 2) put_word(half_word[cb][pb], half_word[cb][pb + 1], 32 * (pb + hsel) + j, cb, true);
        } else {
            static_assert(PB == 1, "pixel blocks in pairs, or one");
#pragma unroll
            for (int cb = 0; cb + 1 < CB; cb += 2) put_word(half_word[cb][0], half_word[cb + 1][0], j, cb + hsel, true);
            if constexpr (CB % 2) put_word(half_word[CB - 1][0], half_word[CB - 1][0], j, CB - 1, hsel == 0);
        }
        return;
    }
    const float zf = (float)a.z;
    // per-channel parameters of the lane's four channels, through buffers: a channel past the end and a missing array
    // (no bytes) read as zero, without branches
    int th[4];
    float pg[4], pbi[4], pa[4], pc[4];
    auto load_params = [&](const void* p, auto& v) {
        const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, p ? s.c_out * 4 : 0, 0x00020000);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t q = __builtin_amdgcn_raw_buffer_load_b32(res, (c0 + k) * 4, 0, 0);
            v[k] = __builtin_bit_cast(std::decay_t<decltype(v[0])>, q);
        }
    };
    if constexpr (OUT == OUT_BITS && !BR) load_params(thr, th);
    if constexpr (MODULE) {
        if constexpr (!BR) {
            load_params(ep.scale, pg);
            load_params(ep.bias, pbi);
        }
        load_params(ep.slope, pa);
        load_params(ep.next_bias, pc);
        if (!ep.slope) {                                     // a missing slope is the slope 1 (1 * t is t)
#pragma unroll
            for (int k = 0; k < 4; ++k) pa[k] = 1.0f;
        }
    }
    const int nch = s.c_out - c0;                            // real channels from c0 on (may be <= 0)
    const int out_row = (OUT == OUT_I32 ? s.c_out : OUT == OUT_BITS ? s.cwo : 0) * 4;
    const auto out_res = rows_of(MODULE ? nullptr : out, out_row);
    const int r_row = s.c_out * ESZ, xn_row = s.cwo * 4;
    const auto r_res = rows_of(MODULE ? ep.r : nullptr, r_row);
    const auto xn_res = rows_of(MODULE ? ep.x_next : nullptr, xn_row);
    const uint32_t word_off = chan_ok && (lane & 7) == 0 ? (uint32_t)(c0 >> 5) * 4u : NOWHERE;
    // an identity row that starts again within the lane's channels, or that is shorter than a vector, is read channel by channel
    int id0 = 0, turn = 0;
    bool id_walk = false;
    if constexpr (MODULE) {
        if (!vec && ep.identity) {                           // (computed again: no register is kept through the K loop)
            int c = c0;
            asm volatile("" : "+v"(c));
            id0 = first_id(c);
            turn = turn_of(id0);
            id_walk = chan_ok && (ep.id_channels < 4 || (turn && nch > ep.id_channels - id0));
        }
    }
    // four sums (still with the constant z) of the tile's pixel px, channels c0 ..; every lane of the wave calls it
    auto emit = [&](v4f v, int px, int g) {
        uint32_t nib = 0;
        if constexpr (OUT == OUT_I32) {
            v4i q;
            if constexpr (BR) q = __builtin_bit_cast(v4i, v);
            else q = v4i{(int)(v[0] - zf), (int)(v[1] - zf), (int)(v[2] - zf), (int)(v[3] - zf)};
            const uint32_t at = (uint32_t)(px * out_row + c0 * 4);
            // whole groups of four, non-temporal (aux 2) where a block's 32 channels are whole cache lines; written that
            // way, partial lines cost twice (1x1, 128 -> 100 on 200 704 pixels 35 us against 16)
            const int off = (int)(chan_ok && nch >= 4 ? at : NOWHERE);
            if (s.c_out % 32 == 0) __builtin_amdgcn_raw_buffer_store_b128(q, out_res, off, 0, 2);
            else __builtin_amdgcn_raw_buffer_store_b128(q, out_res, off, 0, 0);
            if (s.c_out % 4 != 0) {                          // the row's last group
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    __builtin_amdgcn_raw_buffer_store_b32(q[k], out_res, (int)(chan_ok && nch < 4 && k < nch ? at + 4 * k : NOWHERE), 0, 0);
            }
            return;
        } else if constexpr (OUT == OUT_BITS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (BR) nib |= (uint32_t)(k < nch && v[k] >= 0.0f) << k;
                else nib |= (uint32_t)(k < nch && (int)(v[k] - zf) >= th[k]) << k;
            }
        } else {
            const int m = m0 + px;
            const bool ok = some && m < s.m;
            real4 id = ids[g];
            if (!vec && ep.identity) {
                if constexpr (HALF) id = __builtin_bit_cast(real4, __builtin_bit_cast(uint64_t, id) >> (16 * (turn & 3)));
                else {
                    if (turn & 1) id = real4{id[1], id[2], id[3], id[3]};
                    if (turn & 2) id = real4{id[2], id[3], id[3], id[3]};
                }
                if (id_walk && ok) {
                    const real_t* const idrow = static_cast<const real_t*>(ep.identity) + (int64_t)m * ep.id_channels;
                    int c = id0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        id[k] = idrow[c];
                        if (++c == ep.id_channels) c = 0;
                    }
                }
            }
            real4 st;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float val;
                if constexpr (BR) val = module_tail<REAL>(v[k], ep.identity != nullptr, (float)id[k], true, pa[k]);
                else val = module_value<REAL>(v[k] - zf, pg[k], pbi[k], ep.identity != nullptr, (float)id[k], true, pa[k]);
                nib |= (uint32_t)(k < nch && val + pc[k] >= 0.0f) << k;
                st[k] = (real_t)val;
            }
            if (vec) {
                const int at = (int)(chan_ok ? (uint32_t)(px * r_row + c0 * ESZ) : NOWHERE);
                if constexpr (HALF) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2i, st), r_res, at, 0, 0);
                else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, st), r_res, at, 0, 0);
            } else if (ok && ep.r) {
                real_t* rp = static_cast<real_t*>(ep.r) + (size_t)m * s.c_out + c0;
                if (nch >= 4) *reinterpret_cast<real4_any*>(rp) = st;
                else {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (k < nch) rp[k] = st[k];
                }
            }
        }
        // eight neighbouring lanes hold the 32 channels of one packed word
        uint32_t wd = nib << (4 * (lane & 7));
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x141, 0xF, 0xF, true);  // row_half_mirror
        __builtin_amdgcn_raw_buffer_store_b32((int)wd, MODULE ? xn_res : out_res, (int)(word_off + (uint32_t)(px * xn_row)), 0, 0);
    };
    if constexpr (TAPS_APART) {
        // tot = fma(scale, y_t, tot) in the order t = 0, 1, ..., every thread for its four outputs
        float first[4];
        load_params(br.bias, first);
        __syncthreads();
        static_assert(GROUPS == 1, "four outputs a thread");
        v4f sum = {first[0], first[1], first[2], first[3]};
        const uint32_t valid = PAD == PAD_NOTHING ? apart_mask[px0] : ~0u;
        for (int tap = 0; tap < a.taps; ++tap) {
            const v4f y = *reinterpret_cast<const v4f*>(lds + tap * REGION + px0 * ROW + 4 * (lt % CG));
            const v4f sc = *reinterpret_cast<const v4f*>(&apart_scale[tap][4 * (lt % CG)]);
            const bool in = (valid >> tap) & 1u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float zn = __builtin_fmaf(sc[k], y[k], sum[k]);
                sum[k] = in ? zn : sum[k];
            }
        }
        emit(sum, px0, 0);
    } else if constexpr (WK > 1) {
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
            emit(sum, px, g);
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
                emit(sum, 32 * pb + px, pb * (GROUPS / PB) + g);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

}  // namespace
}  // namespace bcnn
