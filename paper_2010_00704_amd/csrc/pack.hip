// Sign-binarise + channel-pack kernels and the stand-alone threshold epilogue
// (BCNN paper, Section 4.2.1: sign before every binary convolution; Section
// 2.4: storage scales with the number of bits).  Both are pure streaming
// kernels: 4 bytes (or 2, or 1) read and 1 bit written per element, so HBM
// bandwidth is the only bound and the design goal is wide, coalesced reads
// with many of them in flight.
#include "bcnn_common.h"
#include "div_by.h"
#include "pack_plan.h"
#include "sign_bits.h"

#include <type_traits>
#include <utility>


namespace bcnn {
namespace {

__device__ __forceinline__ bool nonneg(float v) { return v >= 0.0f; }
__device__ __forceinline__ bool nonneg(_Float16 v) { return (float)v >= 0.0f; }
__device__ __forceinline__ bool nonneg(__bf16 v) { return (float)v >= 0.0f; }
__device__ __forceinline__ bool nonneg(int8_t v) { return v >= 0; }

// The bit of one element: sign of the value, or (BIAS) of value + bias[channel]
// with the sum rounded to float (Section 4.2.1: learnable bias, then sign).
template <bool BIAS, typename T>
__device__ __forceinline__ bool bit_of(T v, const float* __restrict__ bias, int64_t c)
{
    if constexpr (BIAS) return (float)v + bias[c] >= 0.0f;
    else return nonneg(v);
}

// Channel replication by bookkeeping (Section 4.2.2 of the paper: a building
// block that widens the network sees every real channel R times; no copy of the
// real map is made): output channel c reads source channel c mod src_channels,
// while the bias stays indexed by c.  REP == false: src_channels == channels.
template <bool REP>
__device__ __forceinline__ int64_t src_channel(int64_t c, int64_t src_channels)
{
    if constexpr (REP) return (int64_t)((uint32_t)c % (uint32_t)src_channels);   // both below 2^31
    else return c;
}

// Compile-time loop: f(std::integral_constant<int, 0>) ... f(<N-1>).
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// `old` with the wave-uniform `word` in lane LANE.  (The words come from a scalar AND, not from a comparison directly: a
// mask that a vector instruction wrote could not be read here at once.)
template <int LANE>
__device__ __forceinline__ uint32_t writelane(uint32_t word, uint32_t old)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(old) : "s"(word), "n"(LANE));
    return old;
}

// ---- [outer][C][inner] with inner >= 64: lanes run along `inner` ------------
// One thread owns one inner position and builds `cwg` consecutive words of that
// pixel.  For a fixed channel the 256 threads of a block read 256 consecutive
// elements; the 32 channel reads of a word are independent and all in flight.
// The block's words are staged through LDS so that each pixel's words leave
// in one contiguous run.  The channel words are split over blocks (cwg per
// block) until the launch has enough blocks to fill the chip.
constexpr int PACK_THREADS = 256;
constexpr int PACK_CW_CHUNK = 8;  // most words per block: 256*8*4 B = 8 KB LDS

template <typename T, bool BIAS, bool REP>
__global__ __launch_bounds__(PACK_THREADS) void pack_columns_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int64_t channels, int64_t src_channels,
    int64_t inner, int64_t cw_total, int cwg, int groups, uint32_t* __restrict__ dst)
{
    __shared__ uint32_t stage[PACK_THREADS * PACK_CW_CHUNK];
    const int64_t a = blockIdx.y / groups;
    const int64_t j0 = (int64_t)(blockIdx.y % groups) * cwg;
    const int64_t i0 = (int64_t)blockIdx.x * PACK_THREADS;
    const int tid = threadIdx.x;
    const int64_t i = i0 + tid;
    const bool live = i < inner;
    const int64_t icl = live ? i : inner - 1;
    const T* col = src + a * src_channels * inner + icl;
    const int rows_here = (int)((inner - i0 < PACK_THREADS) ? (inner - i0) : PACK_THREADS);
    const int jn = (int)((cw_total - j0 < cwg) ? (cw_total - j0) : cwg);

    for (int j = 0; j < jn; ++j) {
        const int64_t c0 = (j0 + j) * 32;
        uint32_t word = 0;
        if (c0 + 32 <= channels) {
            T v[32];
#pragma unroll
            for (int b = 0; b < 32; ++b)
                v[b] = __builtin_nontemporal_load(col + src_channel<REP>(c0 + b, src_channels) * inner);
#pragma unroll
            for (int b = 0; b < 32; ++b) word |= (uint32_t)bit_of<BIAS>(v[b], bias, c0 + b) << b;
        } else {
            for (int b = 0; c0 + b < channels; ++b)
                word |= (uint32_t)bit_of<BIAS>(col[src_channel<REP>(c0 + b, src_channels) * inner], bias, c0 + b) << b;
        }
        stage[tid * jn + j] = word;
    }
    __syncthreads();
    // rows_here*jn words: word t of the stage belongs to pixel t/jn, word t%jn of the group
    const int total = rows_here * jn;
    for (int t = tid; t < total; t += PACK_THREADS) {
        const int r = t / jn, j = t - r * jn;
        dst[(a * inner + i0 + r) * cw_total + j0 + j] = stage[t];
    }
}

// ---- fp32, inner a multiple of 4: four pixels per thread, whole rows per block ----
// The pixels of all images are numbered through (pixel a*inner + i is unit (a*inner + i) / 4, lane
// position i % 4), so every lane of every wave has work whatever `inner` is.  A block owns 64
// units = 256 consecutive output pixels and builds ALL packed words of them: wave w takes the
// words w, w+4, ... (up to PACK4_WORDS per block; more channels go to further blocks along y), 32
// independent 16-byte non-temporal loads per word in two batches of 16.  The words meet in LDS and leave
// as one contiguous run of 256 * words * 4 bytes: whole cache lines, written once.
constexpr int PACK4_WORDS = 32;   // packed words per pixel and block: 256 * 32 * 4 B = 32 KB of LDS

template <bool BIAS, bool REP>
__global__ __launch_bounds__(PACK_THREADS) void pack_units4_kernel(
    const float* __restrict__ src, const float* __restrict__ bias, int64_t channels, int64_t src_channels,
    int64_t inner, int64_t units, int64_t cw_total, uint32_t* __restrict__ dst)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    extern __shared__ uint32_t stage[];               // [256 pixels][jn words]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j0 = (int64_t)blockIdx.y * PACK4_WORDS;
    const int jn = (int)((cw_total - j0 < PACK4_WORDS) ? (cw_total - j0) : PACK4_WORDS);
    const int64_t u0 = (int64_t)blockIdx.x * 64;
    const int64_t u = u0 + lane < units ? u0 + lane : units - 1;       // clamped: duplicates, not stored
    const int64_t per_image = inner >> 2;
    const int64_t a = u / per_image;
    const float* col = src + a * src_channels * inner + 4 * (u - a * per_image);

    for (int j = wave; j < jn; j += 4) {
        const int64_t c0 = (j0 + j) * 32;
        uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
        if (c0 + 32 <= channels) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {      // two batches of 16 loads: 64 registers in flight
                f4 v[16];
#pragma unroll
                for (int b = 0; b < 16; ++b)
                    v[b] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(
                        col + src_channel<REP>(c0 + 16 * half + b, src_channels) * inner));
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    w0 |= (uint32_t)bit_of<BIAS>(v[b][0], bias, c0 + 16 * half + b) << (16 * half + b);
                    w1 |= (uint32_t)bit_of<BIAS>(v[b][1], bias, c0 + 16 * half + b) << (16 * half + b);
                    w2 |= (uint32_t)bit_of<BIAS>(v[b][2], bias, c0 + 16 * half + b) << (16 * half + b);
                    w3 |= (uint32_t)bit_of<BIAS>(v[b][3], bias, c0 + 16 * half + b) << (16 * half + b);
                }
            }
        } else {
            for (int b = 0; c0 + b < channels; ++b) {
                const f4 v = *reinterpret_cast<const f4*>(col + src_channel<REP>(c0 + b, src_channels) * inner);
                w0 |= (uint32_t)bit_of<BIAS>(v[0], bias, c0 + b) << b;
                w1 |= (uint32_t)bit_of<BIAS>(v[1], bias, c0 + b) << b;
                w2 |= (uint32_t)bit_of<BIAS>(v[2], bias, c0 + b) << b;
                w3 |= (uint32_t)bit_of<BIAS>(v[3], bias, c0 + b) << b;
            }
        }
        stage[(4 * lane + 0) * jn + j] = w0;
        stage[(4 * lane + 1) * jn + j] = w1;
        stage[(4 * lane + 2) * jn + j] = w2;
        stage[(4 * lane + 3) * jn + j] = w3;
    }
    __syncthreads();
    // pixel 4*u0 + r, word j0 + j; rows of a block that owns every word are contiguous in dst
    const int64_t live = units - u0 < 64 ? units - u0 : 64;
    const int total = (int)(4 * live) * jn;
    uint32_t* out = dst + 4 * u0 * cw_total + j0;
    if (jn == cw_total) {
        for (int t = threadIdx.x; t < total; t += PACK_THREADS) out[t] = stage[t];
    } else {
        for (int t = threadIdx.x; t < total; t += PACK_THREADS) {
            const int r = t / jn, j = t - r * jn;
            out[(int64_t)r * cw_total + j] = stage[t];
        }
    }
}

// ---- 1 < inner < 64 (7x7 feature maps, 3x3 filter taps): 2D thread tile ------
// IP = inner rounded up to a power of two; thread (i = t % IP, q = t / IP)
// reads element i of channel rows q, q+R, q+2R, ... (R = 256/IP rows per pass:
// consecutive rows are contiguous in memory, so a pass reads R*inner
// consecutive elements).  A thread ORs its rows' sign bits into partial words,
// the R partials of a pixel meet in LDS.  A block packs up to 8 words (256
// channels) of one `outer` index.
template <typename T, int IP, bool BIAS, bool REP>
__global__ __launch_bounds__(256) void pack_small_inner_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int64_t channels, int64_t src_channels,
    int inner, int64_t cw_total, int groups, uint32_t* __restrict__ dst)
{
    constexpr int R = 256 / IP;          // channel rows per pass
    constexpr int PASSES = 32 / R;       // passes per output word (R divides 32 as IP >= 8)
    constexpr int G = 8;                 // words per block
    __shared__ uint32_t part[G][R][IP];
    const int64_t a = blockIdx.x / groups;
    const int64_t j0 = (int64_t)(blockIdx.x % groups) * G;
    const int i = threadIdx.x % IP, q = threadIdx.x / IP;
    const bool live = i < inner;
    const T* base = src + a * src_channels * inner + (live ? i : 0);
    const int jn = (int)((cw_total - j0 < G) ? (cw_total - j0) : G);
    for (int j = 0; j < jn; ++j) {
        const int64_t c0 = (j0 + j) * 32;
        uint32_t word = 0;
        if (c0 + 32 <= channels) {
            T v[PASSES];
#pragma unroll
            for (int k = 0; k < PASSES; ++k)
                v[k] = __builtin_nontemporal_load(base + src_channel<REP>(c0 + q + R * k, src_channels) * inner);
#pragma unroll
            for (int k = 0; k < PASSES; ++k)
                word |= (uint32_t)bit_of<BIAS>(v[k], bias, c0 + q + R * k) << (q + R * k);
        } else {
            for (int k = 0; k < PASSES; ++k) {
                const int64_t c = c0 + q + R * k;
                if (c < channels)
                    word |= (uint32_t)bit_of<BIAS>(base[src_channel<REP>(c, src_channels) * inner], bias, c) << (q + R * k);
            }
        }
        part[j][q][i] = live ? word : 0u;
    }
    __syncthreads();
    // thread t -> (pixel t / jn, word t % jn): each pixel's words leave together
    for (int t = threadIdx.x; t < inner * jn; t += 256) {
        const int px = t / jn, j = t - px * jn;
        uint32_t word = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) word |= part[j][r][px];
        dst[(a * inner + px) * cw_total + j0 + j] = word;
    }
}

// What the kernels with lanes along the channels do with a lane's row of 4 NV dwords: the wave-wide comparison of each position, its
// two words into lane `position`, and out.  `byte`: where in its first dword a row starts; dst: the tile's first position.
template <typename T, int NV, bool BIAS, bool MIS>
__device__ __forceinline__ void ballot_and_store(const uint32_t (&d)[4 * NV + 1], uint32_t byte, float b, uint64_t valid, int lane,
                                                 int here, int g, int cw, uint32_t* dst)
{
    constexpr int ESZ = (int)sizeof(T);
    uint32_t lo = 0, hi = 0;
    static_for<4 * NV>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        const uint32_t w = MIS ? __builtin_amdgcn_alignbyte(d[k + 1], d[k], byte) : d[k];
        static_for<4 / ESZ>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            bool on;
            if constexpr (ESZ == 4) {
                const float v = __builtin_bit_cast(float, w);
                on = (BIAS ? v + b : v) >= 0.0f;
            } else if constexpr (ESZ == 1) {
                const int v = __builtin_amdgcn_sbfe((int)w, 8 * e, 8);
                on = BIAS ? (float)v + b >= 0.0f : v >= 0;
            } else {
                const T h = __builtin_bit_cast(T, (uint16_t)(w >> (16 * e)));
                on = (BIAS ? (float)h + b : (float)h) >= 0.0f;
            }
            const uint64_t mask = __ballot(on) & valid;
            lo = writelane<k * (4 / ESZ) + e>((uint32_t)mask, lo);
            hi = writelane<k * (4 / ESZ) + e>((uint32_t)(mask >> 32), hi);
        });
    });
    // lane p: the two words of position p
    const auto dres = __builtin_amdgcn_make_buffer_rsrc(dst, 0, here * cw * 4, 0x00020000);
    const uint32_t to = lane < here ? (uint32_t)(lane * cw + 2 * g) * 4u : 0x7FFFFF00u;
    if (2 * g + 1 < cw) {
        typedef int v2i __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(v2i{(int)lo, (int)hi}, dres, (int)to, 0, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32((int)lo, dres, (int)to, 0, 0);
    }
}

// ---- [outer][C][inner], lanes along the channels, ballot = packed words -------
// A wave owns 64 channels and P positions; lane l reads P consecutive positions of channel l as NV 16-byte vectors, all
// in flight together, so the wave-wide comparison of position p IS two packed words of that position.  They are
// collected in two registers, lane p holding position p, and leave as one 8-byte store per lane.  Five vector
// instructions for 64 elements; biases stay in one register.  A lane's vectors cover one or two cache lines of its row,
// which the wave's loads share in the first-level cache.  Rows start at any byte: vectors are loaded from the dword
// below and shifted into place (MIS).  Buffer accesses: channels past the end, and what a row's last vector
// reads past the image, are zero and not used.
template <typename T, int NV, bool BIAS, bool MIS>
__global__ __launch_bounds__(256) void pack_ballot_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int channels, int src_channels, int inner, int cw,
    int groups, int tiles, int tw_shift, int64_t blocks_per_image, uint32_t* __restrict__ dst)
{
    typedef int v4i __attribute__((ext_vector_type(4)));
    constexpr int ESZ = (int)sizeof(T);
    constexpr int PER = 16 / ESZ, P = NV * PER;
    static_assert(P <= 64, "a lane per position");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t a = (uint32_t)blockIdx.x / (uint32_t)blocks_per_image;
    const int at = (int)(blockIdx.x - (uint32_t)a * (uint32_t)blocks_per_image);
    int tile, g;
    if (!ballot_place(at, wave, tw_shift, groups, tiles, tile, g)) return;
    const int i0 = tile * P;
    const int c = 64 * g + lane;
    const bool live = c < channels;
    const int cs = src_channels == channels ? c : (int)((uint32_t)c % (uint32_t)src_channels);
    const int image = src_channels * inner * ESZ;            // bytes, a multiple of 4
    const auto sres = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(src) + a * image), 0, image, 0x00020000);
    const uint32_t byte = (uint32_t)(cs * inner + i0) * ESZ;
    const int off = live ? (int)(byte & ~3u) : 0x7FFFFF00;   // past every buffer
    uint32_t d[4 * NV + 1];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const v4i q = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(sres, off + 16 * k, 0, 0));
        d[4 * k] = q[0]; d[4 * k + 1] = q[1]; d[4 * k + 2] = q[2]; d[4 * k + 3] = q[3];
    }
    d[4 * NV] = 0;
    if constexpr (MIS) d[4 * NV] = __builtin_amdgcn_raw_buffer_load_b32(sres, off + 16 * NV, 0, 0);
    float b = 0.0f;
    if constexpr (BIAS) b = bias[live ? c : 0];
    ballot_and_store<T, NV, BIAS, MIS>(d, byte, b, __ballot(live), lane, inner - i0 < P ? inner - i0 : P, g, cw, dst + (a * inner + i0) * cw);
}

// The same for rows of at most 64 positions, which 64 channels hold in one piece of memory: the wave loads it lane by lane, 16 bytes
// next to 16 bytes, and turns it around in LDS of its own, so that no load touches 64 cache lines (each a cycle of the CU's address
// unit, eight times over for rows of 98 bytes).
// Memory bound where the launch is long enough.  us, calls in a row on buffers beyond the last-level cache, graph replays, against the kernels that ran these calls
// before: bfloat16 with bias, 1024 channels, 256 maps of 7 x 7 9.4 -> 8.4 (3.1 TB/s); half, 64 channels, 11 196 of 3 x 3 8.7 -> 5.2; float, 300 channels, 800 of
// 6 x 7 18.2 -> 10.4 (3.9 TB/s), 1024 channels, 128 of 7 x 7 9.4 -> 6.9, 1024 x 1024 x 3 x 3 weights 9.4 -> 9.1 (4.1 TB/s).
// Rows of whole vectors are read back as vectors, with a vector of padding in 256 bytes (VEC: 16 lanes reach all banks); others by
// dwords, whose odd or half strides share a bank between two lanes at most.  NV: vectors a row, rounded up.
// NT: loads that leave no lines behind (staged_streams).
template <typename T, int NV, bool BIAS, bool MIS, bool VEC, bool NT>
__global__ __launch_bounds__(256) void pack_staged_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int channels, int src_channels, int inner, int cw,
    int groups, int waves, DivBy div_groups, uint32_t* __restrict__ dst)
{
    typedef int v4i __attribute__((ext_vector_type(4)));
    constexpr int ESZ = (int)sizeof(T);
    static_assert(NV * 16 / ESZ <= 64, "a lane per position");
    constexpr int VECTORS = 64 * NV + (VEC ? 4 * NV : 1);    // (one past the last row: a dword more for a row that starts inside one)
    __shared__ v4i stage[4][VECTORS];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int at = (int)blockIdx.x * 4 + wave;
    if (at >= waves) return;
    const int a = div_groups(at), g = at - a * groups;
    const int c = 64 * g + lane;
    const bool live = c < channels;
    const int row = inner * ESZ;
    const int cs = src_channels == channels ? 64 * g : (int)((uint32_t)(64 * g) % (uint32_t)src_channels);
    const int size = (channels - 64 * g < 64 ? channels - 64 * g : 64) * row;
    const char* const from = reinterpret_cast<const char*>(src) + ((int64_t)a * src_channels + cs) * row;
    const auto sres = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(from), 0, size, 0x00020000);
    v4i v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(sres, 16 * lane + 1024 * k, 0, NT ? 2 : 0));
    float b = 0.0f;
    if constexpr (BIAS) b = bias[live ? c : 0];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = lane + 64 * k;
        stage[wave][VEC ? i + (i >> 4) : i] = v[k];
    }
    // (a wave's LDS accesses are carried out in order: only the compiler has to keep it)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t byte = (uint32_t)(lane * row);
    uint32_t d[4 * NV + 1];
    d[4 * NV] = 0;
    if constexpr (VEC) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i = (int)(byte >> 4) + k;
            const v4i q = stage[wave][i + (i >> 4)];
            d[4 * k] = q[0]; d[4 * k + 1] = q[1]; d[4 * k + 2] = q[2]; d[4 * k + 3] = q[3];
        }
    } else {
        const uint32_t* const words = reinterpret_cast<const uint32_t*>(&stage[wave][0]) + (byte >> 2);
#pragma unroll
        for (int k = 0; k < 4 * NV + (MIS ? 1 : 0); ++k) d[k] = words[k];
    }
    ballot_and_store<T, NV, BIAS, MIS>(d, byte, b, __ballot(live), lane, inner, g, cw, dst + (int64_t)a * inner * cw);
}

// ---- inner == 1 (channel-last rows): lanes run along the channels ----------
// One wave per (row, 64-channel group); the wave-wide ballot IS the two packed
// words.  Reads are perfectly coalesced.  ROWS rows are handled per wave so
// that several loads are in flight.
template <typename T, int ROWS, bool BIAS, bool REP>
__global__ __launch_bounds__(256) void pack_rows_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int64_t rows, int64_t channels,
    int64_t src_channels, int64_t cw_total, uint32_t* __restrict__ dst)
{
    const int lane = threadIdx.x & 63;
    const int64_t groups = (channels + 63) / 64;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t g = wave % groups;
    const int64_t r0 = (wave / groups) * ROWS;
    if (r0 >= rows) return;
    const int64_t c = g * 64 + lane;
    bool bit[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int64_t r = r0 + k;
        bit[k] = (r < rows && c < channels)
                     ? bit_of<BIAS>(src[r * src_channels + src_channel<REP>(c, src_channels)], bias, c) : false;
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const uint64_t mask = __ballot(bit[k]);
        const int64_t r = r0 + k;
        if (r < rows && lane < 2 && g * 2 + lane < cw_total)
            dst[r * cw_total + g * 2 + lane] = (uint32_t)(mask >> (32 * lane));
    }
}

// ---- inner == 1, source rows of whole dwords ----------------------------------
// A thread owns eight consecutive channels, 16 bytes of a 16-bit row, and four threads a packed word.  Its place
// along the row, and with it its eight biases, is the same for all its rows: the block's 256 threads are cut into
// runs of `per_row` threads, one run per row, and a thread takes one row per pass, all passes' loads in flight
// before the first is used.  Replicated channels read the source row again (channel c reads c mod src_channels).
// HBM bound.  Graph replays, us, against the kernels that ran these calls before, on rotating buffers beyond the last-level
// cache: half, 64 channels with bias, 312 500 rows 13.4 -> 9.2 (4.6 TB/s); replicated twice from 156 250 rows 30.5 -> 6.8;
// int8, 1000 channels, 20 000 rows 27.9 -> 7.0; float, 64 channels, 312 500 rows 18.7 -> 15.9 (5.2 TB/s).  From the
// cache: half, 128 channels, 100 352 rows 8.0 -> 4.2; four passes there: one is 5.0, two 4.4, eight 4.4, and on 300 rows
// all are level.
// Every access is a raw buffer access with a 32-bit offset from the block's first row: what does not exist (rows past
// the end, channels past the last row's end) reads as zero and stores nothing, without branches between the loads;
// the first form of this kernel, with predicated loads, took 8.4 us where this one takes 4.2 (both from the cache).
constexpr int LAST8_PASSES = 4;
// rows a whole number of dwords apart; the eight channels of a thread must not wrap inside a replica; 256 threads a row
bool last8_applies(size_t esz, const void* src, int64_t channels, int64_t src_channels)
{
    return (src_channels * (int64_t)esz) % 4 == 0 && (reinterpret_cast<uintptr_t>(src) & 3) == 0 && channels <= 2048 &&
           (src_channels == channels || src_channels % 8 == 0);
}

template <typename T, bool BIAS>
__global__ __launch_bounds__(256) void pack_last8_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int64_t rows, int channels, int src_channels,
    int cw, int per_row, int rows_per_pass, DivBy div_row, uint32_t* __restrict__ dst)
{
    typedef T t8 __attribute__((ext_vector_type(8)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int ESZ = (int)sizeof(T);
    constexpr int PASSES = LAST8_PASSES;
    const int t = threadIdx.x;
    const int r = div_row(t), q = t - r * per_row;
    const int c0 = 8 * q;
    const bool live = c0 < channels;                         // the row's last word may have lanes without channels
    const int left = channels - c0;
    const uint32_t valid = left >= 8 ? 0xFFu : left > 0 ? (1u << left) - 1u : 0u;
    const int64_t first = (int64_t)blockIdx.x * (rows_per_pass * PASSES);
    const int here = (int)(rows - first < rows_per_pass * PASSES ? rows - first : rows_per_pass * PASSES);
    const int src_row = src_channels * ESZ, dst_row = cw * 4;
    const auto sres = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src + first * src_channels), 0, here * src_row, 0x00020000);
    const auto dres = __builtin_amdgcn_make_buffer_rsrc(dst + first * cw, 0, here * dst_row, 0x00020000);
    const auto bres = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(bias), 0, BIAS ? channels * 4 : 0, 0x00020000);
    constexpr uint32_t NOWHERE = 0x7FFFFF00u;                // past every buffer
    const bool mine = r < rows_per_pass;
    const int cs = src_channels == channels ? c0 : (int)((uint32_t)c0 % (uint32_t)src_channels);
    const uint32_t from = mine && live ? (uint32_t)(r * src_row + cs * ESZ) : NOWHERE;
    const uint32_t to = mine && (q & 3) == 0 ? (uint32_t)(r * dst_row + q) : NOWHERE;      // word q / 4
    t8 v[PASSES];
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int off = (int)(from + (uint32_t)(k * rows_per_pass * src_row));
        if constexpr (ESZ == 2) {
            v[k] = __builtin_bit_cast(t8, __builtin_amdgcn_raw_buffer_load_b128(sres, off, 0, 0));
        } else if constexpr (ESZ == 1) {
            v[k] = __builtin_bit_cast(t8, __builtin_amdgcn_raw_buffer_load_b64(sres, off, 0, 0));
        } else {
            const f4 lo = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(sres, off, 0, 0));
            const f4 hi = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(sres, off + 16, 0, 0));
            v[k] = t8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    }
    float b[8];
#pragma unroll
    for (int h = 0; h < 8; h += 4) {
        f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (BIAS) w = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(bres, (c0 + h) * 4, 0, 0));
        b[h] = w[0]; b[h + 1] = w[1]; b[h + 2] = w[2]; b[h + 3] = w[3];
    }
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        uint32_t bits = 0;
        if constexpr (ESZ == 1 && !BIAS) {
#pragma unroll
            for (int i = 7; i >= 0; --i) bits = 2 * bits + (uint32_t)(v[k][i] >= 0);
        } else {
            float f[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] = BIAS ? (float)v[k][i] + b[i] : (float)v[k][i];
            bits = sign_bits(f);
        }
        uint32_t wd = (bits & valid) << (8 * (q & 3));
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
        __builtin_amdgcn_raw_buffer_store_b32((int)wd, dres, (int)(to + (uint32_t)(k * rows_per_pass * dst_row)), 0, 0);
    }
}

// The same for rows at any address: loads of eight elements at the elements' own alignment.  A thread whose eight channels reach past its
// source row loads the row's last eight instead, `turn` elements back, and shifts its bits; where channels are replicated, what wraps
// comes from the row's first eight (WRAP).  Every load is inside the tensor, without branches: rows past the end read the last one again.
// Kernel times, us, against the lanes along the channels (waves full of predicated two-byte loads, bound by their number): bfloat16
// with bias, 291 channels, 29 624 rows 10.7 -> 4.8; replicated twice from 7406 rows 7.6 -> 5.3; half, 493 channels, 15 548 rows
// 7.8 -> 4.4; 301 channels twice from 20 000 rows 17.6 -> 8.2.
template <typename T, bool BIAS, bool WRAP>
__global__ __launch_bounds__(256) void pack_ragged8_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int64_t rows, int channels, int src_channels,
    int cw, int per_row, int rows_per_pass, DivBy div_row, uint32_t* __restrict__ dst)
{
    typedef T t8 __attribute__((ext_vector_type(8)));
    typedef T t8_any __attribute__((ext_vector_type(8), aligned(sizeof(T))));
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int PASSES = LAST8_PASSES;
    const int t = threadIdx.x;
    const int r = div_row(t), q = t - r * per_row;
    const int c0 = 8 * q;
    const int left = channels - c0;
    const uint32_t valid = left >= 8 ? 0xFFu : left > 0 ? (1u << left) - 1u : 0u;
    const int64_t first = (int64_t)blockIdx.x * (rows_per_pass * PASSES);
    const int here = (int)(rows - first < rows_per_pass * PASSES ? rows - first : rows_per_pass * PASSES);
    const int dst_row = cw * 4;
    const auto dres = __builtin_amdgcn_make_buffer_rsrc(dst + first * cw, 0, here * dst_row, 0x00020000);
    const auto bres = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(bias), 0, BIAS ? channels * 4 : 0, 0x00020000);
    constexpr uint32_t NOWHERE = 0x7FFFFF00u;                // past every buffer
    const bool mine = r < rows_per_pass;
    const uint32_t to = mine && (q & 3) == 0 ? (uint32_t)(r * dst_row + q) : NOWHERE;      // word q / 4
    const int cs = WRAP ? (int)((uint32_t)c0 % (uint32_t)src_channels) : c0;
    const int from = cs < src_channels - 8 ? cs : src_channels - 8;
    const int turn = cs - from;                              // 8 and more: a thread without channels
    const T* const block = src + first * src_channels;
    t8 v[PASSES], u[WRAP ? PASSES : 1];
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int row = r + k * rows_per_pass;
        const T* const at = block + (row < here ? row : here - 1) * src_channels;
        v[k] = *reinterpret_cast<const t8_any*>(at + from);
        if constexpr (WRAP) u[k] = *reinterpret_cast<const t8_any*>(at);
    }
    auto biases = [&](int c, float (&b)[8]) {                // (a channel that does not exist reads as zero)
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (BIAS) w = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(bres, (c + h) * 4, 0, 0));
            b[h] = w[0]; b[h + 1] = w[1]; b[h + 2] = w[2]; b[h + 3] = w[3];
        }
    };
    auto bits_of = [&](const t8& e, const float (&b)[8]) -> uint32_t {
        float f[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = BIAS ? (float)e[i] + b[i] : (float)e[i];
        return sign_bits(f);
    };
    float bv[8], bu[8];
    biases(c0 - turn, bv);
    if constexpr (WRAP) biases(c0 + 8 - turn, bu);
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        uint32_t bits = turn < 8 ? bits_of(v[k], bv) >> turn : 0u;
        if constexpr (WRAP) bits |= turn < 8 ? bits_of(u[k], bu) << (8 - turn) : 0u;
        uint32_t wd = (bits & valid) << (8 * (q & 3));
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
        wd |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wd, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
        __builtin_amdgcn_raw_buffer_store_b32((int)wd, dres, (int)(to + (uint32_t)(k * rows_per_pass * dst_row)), 0, 0);
    }
}

// ---- anything else (small inner, e.g. 3x3 filter taps): one thread per word --
template <typename T, bool BIAS, bool REP>
__global__ __launch_bounds__(256) void pack_generic_kernel(
    const T* __restrict__ src, const float* __restrict__ bias, int64_t outer, int64_t channels,
    int64_t src_channels, int64_t inner, int64_t cw_total, uint32_t* __restrict__ dst)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= outer * inner * cw_total) return;
    const int64_t j = t % cw_total;
    const int64_t i = (t / cw_total) % inner;
    const int64_t a = t / (cw_total * inner);
    uint32_t word = 0;
    for (int b = 0; b < 32; ++b) {
        const int64_t c = j * 32 + b;
        if (c < channels)
            word |= (uint32_t)bit_of<BIAS>(src[(a * src_channels + src_channel<REP>(c, src_channels)) * inner + i],
                                           bias, c) << b;
    }
    dst[t] = word;
}

template <typename T, bool BIAS, bool REP>
hipError_t pack_dispatch(const T* src, const float* bias, int64_t outer, int64_t channels,
                         int64_t src_channels, int64_t inner, uint32_t* dst, hipStream_t stream)
{
    const int64_t cw = (channels + 31) / 32;
    if (inner == 1 && last8_applies(sizeof(T), src, channels, src_channels)) {
        const int per_row = (int)cw * 4, rows_per_pass = 256 / per_row, per_block = rows_per_pass * LAST8_PASSES;
        hipLaunchKernelGGL((pack_last8_kernel<T, BIAS>), dim3((unsigned)((outer + per_block - 1) / per_block)), dim3(256), 0, stream,
                           src, bias, outer, (int)channels, (int)src_channels, (int)cw, per_row, rows_per_pass,
                           DivBy::make(per_row), dst);
    } else if (inner == 1 && ragged8_applies(outer, channels, src_channels)) {
        const int per_row = (int)cw * 4, rows_per_pass = 256 / per_row, per_block = rows_per_pass * LAST8_PASSES;
        hipLaunchKernelGGL((pack_ragged8_kernel<T, BIAS, REP>), dim3((unsigned)((outer + per_block - 1) / per_block)), dim3(256), 0, stream,
                           src, bias, outer, (int)channels, (int)src_channels, (int)cw, per_row, rows_per_pass,
                           DivBy::make(per_row), dst);
    } else if (inner == 1 && (outer + 7) / 8 * ((channels + 63) / 64) <= 4 * MAX_BLOCKS_256) {
        constexpr int ROWS = 8;
        const int64_t groups = (channels + 63) / 64;
        const int64_t waves = ((outer + ROWS - 1) / ROWS) * groups;
        const int64_t blocks = (waves + 3) / 4;
        hipLaunchKernelGGL((pack_rows_kernel<T, ROWS, BIAS, REP>), dim3((unsigned)blocks), dim3(256), 0, stream,
                           src, bias, outer, channels, src_channels, cw, dst);
    } else if (const int nv = staged_vectors((int)sizeof(T), reinterpret_cast<uintptr_t>(src), outer, channels, src_channels, inner); nv) {
        const int64_t groups = (channels + 63) / 64, waves = outer * groups;
        const int64_t row = inner * (int64_t)sizeof(T);
        auto go = [&](auto size) {
            constexpr int N = decltype(size)::value, ESZ = (int)sizeof(T);
            if constexpr (N * 16 / ESZ <= 64) {
                auto launch = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, stream, src, bias, (int)channels, (int)src_channels,
                                       (int)inner, (int)cw, (int)groups, (int)waves, DivBy::make((int)groups), dst);
                };
                auto of = [&](auto nt) {
                    constexpr bool NT = decltype(nt)::value;
                    if (row % 16 == 0) launch(pack_staged_kernel<T, N, BIAS, false, true, NT>);
                    else if (row % 4 == 0) launch(pack_staged_kernel<T, N, BIAS, false, false, NT>);
                    else launch(pack_staged_kernel<T, N, BIAS, ESZ < 4, false, NT>);
                };
                if (staged_streams(ESZ, row, outer * src_channels * row)) of(std::true_type{});
                else of(std::false_type{});
            }
        };
        switch (nv) {
            case 2: go(std::integral_constant<int, 2>{}); break;
            case 3: go(std::integral_constant<int, 3>{}); break;
            case 4: go(std::integral_constant<int, 4>{}); break;
            case 5: go(std::integral_constant<int, 5>{}); break;
            case 6: go(std::integral_constant<int, 6>{}); break;
            case 7: go(std::integral_constant<int, 7>{}); break;
            case 8: go(std::integral_constant<int, 8>{}); break;
            case 10: go(std::integral_constant<int, 10>{}); break;
            default: go(std::integral_constant<int, 13>{}); break;
        }
    } else if (const BallotPlan plan = plan_ballot((int)sizeof(T), reinterpret_cast<uintptr_t>(src), outer, channels, src_channels, inner); plan.nv) {
        const bool mis = (inner * (int64_t)sizeof(T)) % 4 != 0;
        auto go = [&](auto nv) {
            constexpr int N = decltype(nv)::value;
            if constexpr (N * 16 / (int)sizeof(T) <= 64) {
                const dim3 grid((unsigned)(plan.blocks_per_image * outer));
                auto launch = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, src, bias, (int)channels, (int)src_channels, (int)inner,
                                       (int)cw, plan.groups, plan.tiles, plan.tw_shift, plan.blocks_per_image, dst);
                };
                if (mis) launch(pack_ballot_kernel<T, N, BIAS, true>);
                else launch(pack_ballot_kernel<T, N, BIAS, false>);
            }
        };
        switch (plan.nv) {
            case 1: go(std::integral_constant<int, 1>{}); break;
            case 2: go(std::integral_constant<int, 2>{}); break;
            case 4: go(std::integral_constant<int, 4>{}); break;
            default: go(std::integral_constant<int, 8>{}); break;
        }
    } else if (std::is_same<T, float>::value && inner >= 64 && inner % 4 == 0 && outer * (inner / 4) >= 64 * 128 &&
               (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
        // (from 128 blocks on; smaller inputs spread better over the chip with one pixel per thread)
        const int64_t units = outer * (inner / 4);
        const int64_t bx = (units + 63) / 64;
        const int64_t by = (cw + PACK4_WORDS - 1) / PACK4_WORDS;
        if (bx > 0x7FFFFFFF || by > 65535) goto generic;
        const int words = (int)(cw < PACK4_WORDS ? cw : PACK4_WORDS);
        hipLaunchKernelGGL((pack_units4_kernel<BIAS, REP>), dim3((unsigned)bx, (unsigned)by), dim3(PACK_THREADS),
                           (size_t)256 * words * 4, stream, reinterpret_cast<const float*>(src), bias, channels,
                           src_channels, inner, units, cw, dst);
    } else if (inner >= 64) {
        const int64_t bx = (inner + PACK_THREADS - 1) / PACK_THREADS;
        // words per block: as many as possible (up to 8) while two blocks per CU remain
        int cwg = PACK_CW_CHUNK;
        while (cwg > 1 && bx * outer * ((cw + cwg - 1) / cwg) < 512) cwg >>= 1;
        const int64_t groups = (cw + cwg - 1) / cwg;
        if (outer * groups > 65535) goto generic;
        hipLaunchKernelGGL((pack_columns_kernel<T, BIAS, REP>), dim3((unsigned)bx, (unsigned)(outer * groups)),
                           dim3(PACK_THREADS), 0, stream, src, bias, channels, src_channels, inner, cw, cwg,
                           (int)groups, dst);
    } else if (inner >= 5) {
        const int64_t groups = (cw + 7) / 8;
        const int64_t blocks = outer * groups;
        if (blocks > MAX_BLOCKS_256) goto generic;
        if (inner > 32)
            hipLaunchKernelGGL((pack_small_inner_kernel<T, 64, BIAS, REP>), dim3((unsigned)blocks), dim3(256), 0, stream,
                               src, bias, channels, src_channels, (int)inner, cw, (int)groups, dst);
        else if (inner > 16)
            hipLaunchKernelGGL((pack_small_inner_kernel<T, 32, BIAS, REP>), dim3((unsigned)blocks), dim3(256), 0, stream,
                               src, bias, channels, src_channels, (int)inner, cw, (int)groups, dst);
        else if (inner > 8)
            hipLaunchKernelGGL((pack_small_inner_kernel<T, 16, BIAS, REP>), dim3((unsigned)blocks), dim3(256), 0, stream,
                               src, bias, channels, src_channels, (int)inner, cw, (int)groups, dst);
        else
            hipLaunchKernelGGL((pack_small_inner_kernel<T, 8, BIAS, REP>), dim3((unsigned)blocks), dim3(256), 0, stream,
                               src, bias, channels, src_channels, (int)inner, cw, (int)groups, dst);
    } else {
    generic:
        const int64_t total = outer * inner * cw;
        const int64_t blocks = (total + 255) / 256;
        hipLaunchKernelGGL((pack_generic_kernel<T, BIAS, REP>), dim3((unsigned)blocks), dim3(256), 0, stream,
                           src, bias, outer, channels, src_channels, inner, cw, dst);
    }
    return hipGetLastError();
}

// ---- stand-alone epilogue: int32 sums [rows][c_out] -> packed bits ---------
template <int ROWS>
__global__ __launch_bounds__(256) void threshold_sign_pack_kernel(
    const int32_t* __restrict__ y, const int32_t* __restrict__ thr, int64_t rows, int64_t c_out,
    int64_t cwo, uint32_t* __restrict__ yp)
{
    const int lane = threadIdx.x & 63;
    const int64_t groups = (c_out + 63) / 64;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t g = wave % groups;
    const int64_t r0 = (wave / groups) * ROWS;
    if (r0 >= rows) return;
    const int64_t c = g * 64 + lane;
    const bool cl = c < c_out;
    const int32_t t = cl ? thr[c] : 0;
    int32_t v[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int64_t r = r0 + k;
        v[k] = (r < rows && cl) ? __builtin_nontemporal_load(y + r * c_out + c) : 0;
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const uint64_t mask = __ballot(cl && v[k] >= t);
        const int64_t r = r0 + k;
        if (r < rows && lane < 2 && g * 2 + lane < cwo)
            yp[r * cwo + g * 2 + lane] = (uint32_t)(mask >> (32 * lane));
    }
}

// The same for c_out a multiple of 32 and 16-byte aligned sums: the tensor is
// a flat stream of 16-byte units (4 channels of one row), a lane takes UNROLL
// units per round with non-temporal 16-byte loads, eight neighbouring lanes
// hold the 32 channels of one output word and combine their nibbles with three
// DPP exchanges.
template <int UNROLL>
__global__ __launch_bounds__(256) void threshold_sign_pack4_kernel(
    const int32_t* __restrict__ y, const int32_t* __restrict__ thr, int64_t units, int c_out,
    uint32_t* __restrict__ yp)
{
    typedef int i4 __attribute__((ext_vector_type(4)));
    const int lane8 = threadIdx.x & 7;
    const int64_t stride = (int64_t)gridDim.x * 256;
    int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // channel of this lane's unit, kept up to date by adding the stride modulo c_out
    int c = (int)((u * 4) % c_out);
    const int cstep = (int)((stride * 4) % c_out);
    for (; u < units; u += stride * UNROLL) {
        i4 v[UNROLL], t[UNROLL];
        int cc = c;
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            const int64_t uk = u + stride * k;
            const bool ok = uk < units;
            v[k] = ok ? __builtin_nontemporal_load(reinterpret_cast<const i4*>(y) + uk) : i4{0, 0, 0, 0};
            t[k] = *reinterpret_cast<const i4*>(thr + cc);
            cc += cstep; cc -= cc >= c_out ? c_out : 0;
        }
        c = cc;
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            const int64_t uk = u + stride * k;
            uint32_t w = ((uint32_t)(v[k][0] >= t[k][0]) | ((uint32_t)(v[k][1] >= t[k][1]) << 1) |
                          ((uint32_t)(v[k][2] >= t[k][2]) << 2) | ((uint32_t)(v[k][3] >= t[k][3]) << 3))
                         << (4 * lane8);
            // OR over the 8 lanes of the word: neighbours, pairs, then the other quad
            w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
            w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
            w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x141, 0xF, 0xF, true);  // row_half_mirror
            if (lane8 == 0 && uk < units) yp[uk >> 3] = w;
        }
    }
}

}  // namespace

template <typename T>
hipError_t pack_typed(const void* src, const float* bias, int64_t outer, int64_t channels,
                      int64_t src_channels, int64_t inner, uint32_t* dst, hipStream_t stream)
{
    const T* p = static_cast<const T*>(src);
    if (src_channels != channels)   // replication always comes with a bias
        return pack_dispatch<T, true, true>(p, bias, outer, channels, src_channels, inner, dst, stream);
    if (bias) return pack_dispatch<T, true, false>(p, bias, outer, channels, channels, inner, dst, stream);
    return pack_dispatch<T, false, false>(p, nullptr, outer, channels, channels, inner, dst, stream);
}

hipError_t launch_pack(const void* src, int dtype, const float* bias, int64_t outer, int64_t channels,
                       int64_t src_channels, int64_t inner, uint32_t* dst, hipStream_t stream)
{
    // A channel-last source (inner = 1) of more channels than pack_last8_kernel takes, with whole 16-byte (float) /
    // 8-byte (half) groups of four channels, is the pooling kernel's case with a 1 x 1 window: a lane takes four
    // channels of a row, eight lanes make a packed word.  Twice to three times the rate of the
    // lanes-along-channels kernel.
    if (inner == 1 && src_channels == channels && channels > 2048 && (dtype == 0 || dtype == 1) && channels % 4 == 0 &&
        outer * 8 * ((channels + 31) / 32) <= 0x7FFFFFFF &&
        (reinterpret_cast<uintptr_t>(src) % (dtype == 0 ? 16 : 8)) == 0 &&
        (reinterpret_cast<uintptr_t>(bias) % 16) == 0)
        return launch_avgpool_pack(src, dtype == 1 ? REAL_F16 : REAL_F32, (int)outer, 1, 1, (int)channels, 1, bias, nullptr,
                                   dst, stream);
    switch (dtype) {
        case 0: return pack_typed<float>(src, bias, outer, channels, src_channels, inner, dst, stream);
        case 1: return pack_typed<_Float16>(src, bias, outer, channels, src_channels, inner, dst, stream);
        case 2: return pack_typed<int8_t>(src, bias, outer, channels, src_channels, inner, dst, stream);
        case 3: return pack_typed<__bf16>(src, bias, outer, channels, src_channels, inner, dst, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_threshold_sign_pack(const int32_t* y, const int32_t* thr, int64_t rows,
                                      int64_t c_out, uint32_t* y_packed, hipStream_t stream)
{
    if (c_out % 32 == 0 && ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(thr)) & 15) == 0) {
        constexpr int UNROLL = 4;
        const int64_t units = rows * (c_out / 4);
        // one round per block: blocks that finish early make room for the rest, so the tail stays short
        // (the kernel's loop only matters beyond 2^31 - 1 blocks, which the row limit excludes)
        const int64_t blocks = (units + 256 * UNROLL - 1) / (256 * UNROLL);
        hipLaunchKernelGGL((threshold_sign_pack4_kernel<UNROLL>), dim3((unsigned)blocks), dim3(256), 0,
                           stream, y, thr, units, (int)c_out, y_packed);
        return hipGetLastError();
    }
    constexpr int ROWS = 8;
    const int64_t groups = (c_out + 63) / 64;
    const int64_t waves = ((rows + ROWS - 1) / ROWS) * groups;
    const int64_t blocks = (waves + 3) / 4;
    hipLaunchKernelGGL((threshold_sign_pack_kernel<ROWS>), dim3((unsigned)blocks), dim3(256), 0,
                       stream, y, thr, rows, c_out, (c_out + 31) / 32, y_packed);
    return hipGetLastError();
}

}  // namespace bcnn
