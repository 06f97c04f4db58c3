// Comparison results of a lane's values as the low bits of one word.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bcnn {

// Bit k = (v[k] >= 0): both zeros set it, NaN does not.
// Plain code: between a vector instruction that writes a lane mask and one that reads it gfx950 wants two wait states, which
// the compiler keeps by placing other instructions or s_nop there and cannot keep inside an asm statement.  A comparison
// and v_addc_co_u32 (bits = 2 * bits + mask) in groups of four, at that distance by hand, is three quarters of the
// instructions and at most 1.5 % faster: half, 64 channels, 32 maps of 112 x 112 22.5 against 22.7 us a module, the
// 128-channel level 45.4 against 46.0, eight other calls level.
template <int N>
__device__ __forceinline__ uint32_t sign_bits(const float (&v)[N])
{
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) bits |= (uint32_t)(v[k] >= 0.0f) << k;
    return bits;
}

// The same for results of an addition of which none is -0 (one summand was not -0): two instructions a value, no lane masks.
// The maximum turns NaN, and nothing else of that sign, into a negative number.
template <int N>
__device__ __forceinline__ uint32_t sign_bits_of_sums(const float (&v)[N])
{
    uint32_t negative = 0;
#pragma unroll
    for (int k = N - 1; k >= 0; --k)
        negative = __builtin_amdgcn_alignbit(negative, __float_as_uint(__builtin_fmaxf(v[k], -3.402823466e38f)), 31);
    return ~negative & ((1u << N) - 1u);
}

}  // namespace bcnn
