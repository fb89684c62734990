// Shared by the attention kernels: the exchange between the two half-waves of a query, and the chunk swizzles of those that keep
// K and V in LDS as they lie in memory.
#pragma once

#include "qk_common.h"

namespace attnw {

// value of the other half-wave's lane (l ^ 32) combined with the own one
__device__ __forceinline__ float half_wave_max(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
#else
    return x;
#endif
}
__device__ __forceinline__ float half_wave_sum(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
#else
    return x;
#endif
}

// the same over the four lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ __forceinline__ float quarter_wave_max(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return half_wave_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
#else
    return x;
#endif
}
__device__ __forceinline__ float quarter_wave_sum(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return half_wave_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
#else
    return x;
#endif
}

// The exponent that a query's weights are taken against follows its running maximum only when the 16 weights that a lane makes of
// a sub-tile sum to more than this: a look at the sum that is needed anyway instead of at the maximum of the scores in front of the
// exponentials (7 v_max3, an exchange between the half-waves and a branch per 32 keys, all of it in the way).  No weight is larger: fp32
// sums and bf16 operands have the same relative precision at every magnitude.  The exponent then moves to the largest weight, which comes to
// be 1 (and has no rounding as a bf16 operand: in sharp rows most of the error).  Sums above 2^100 have their weights made again from the scores:
// the factor between the exponents stays a normal number (v_exp_f32 gives 0 below 2^-126, for the largest weight too).
constexpr float kFarSum = 256.0f, kOverflow = 0x1p100f;

// the largest of a lane's 16 scores of a sub-tile
__device__ __forceinline__ float max16(const f32x16& s)
{
    float m = max3(s[0], s[1], s[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) m = max3(m, s[r], s[r + 1]);
    return fmaxf(m, s[15]);
}

// By so much the exponent moves: log2 of the largest of a query's weights, 16 in each of two lanes, where that is above 0.
__device__ __forceinline__ float far_exponent(const float (&p)[16])
{
    float m = max3(p[0], p[1], p[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) m = max3(m, p[r], p[r + 1]);
    return fmaxf(fast_log2(half_wave_max(fmaxf(m, p[15]))), 0.0f);
}

// Rows of DVB x 64 bytes on chip (DVB x 32 bf16 columns), 16-byte chunks swizzled within the row (involutions that stay
// inside it).  A K fragment read takes one chunk of 32 consecutive rows: 16 rows hit 16 different chunk positions modulo
// 256 bytes.  The transposing read of V takes 64 bytes of four consecutive rows: those lie in different quarters of 256.
template <int DVB> struct RowLayout {
    static constexpr int KPERIOD = DVB % 4 == 0 ? 8 : DVB % 4 == 2 ? 4 : 2;   // 32-byte groups after which the swizzled bits repeat
    static constexpr int VPERIOD = DVB % 4 == 0 ? 4 : DVB % 4 == 2 ? 2 : 1;   // the same in 64-byte column blocks
    static __device__ __forceinline__ int k_chunk(int key)
    {
        return DVB % 4 == 0 ? key & 15 : DVB % 4 == 2 ? (key >> 1) & 7 : (key >> 2) & 3;
    }
    static __device__ __forceinline__ int v_block(int key) { return DVB % 4 == 0 ? key & 3 : DVB % 4 == 2 ? (key >> 1) & 1 : 0; }
    // Blocks of 16 columns (16 x 16 matrix instruction): half of a wave reads 32 bytes of eight consecutive rows.
    static constexpr int V16PERIOD = DVB % 4 == 0 ? 8 : DVB % 4 == 2 ? 4 : 2;
    static __device__ __forceinline__ int v16_block(int key) { return DVB % 4 == 0 ? key & 7 : DVB % 4 == 2 ? (key >> 1) & 3 : (key >> 2) & 1; }
};

}  // namespace attnw
