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
};

}  // namespace attnw
