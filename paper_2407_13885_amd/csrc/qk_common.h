// Building blocks shared by the Q K^T kernels: MFMA wrappers per element type,
// direct global-to-LDS transfers, wait-count helpers and compile-time loop helpers.
#pragma once

#include "device_utils.h"

namespace attnw {

typedef const void __attribute__((address_space(1)))* global_cptr;
typedef void __attribute__((address_space(3)))* lds_ptr;

template <typename T> struct Mma;

// bf16: one 16-byte chunk holds 8 consecutive d-elements; lanes 0..31 carry chunk
// 2g, lanes 32..63 chunk 2g+1 of a 32-byte group = the k = 16 of one instruction.
template <> struct Mma<uint16_t> {
    static __device__ __forceinline__ void run(f32x16& acc, const u32x4& a, const u32x4& b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                      acc, 0, 0, 0);
    }
    static constexpr uint32_t kSignMask = 0x80008000u;
};

// fp32: a chunk holds 4 floats; the 32-byte group (8 floats) is contracted by four
// 32x32x2 instructions, instruction i taking floats i (lanes 0..31) and 4+i (lanes
// 32..63).  Any pairing is valid as long as both operands use the same one.
template <> struct Mma<float> {
    static __device__ __forceinline__ void run(f32x16& acc, const u32x4& a, const u32x4& b)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[i]), __uint_as_float(b[i]), acc, 0, 0, 0);
    }
    static constexpr uint32_t kSignMask = 0x80000000u;
};

// The same contraction in blocks of 16 x 16: 32 elements of the contraction per instruction, lane l carries chunk l / 16 (8 elements) of
// row l % 16 of either operand and accumulator r is element (4 (l / 16) + r, l % 16).  Half the accumulator traffic per product of the
// 32 x 32 shape: under the board's power cap normal operands run at 2.09 instead of 1.82 PFLOP/s (both sustained for 0.1 s, from one instruction to the
// next changing one operand only; changing both 2.02 and 1.80; zeros 2.46 either way).
__device__ __forceinline__ void mma16(f32x4& acc, const u32x4& a, const u32x4& b)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// vmcnt(0) with the other counters left alone (gfx9 encoding of s_waitcnt)
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// lgkmcnt(0): the LDS reads issued so far have returned their data
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }
// vmcnt(N): wait until at most the N youngest vector-memory operations are outstanding
template <int N> __device__ __forceinline__ void wait_vmem_le()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// 16 bytes per lane from global memory straight into LDS (lane i lands at dst + 16*i;
// dst is wave-uniform).  The __restrict__ parameters give the transfer an alias scope of
// its own once inlined, which is what lets the compiler see that LDS reads from the
// OTHER tile buffer need not wait for it.
__device__ __forceinline__ void dma16(const char* __restrict__ src, char* __restrict__ dst)
{
    __builtin_amdgcn_global_load_lds((global_cptr)src, (lds_ptr)dst, 16, 0, 0);
}

// The same transfer issued from inline assembly, which the compiler's wait-count pass does not see: the
// only waits on it are the explicit vmcnt waits of the caller (vector-memory operations retire in order).
// lds_base = byte offset in LDS, wave-uniform (it travels in M0), the transfer inside the first kDirectLds bytes.
// (More than 64 KiB: attention_f32.hip stages V from there up to 128 KiB, and its results there agree with the oracle.)
constexpr int kDirectLds = 128 * 1024;
__device__ __forceinline__ void dma16_untracked(const char* src, uint32_t lds_base)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(src) : "memory", "m0");
#endif
}

// The same from a wave-uniform base and a byte offset per lane.
__device__ __forceinline__ void dma16_untracked(const char* base, uint32_t offset, uint32_t lds_base)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(offset), "s"(base) : "memory", "m0");
#endif
}

__device__ __forceinline__ uint32_t lds_offset_of(const void* p)
{
    return (uint32_t)(uintptr_t)(lds_ptr)(p);
}

// Transposing LDS read (ds_read_b64_tr_b16): each group of 16 lanes reads four runs of 16 elements of 2 bytes, lanes
// 4j .. 4j + 3 run j (8 bytes a lane), and lane i of the group gets element i of the four runs.
__device__ __forceinline__ u32x2 lds_read_tr16(const char* p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef s16x4 __attribute__((address_space(3)))* tr_ptr;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(p)));
#else
    (void)p;
    return u32x2{0u, 0u};
#endif
}
__device__ __forceinline__ u32x4 u32x4_of(u32x2 lo, u32x2 hi) { return u32x4{lo[0], lo[1], hi[0], hi[1]}; }

template <int I> struct IC { static constexpr int value = I; };

// f(IC<0>{}), f(IC<1>{}), ... f(IC<N-1>{})
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(IC<N - 1>{});
    }
}

// Calls body(t, IC<buffer>) for t = first .. n-1 with the LDS buffer alternating from
// `buf_first`; the buffer is a compile-time constant inside body.
template <typename Body>
__device__ __forceinline__ void for_tiles(int first, int buf_first, int n, Body&& body)
{
    int t = first;
    if (buf_first == 1 && t < n) { body(t, IC<1>{}); ++t; }
    for (; t + 1 < n; t += 2) {
        body(t, IC<0>{});
        body(t + 1, IC<1>{});
    }
    if (t < n) body(t, IC<0>{});
}

}  // namespace attnw
