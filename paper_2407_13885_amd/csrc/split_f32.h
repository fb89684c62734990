// fp32 contractions on the bf16 matrix instruction.
//
// x = hi + mid + lo with three bf16 numbers, each the rest rounded to nearest: 24 significand bits, the whole of x
// (|x| below 2^-110 loses bits of lo to bf16's smallest numbers; infinities and |x| above 3.38e38 make NaN, which the
// callers look for in their results).  Of the nine products of two such numbers the six above 2^-24 of the whole are
// kept.  Six v_mfma_f32_32x32x16_bf16 do the work of eight v_mfma_f32_32x32x2_f32 in 6 x 32 instead of 8 x 64 cycles.
// Against 64 bits (32 x 32 scores of normal vectors, relative error in units of 1e-7): fp32 instruction 1.02 / 1.45 / 2.06 /
// 2.92 at d = 32 / 64 / 128 / 256, the six products in one accumulator, smallest first, 0.69 / 1.10 / 1.64 / 2.39.
#pragma once

#include "qk_common.h"

namespace attnw {

struct Split8 { u32x4 hi, mid, lo; };             // 8 consecutive elements of the contraction

__device__ __forceinline__ Split8 split8(const float (&x)[8])
{
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
        s.hi[i] = pack_bf16x2(a, b);
        a -= bf16_lo_to_f32(s.hi[i]);
        b -= bf16_hi_to_f32(s.hi[i]);
        s.mid[i] = pack_bf16x2(a, b);
        a -= bf16_lo_to_f32(s.mid[i]);
        b -= bf16_hi_to_f32(s.mid[i]);
        s.lo[i] = pack_bf16x2(a, b);
    }
    return s;
}

__device__ __forceinline__ void mma_split(f32x16& acc, const Split8& a, const Split8& b)
{
    Mma<uint16_t>::run(acc, a.lo, b.hi);
    Mma<uint16_t>::run(acc, a.hi, b.lo);
    Mma<uint16_t>::run(acc, a.mid, b.mid);
    Mma<uint16_t>::run(acc, a.mid, b.hi);
    Mma<uint16_t>::run(acc, a.hi, b.mid);
    Mma<uint16_t>::run(acc, a.hi, b.hi);
}

// The same in two sums that the caller adds (0.5 to 0.8 of the error).
__device__ __forceinline__ void mma_split(f32x16& acc, f32x16& rest, const Split8& a, const Split8& b)
{
    Mma<uint16_t>::run(rest, a.lo, b.hi);
    Mma<uint16_t>::run(acc, a.mid, b.hi);
    Mma<uint16_t>::run(rest, a.hi, b.lo);
    Mma<uint16_t>::run(acc, a.hi, b.mid);
    Mma<uint16_t>::run(rest, a.mid, b.mid);
    Mma<uint16_t>::run(acc, a.hi, b.hi);
}

}  // namespace attnw
