// fp32 contractions on the bf16 matrix instruction (the three-way split and its six products: G. Henry, P. T. P. Tang and
// A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019).
//
// 2^24 x = hi + mid + lo with three bf16 numbers, each the rest rounded to nearest: 24 significand bits, the whole of x.  The
// factor keeps the last part of the smallest fp32 number a normal bf16 number: without it |x| below 2^-110 lost up to 16 of its bits
// (attention over V of 2^-118 / 2^-122: 9.5e-6 / 1.4e-4 off, 3e-7 in fp32).  Infinities, NaN and |x| from 2^104 on make NaN, sums of
// products from 2^80 on infinity: the callers look for either in their scores and sums and start again in fp32.
// Of the nine products of two such numbers the six above 2^-24 of the whole are kept.  Six v_mfma_f32_32x32x16_bf16 do the work of
// eight v_mfma_f32_32x32x2_f32 in 6 x 32 instead of 8 x 64 cycles.
// Against 64 bits (32 x 32 scores of normal vectors, relative error in units of 1e-7): fp32 instruction 1.02 / 1.45 / 2.06 /
// 2.92 at d = 32 / 64 / 128 / 256, the six products in one accumulator, smallest first, 0.69 / 1.10 / 1.64 / 2.39.
#pragma once

#include "qk_common.h"

namespace attnw {

constexpr float kSplitUp = 0x1p24f;               // of an operand
constexpr float kSplitDown = 0x1p-48f;            // of a product of two

struct Split8 { u32x4 hi, mid, lo; };             // 8 consecutive elements of the contraction

__device__ __forceinline__ Split8 split8(const float (&x)[8])   // (x: already times kSplitUp)
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

// 8 elements of a row of d from column col on (d is a multiple of 4: a half lies inside the row or past it, and is then a copy
// of the row's first four)
struct Row8 { f32x4 a, b; };

__device__ __forceinline__ Row8 load_row8(const float* row, int col, int d)
{
    return {*reinterpret_cast<const f32x4*>(row + (col < d ? col : 0)), *reinterpret_cast<const f32x4*>(row + (col + 4 < d ? col + 4 : 0))};
}

__device__ __forceinline__ float largest(const Row8& r)   // |element|, NaN aside
{
    const float x = fmaxf(max3(fabsf(r.a[0]), fabsf(r.a[1]), fabsf(r.a[2])), fabsf(r.a[3]));
    return max3(max3(x, fabsf(r.b[0]), fabsf(r.b[1])), fabsf(r.b[2]), fabsf(r.b[3]));
}

// Their parts, zeros past the row's end (NaN where the copies are not finite: as the elements that they are copies of)
__device__ __forceinline__ Split8 split_row8(const Row8& r, int col, int d, float up = kSplitUp)
{
    const float ua = col < d ? up : 0.0f, ub = col + 4 < d ? up : 0.0f;
    float x[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = r.a[e] * ua;
        x[4 + e] = r.b[e] * ub;
    }
    return split8(x);
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
