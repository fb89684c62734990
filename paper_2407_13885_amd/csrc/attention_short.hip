// Attention output  O = softmax(scale * Q K^T) V  for sequences of at most 32 tokens with d above 128 (bf16: a multiple of 16, fp32:
// of 4, up to 256).
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the max-subtracted softmax of the
// Softmax section, Eq. 1: all keys of a row are at hand at once.)
//
// One wave per head, operands straight from global memory: nothing is read by two waves, so a way through LDS only takes
// the room of other waves (K and V of a head are 64 KiB in fp32 at d = 256).  What bounds it: the loads of a head one batch behind the
// other, two waves to a SIMD.  The next batch is always under way (a compiler barrier keeps its loads ahead of the
// matrix instructions of the batch before; without, they went one at a time: 2000 fp32 heads of N = 32, d = 184 40 -> 35.5 us, 500
// 27 -> 14).  Measured, us, against the kernels that stage K and V: fp32 2000 heads of N = 32, d = 256 88 -> 46 (5.7 TB/s of Q, K, V
// and O), of 17, d = 200 99 -> 29, two heads of 17, d = 256 18 -> 13; bf16 3500 of 17, d = 176 40 -> 19, of 32, d = 256 64 -> 49, 300 of 17,
// d = 144 5.6 -> 4.2.
//   S^T = K * Q^T        lane (query l32, half h) holds keys 8i + 4h + j of its query
//   O^T += V^T * P^T     fp32: one v_mfma_f32_32x32x2_f32 per accumulator r and 32 columns: the key pair (r, half 0 and 1) against one
//                        float of V per lane.  bf16: 16 keys per instruction, the lane's 8 weights (rounded to bf16) are its
//                        operand, the 8 values of V are gathered by 2-byte loads.
#include "attention_common.h"
#include "launchers.h"

namespace attnw {
namespace {

constexpr int largest_divisor_up_to_8(int n)
{
    int best = 1;
    for (int k = 2; k <= 8; ++k)
        if (n % k == 0) best = k;
    return best;
}

// DVB: 32-column blocks of a row, ceil(d / 32).  rb: bytes of a row.  Every load is unconditional, at an address inside the arrays,
// and replaced by zero where it lies past the end of the row or (V) of the sequence: loads under a branch would be waited
// for one by one.
template <typename T, int DVB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attention_short_kernel(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
                            int N, int rb, float c, uint32_t sign_flip, uint32_t total)
{
    constexpr int E = (int)sizeof(T);
    constexpr int G = DVB * E;                    // 32-byte contraction groups of a padded row
    constexpr int GB = largest_divisor_up_to_8(G);   // groups per batch of loads

    const uint32_t bh = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (bh >= total) return;
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int d = rb / E;
    const int last_chunk = rb / 16 - 1;
    const int64_t at = (int64_t)bh * N * rb;
    const char* const Vh = reinterpret_cast<const char*>(V) + at;
    const int row = min(l32, N - 1);              // (keys past the end are copies of key N - 1: no new maximum)

    // ---- scores ----------------------------------------------------------------------------------------------------------
    const char* const qrow = reinterpret_cast<const char*>(Q) + at + row * rb;
    const char* const krow = reinterpret_cast<const char*>(K) + at + row * rb;
    // (batch b + 1 is requested before the instructions of batch b: left to itself the compiler loads one chunk at a time)
    u32x4 kf[2][GB], qf[2][GB];
    auto load = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            const int off = min(2 * (b * GB + g) + half, last_chunk) * 16;
            kf[b & 1][g] = *reinterpret_cast<const u32x4*>(krow + off);
            qf[b & 1][g] = *reinterpret_cast<const u32x4*>(qrow + off);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.0f;
    load(0);
#pragma unroll
    for (int b = 0; b < G / GB; ++b) {
        if (b + 1 < G / GB) load(b + 1);
#pragma unroll
        for (int g = 0; g < GB; ++g) {            // (a negative scale negates Q; only the last block of columns has padding)
            const bool in = b * GB + g < (DVB - 1) * E || 2 * (b * GB + g) + half <= last_chunk;
            Mma<T>::run(s, in ? kf[b & 1][g] : u32x4{0u, 0u, 0u, 0u}, in ? qf[b & 1][g] ^ sign_flip : u32x4{0u, 0u, 0u, 0u});
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- the first values of V, for the time of the softmax ------------------------------------------------------------------
    int vcol[DVB];                                // the lane's column of every output block, inside the row
#pragma unroll
    for (int b = 0; b < DVB; ++b) vcol[b] = min(b * 32 + l32, d - 1) * E;
    // fp32: accumulator r is the weight of key 8 (r / 4) + 4 half + r % 4, a batch is four keys (one r / 4).  bf16: operand slot e of
    // a lane is key 16m + 8 (e / 4) + 4 half + e % 4 (the key of accumulator 8m + e), a batch is the eight of one m.
    constexpr int VK = E == 4 ? 4 : 8, VB = 16 / VK;
    auto vkey = [&](int m, int e) __attribute__((always_inline)) { return 32 / VB * m + 8 * (e / 4) + 4 * half + e % 4; };
    T v[2][VK][DVB];
    auto v_load = [&](int m) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < VK; ++e)
#pragma unroll
            for (int b = 0; b < DVB; ++b) v[m & 1][e][b] = *reinterpret_cast<const T*>(Vh + min(vkey(m, e), N - 1) * rb + vcol[b]);
        __builtin_amdgcn_sched_barrier(0);
    };
    v_load(0);

    // ---- weights ---------------------------------------------------------------------------------------------------------
    float tm = max3(s[0], s[1], s[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
    const float mb = fmaxf(half_wave_max(fmaxf(tm, s[15])) * c, kNegBig);
    float p[16], sum = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        p[r] = 4 * half + 8 * (r / 4) + (r % 4) < N ? fast_exp2(__builtin_fmaf(s[r], c, -mb)) : 0.0f;
        sum += p[r];
    }

    // ---- output ------------------------------------------------------------------------------------------------------------
    f32x16 oacc[DVB];
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
#pragma unroll
    for (int m = 0; m < VB; ++m) {
        if (m + 1 < VB) v_load(m + 1);
        if constexpr (E == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < DVB; ++b)
                    oacc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vkey(m, e) < N ? v[m & 1][e][b] : 0.0f, p[4 * m + e], oacc[b], 0, 0, 0);
        } else {
            u32x4 pw;
#pragma unroll
            for (int i = 0; i < 4; ++i) pw[i] = pack_bf16x2(p[8 * m + 2 * i], p[8 * m + 2 * i + 1]);
#pragma unroll
            for (int b = 0; b < DVB; ++b) {
                u32x4 vf;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    vf[i] = (vkey(m, 2 * i) < N ? (uint32_t)v[m & 1][2 * i][b] : 0u) | (vkey(m, 2 * i + 1) < N ? (uint32_t)v[m & 1][2 * i + 1][b] << 16 : 0u);
                Mma<uint16_t>::run(oacc[b], vf, pw);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- normalise, round once (bf16), store: a lane owns runs of 4 consecutive output columns of its query ------------------
    const float inv = 1.0f / half_wave_sum(sum);
    if (l32 >= N) return;
    char* const orow = reinterpret_cast<char*>(O) + at + l32 * rb;
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int col = b * 32 + 8 * i + 4 * half;   // (d is a multiple of 4: the run lies inside the row or past it)
            if (col >= d) continue;
            const f32x4 o = f32x4{oacc[b][4 * i], oacc[b][4 * i + 1], oacc[b][4 * i + 2], oacc[b][4 * i + 3]} * inv;
            if constexpr (E == 4) *reinterpret_cast<f32x4*>(orow + col * 4) = o;
            else *reinterpret_cast<u32x2*>(orow + col * 2) = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
        }
}

template <typename T, int DVB>
hipError_t launch_short_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    return launch_by_heads(BH, 1, 64, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * d;
        const uint32_t total = (uint32_t)heads, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_short_kernel<T, DVB>), dim3(grid), dim3(64), 0, stream, static_cast<const T*>(Q) + at,
                           static_cast<const T*>(K) + at, static_cast<const T*>(V) + at, static_cast<T*>(O) + at, N, d * (int)sizeof(T),
                           fabsf(scale) * kLog2e, scale < 0.0f ? Mma<T>::kSignMask : 0u, total);
        return hipGetLastError();
    });
}

template <typename T>
hipError_t launch_short(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    switch ((d + 31) / 32) {
    case 5: return launch_short_t<T, 5>(Q, K, V, O, BH, N, d, scale, stream);
    case 6: return launch_short_t<T, 6>(Q, K, V, O, BH, N, d, scale, stream);
    case 7: return launch_short_t<T, 7>(Q, K, V, O, BH, N, d, scale, stream);
    case 8: return launch_short_t<T, 8>(Q, K, V, O, BH, N, d, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_attention_short(DType dt, const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                  float scale, hipStream_t stream)
{
    if (dt == DType::F32) return launch_short<float>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    return launch_short<uint16_t>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
}

}  // namespace attnw
