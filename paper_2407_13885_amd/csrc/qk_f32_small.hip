// Fused attention weights  P = softmax(scale * Q K^T)  in fp32 for few short heads (N up to 256, d a multiple of 4 from 20 to 256): as little as
// possible between the launch and the store.
//
// (Paper: the fused kernel of the section "Fused Matrix Multiply + Scaling + Softmax": scores stay where the multiply left them, local maxima and sums
// are exchanged once, Softmax section, Eq. 1.)
//
// A workgroup owns 16 queries of a head, its eight waves blocks of 16 keys.  K comes straight from memory in the layout of the fp32 matrix instruction
// (16 x 16 x 4: lane l has chunk l / 16 of 16 columns of row l % 16, instruction e of a group takes element e), all of a block requested at once; Q
// through LDS (every wave for itself is 0.5 us more: the loads of a compute unit leave one after the other); one exchange of (maximum, sum); a lane
// stores runs of four keys.  Nothing is split into parts: of the some 400 instructions that a wave of qk_f32_strip.hip needs for a block, at 7 cycles
// each where it has the SIMD for itself, 200 do that.  Scores are four sums (one for each element of a chunk), up to d = 48 eight, added at the end: error
// against 64 bits 0.96 (d = 20) to 0.52 (256) of that of the strips; up to d = 16 it would be up to 1.1.
// What bounds it: the launch, one way to memory and back, and the loads of a compute unit.  us, strips / here: one head of N = 128, d = 64 5.4 / 4.4, of 64 5.0 / 3.7,
// of 100 6.2 / 4.0, of 128, d = 128 6.7 / 5.8, of 64, d = 256 9.0 / 5.9, one of 206, d = 64 7.3 / 6.2, 128 of 32 5.2 / 3.2.
#include "launchers.h"
#include "qk_common.h"

namespace attnw {
namespace {

// NB: blocks of a wave at most; NG: groups of 16 columns at most.  Rows past N are read as row N - 1, weigh nothing and are not stored.
template <int NB, int NG>
__global__ __launch_bounds__(512)
void qk_f32_small_kernel(const float* __restrict__ Q, const float* __restrict__ K, float* __restrict__ P, int N, int d, float c, float q_sign,
                         uint32_t strips)
{
    constexpr int NW = 8, SUMS = NG <= 3 ? 8 : 4;
    constexpr int QC = NG * 4, QP = QC < 16 ? 16 : QC;           // chunks of a row, of one in LDS
    __shared__ float stat_lds[NW * 32];
    __shared__ f32x4 q_lds[16 * QP];              // chunks swizzled by the row
    const uint32_t bh = blockIdx.x / strips;
    const int q0 = (int)(blockIdx.x - bh * strips) * 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l16 = lane & 15;
    const int quarter = lane >> 4;
    const float* const Qh = Q + (int64_t)bh * N * d;
    const float* const Kh = K + (int64_t)bh * N * d;
    const int all_blocks = (N + 15) / 16;
    const int nb = (all_blocks - wave + NW - 1) / NW;            // blocks of this wave: wave, wave + 8, ..

    // (columns past d: zeros)
    auto chunk = [&](const float* row, int g) __attribute__((always_inline)) {
        const int col = g * 16 + quarter * 4;
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + (col < d ? col : 0));
        return col < d ? v : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    f32x4 kf[2][NG], qf[NG];
    auto load_k = [&](int i, f32x4 (&f)[NG]) __attribute__((always_inline)) {
        const float* const row = Kh + (int64_t)min((wave + NW * i) * 16 + l16, N - 1) * d;
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (g * 16 < d) f[g] = chunk(row, g);
    };
    // (Q first and once for all waves: it is in LDS while K is on its way)
    constexpr int QL = (16 * QC + 511) / 512;     // chunks of a thread
    f32x4 q_raw[QL];
#pragma unroll
    for (int i = 0; i < QL; ++i) {
        const int at = i * 512 + threadIdx.x, col = at % QC * 4;
        if (at < 16 * QC) q_raw[i] = *reinterpret_cast<const f32x4*>(Qh + (int64_t)min(q0 + at / QC, N - 1) * d + (col < d ? col : 0));
    }
    load_k(0, kf[0]);
#pragma unroll
    for (int i = 0; i < QL; ++i) {
        const int at = i * 512 + threadIdx.x, r = at / QC;
        if (at < 16 * QC) q_lds[r * QP + (at % QC ^ r)] = at % QC * 4 < d ? q_raw[i] * q_sign : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < NG; ++g) qf[g] = q_lds[l16 * QP + ((g * 4 + quarter) ^ l16)];

    // ---- scores: keys 16 (wave + 8 i) + 4 quarter .. + 3 of query q0 + l16 ---------------------------------------------------------------------
    f32x4 s[NB];
    float m = -0x1.fffffep127f;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (i >= nb) break;                       // (wave-uniform)
        if (i + 1 < NB && i + 1 < nb) load_k(i + 1, kf[(i + 1) & 1]);
        f32x4 sum[SUMS];
#pragma unroll
        for (int e = 0; e < SUMS; ++e) sum[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (g * 16 < d)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    constexpr int TWO = SUMS / 4 - 1;
                    sum[4 * (g & TWO) + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i & 1][g][e], qf[g][e], sum[4 * (g & TWO) + e], 0, 0, 0);
                }
        s[i] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        if constexpr (SUMS == 8) s[i] += (sum[4] + sum[5]) + (sum[6] + sum[7]);
        m = max3(max3(m, s[i][0], s[i][1]), s[i][2], s[i][3]);   // (keys past the end are copies of key N - 1: no new maximum)
    }
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    // Exponents are products of differences: against fl(m c) the keys of a wave whose scores are all far below the others' (a mask through a column of K)
    // weigh 2 to the rounding of that product, infinity from |m c| of 2^32 on, and infinity times 2^(m - the row's) is NaN in every weight of the row.
    // (Halves: the difference of two scores may leave fp32's range.)
    auto weight = [&](float x, float largest) __attribute__((always_inline)) { return fast_exp2(__builtin_fmaf(x, 0.5f, -0.5f * largest) * c * 2.0f); };
    float l = 0.0f;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (i >= nb) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[i][r] = weight(s[i][r], m);
            if ((wave + NW * i) * 16 + 4 * quarter + r >= N) s[i][r] = 0.0f;
        }
        l += (s[i][0] + s[i][1]) + (s[i][2] + s[i][3]);
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (quarter == 0) {
        stat_lds[wave * 32 + l16] = m;
        stat_lds[wave * 32 + 16 + l16] = l;
    }
    __syncthreads();
    const int waves = min(NW, all_blocks);        // those with keys
    float m_row = stat_lds[l16], l_row = 0.0f;
    for (int w = 1; w < waves; ++w) m_row = fmaxf(m_row, stat_lds[w * 32 + l16]);
    for (int w = 0; w < waves; ++w) l_row += stat_lds[w * 32 + 16 + l16] * weight(stat_lds[w * 32 + l16], m_row);
    const float f = weight(m, m_row) * (1.0f / l_row);

    // ---- weights ----------------------------------------------------------------------------------------------------------------------------
    const int q = q0 + l16;
    if (q >= N) return;
    float* const row = P + ((int64_t)bh * N + q) * N;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (i >= nb) break;
        const int key = (wave + NW * i) * 16 + 4 * quarter;
        if (N % 4 == 0) {
            if (key < N) *reinterpret_cast<f32x4*>(row + key) = s[i] * f;
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (key + r < N) row[key + r] = s[i][r] * f;
        }
    }
}

template <int NB, int NG>
hipError_t launch_small_t(const void* Q, const void* K, void* P, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((N + 15) / 16);
    hipLaunchKernelGGL((qk_f32_small_kernel<NB, NG>), dim3((uint32_t)BH * strips), dim3(512), 0, stream, static_cast<const float*>(Q),
                       static_cast<const float*>(K), static_cast<float*>(P), N, d, fabsf(scale) * kLog2e, scale < 0.0f ? -1.0f : 1.0f, strips);
    return hipGetLastError();
}

template <int NG>
hipError_t launch_small_g(const void* Q, const void* K, void* P, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    return N <= 128 ? launch_small_t<1, NG>(Q, K, P, BH, N, d, scale, stream) : launch_small_t<2, NG>(Q, K, P, BH, N, d, scale, stream);
}

}  // namespace

// One workgroup to a compute unit, half of them where a wave has two blocks.  560 random shapes: 0.4 to 1.0 of the time within; beyond up to 1.3 (N <= 128)
// and 1.65 (N <= 256), as the fp32 instruction takes longer than the strips' bf16 parts; 257 to 512 tokens 0.8 to 1.2.  d above 128 up to 192 tokens only
// (0.83 to 0.91 from 154 on): K of more leaves a compute unit too slowly, 193 to 256 tokens 0.93 to 1.1 (six heads of 247, d = 256 13.1 -> 14.5 us); of those d of 97 to
// 128 but 224 and 256, whole blocks for the strips (1.02 and 1.06; others 0.9 to 0.97).
bool prefers_f32_small(int64_t BH, int64_t N, int64_t d)
{
    if (d <= 16 || N > 256 || (N > 192 && (d > 128 || (d > 96 && N % 32 == 0)))) return false;
    return BH * ((N + 15) / 16) <= (N <= 128 ? 2 : 1) * (int64_t)compute_units() / 2;
}

hipError_t launch_qk_f32_small(const void* Q, const void* K, void* P, int64_t BH, int64_t N, int64_t d, float scale, hipStream_t stream)
{
    if (d <= 32) return launch_small_g<2>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    if (d <= 48) return launch_small_g<3>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    if (d <= 64) return launch_small_g<4>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    return d <= 128 ? launch_small_g<8>(Q, K, P, BH, (int)N, (int)d, scale, stream) : launch_small_g<16>(Q, K, P, BH, (int)N, (int)d, scale, stream);
}

}  // namespace attnw
