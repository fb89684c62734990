// Attention output  O = softmax(scale * Q K^T) V  in fp32 (d a multiple of 4 up to 256, any N).
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the product
// with V is what the section "Limitations and future Directions" names as the next thing to fuse.  The
// max-subtracted softmax of the Softmax section, Eq. 1, is applied incrementally as in the bf16 kernels.)
//
// What bounds it: v_mfma_f32_32x32x2_f32, 64 cycles an instruction (157 TFLOP/s on the chip).  One instruction of
// either contraction needs 256 bytes from LDS, a fraction of what the LDS delivers in that time, so all that
// counts is that a SIMD always has a matrix instruction to issue: K and V are staged in LDS by transfers that run
// while the other contraction of the tile is under way, and the softmax of one wave is covered by the matrix
// instructions of the other wave on its SIMD (two workgroups per compute unit up to d = 128).  Measured, N = 4096, against
// one wave per workgroup with operands straight from the caches: 16 heads of d = 256 3.97 -> 2.11 ms (130 TFLOP/s), one head of
// d = 128 1.03 -> 0.16.  (Many heads with d <= 128: attention_f32_split.hip, attention_f32_turns.hip; at most 32 keys with d > 128: attention_short.hip.)
//
// A workgroup of (usually) four waves: WQ query blocks of 32 x WK key ranges.  A tile is 32 keys per key range; K and V have one
// buffer each, and every tile has two phases:
//   K landed, V wanted:  S^T = K_sub * Q^T, softmax      (V tile under way: it has this whole phase)
//   V landed:            O^T += V_sub^T * P^T            (next K tile under way)
// Accumulator r of a lane is the weight of key 8 (r / 4) + 4 half + r % 4; the second contraction takes one
// instruction per accumulator and 32 output columns: the key pair (r, half 0 and 1) against one float of V per lane,
// so weights go from the exponential to the matrix core as they are.  K rows are swizzled by 16-byte chunks, V rows lie
// as in memory.
// WK > 1 (problems of a few heads): a wave takes one 32-key sub-tile of every tile and the partial results of a query
// block, each with its own reference exponent and sum, are merged through LDS at the end.
#include "attention_common.h"
#include "launchers.h"

namespace attnw {
namespace {

__device__ const u32x4 kZeros = {0u, 0u, 0u, 0u};

// CS: workgroups that share the columns of V and O of a query block
template <int DVB, int WQ, int WK, int CS>
struct F32Cfg {
    static constexpr int NW = WQ * WK;            // waves per workgroup
    static constexpr int BM = 32 * WQ;            // queries per workgroup
    static constexpr int BN = 32 * WK;            // keys per tile
    static constexpr int DB = DVB * 128;          // bytes of a padded row on chip
    static constexpr int CPR = DB / 16;
    static constexpr int TILE = BN * DB;
    static constexpr int LOADS = TILE / 1024 / NW;   // wave-wide transfers per wave and tile
    static constexpr int OB = DVB / CS;           // 32-column blocks of V and O
    static constexpr int V_TILE = TILE / CS;
    static constexpr int SLOTS = 2 + OB * 16;     // merge: reference exponent, sum, output accumulators
    static constexpr int MERGE = WK > 1 ? NW * SLOTS * 256 : 0;
    static constexpr int LDS = TILE + V_TILE > MERGE ? TILE + V_TILE : MERGE;
    static_assert(DVB % CS == 0 && TILE % (1024 * NW) == 0 && V_TILE % (1024 * NW) == 0, "whole column blocks, whole transfers");
    static_assert(TILE + V_TILE <= kDirectLds, "reach of direct transfers");
};

// DVB: 32-column blocks of an output row, ceil(d / 32); rows are padded to 32 DVB elements on chip (rb: bytes of a row
// in memory).  Padding chunks are transferred from an array of zeros (any of the caller's numbers could be infinite, and NaN
// against the zeros of the padded Q fragments).  Rows past N are read as row N - 1.
// CS > 1 (few heads): CS workgroups share a block, each makes all scores but reads and multiplies its share of the columns of V only.  (d >
// 128: the tiles of V are smaller, so that three or four key ranges fit instead of two.)
template <int DVB, int WQ, int WK, int CS>
__global__ __launch_bounds__(64 * WQ * WK, DVB <= 4 ? 2 : 1)
void attention_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                          float* __restrict__ O, int N, int rb, float c, uint32_t sign_flip, uint32_t strips, uint32_t total)
{
    using C = F32Cfg<DVB, WQ, WK, CS>;
    constexpr int NW = C::NW, DB = C::DB, CPR = C::CPR, BN = C::BN, LOADS = C::LOADS, OB = C::OB, DBV = OB * 128;
    constexpr int G = DVB * 4;                    // 32-byte contraction groups of a padded row

    __shared__ __align__(1024) char lds[C::LDS];
    char* const k_lds = lds;
    char* const v_lds = lds + C::TILE;

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t block = logical / CS;
    const int col0 = (int)(logical % CS) * OB * 32;   // this workgroup's first column of V and O
    const uint32_t bh = block / strips;
    const uint32_t strip = block - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int wq = wave / WK, wk = wave % WK;

    const char* Qh = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * rb;
    const char* Kh = reinterpret_cast<const char*>(K) + (int64_t)bh * N * rb;
    const char* Vh = reinterpret_cast<const char*>(V) + (int64_t)bh * N * rb;
    char* Oh = reinterpret_cast<char*>(O) + (int64_t)bh * N * rb;
    const int q0 = strip * C::BM + wq * 32;
    const int row_chunks = rb / 16;

    // ---- Q fragments: chunk 2g + half of the lane's query; a negative scale negates Q --------------------------
    u32x4 qf[G];
    {
        const char* qrow = Qh + (int64_t)min(q0 + l32, N - 1) * rb;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int ch = 2 * g + half;
            const u32x4 v = *reinterpret_cast<const u32x4*>(qrow + min(ch, row_chunks - 1) * 16);
            qf[g] = ch < row_chunks ? v ^ sign_flip : u32x4{0u, 0u, 0u, 0u};
        }
    }

    // ---- tile transfers: chunk s = (wave + NW j) 64 + lane of the tile; the swizzle permutes chunks within a row ----
    const uint32_t k_base = lds_offset_of(k_lds), v_base = lds_offset_of(v_lds);
    auto k_issue = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int s = (wave + NW * j) * 64 + lane;
            const int key = s / CPR;
            const int ch = (s - key * CPR) ^ (key & 7);
            const char* src = Kh + (int64_t)min(t * BN + key, N - 1) * rb + ch * 16;
            if (ch >= row_chunks) src = reinterpret_cast<const char*>(&kZeros);
            dma16_untracked(src, k_base + (wave + NW * j) * 1024);
        }
    };
    auto v_issue = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < LOADS / CS; ++j) {
            const int s = (wave + NW * j) * 64 + lane;
            const int key = s / (CPR / CS);
            const int ch = s - key * (CPR / CS) + col0 / 4;
            const char* src = Vh + (int64_t)min(t * BN + key, N - 1) * rb + ch * 16;
            if (ch >= row_chunks) src = reinterpret_cast<const char*>(&kZeros);
            dma16_untracked(src, v_base + (wave + NW * j) * 1024);
        }
    };

    const char* const krow = k_lds + (wk * 32 + l32) * DB;
    int kswz[4];                                  // chunk (2g + half) ^ (key & 7): its low three bits repeat every four groups
#pragma unroll
    for (int g = 0; g < 4; ++g) kswz[g] = ((2 * g + half) ^ (l32 & 7)) * 16;
    const char* const vrow = v_lds + (wk * 32 + 4 * half) * DBV + l32 * 4;

    f32x16 oacc[OB];
#pragma unroll
    for (int b = 0; b < OB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
    float mb_run = kNegBig, l_run = 0.0f;
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent

    const int n_tiles = (N + BN - 1) / BN;
    k_issue(0);
    for (int t = 0; t < n_tiles; ++t) {
        const int key0 = t * BN + wk * 32;
        const bool active = q0 < N && key0 < N;   // (wave-uniform: otherwise the wave only moves tiles)
        wait_vmem();
        __syncthreads();                          // K tile t has landed; every wave is past the V tile before it
        v_issue(t);
        float p[16];
        if (active) {
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
            for (int g = 0; g < G; ++g)
                Mma<float>::run(s, *reinterpret_cast<const u32x4*>(krow + (g / 4) * 128 + kswz[g % 4]), qf[g]);

            float tm = max3(s[0], s[1], s[2]);
#pragma unroll
            for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
            const float m = half_wave_max(fmaxf(tm, s[15]));   // (keys past the end are copies of key N-1: no new maximum)
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(m * c > mb_run + kLazy) != 0, 0)) {
                const float mb_new = fmaxf(mb_run, reference_exponent(m, c));
                const float alpha = fast_exp2(mb_run - mb_new);   // exactly 1 for lanes whose exponent stands
                l_run *= alpha;
#pragma unroll
                for (int b = 0; b < OB; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[b][r] *= alpha;
                mb_run = mb_new;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mb_run));
            if (key0 + 32 > N) {                  // keys past the end weigh nothing
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (key0 + 4 * half + 8 * (r / 4) + (r % 4) >= N) p[r] = 0.0f;
            }
            float sum = p[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) sum += p[r];
            l_run += sum;
        }
        wait_vmem();
        __syncthreads();                          // V tile t has landed; every wave is past K tile t
        if (t + 1 < n_tiles) k_issue(t + 1);
        if (active) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int b = 0; b < OB; ++b)
                    oacc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                        *reinterpret_cast<const float*>(vrow + (8 * (r / 4) + r % 4) * DBV + b * 128), p[r], oacc[b], 0, 0, 0);
        }
    }
    wait_vmem();                                  // no transfer may be in flight when the LDS is reused or released

    // ---- normalise and store: a lane owns runs of 4 consecutive output columns of its query ----------------------
    const int d = rb / 4 - col0;              // columns from this workgroup's first on
    char* const orow = Oh + (int64_t)(q0 + l32) * rb + col0 * 4 + half * 16;
    if constexpr (WK > 1) {
        constexpr int SLOTS = C::SLOTS;
        float* const part = reinterpret_cast<float*>(lds);
        __syncthreads();
        float* const mine = part + wave * SLOTS * 64 + lane;
        mine[0] = mb_run;
        mine[64] = l_run;
#pragma unroll
        for (int b = 0; b < OB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[(2 + b * 16 + r) * 64] = oacc[b][r];
        __syncthreads();
        const float* const grp = part + wq * WK * SLOTS * 64 + lane;
        float f[WK], M = grp[0], L = 0.0f;
#pragma unroll
        for (int j = 1; j < WK; ++j) M = fmaxf(M, grp[j * SLOTS * 64]);
#pragma unroll
        for (int j = 0; j < WK; ++j) {            // (factor exactly 1 for the largest exponent, 0 for a range without keys)
            f[j] = fast_exp2(grp[j * SLOTS * 64] - M);
            L = __builtin_fmaf(f[j], grp[j * SLOTS * 64 + 64], L);
        }
        const float inv = 1.0f / half_wave_sum(L);
        if (q0 + l32 >= N) return;
        for (int b = wk; b < OB; b += WK)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < WK; ++j)
                        o[e] = __builtin_fmaf(f[j], grp[(j * SLOTS + 2 + b * 16 + 4 * i + e) * 64], o[e]);
                if (b * 32 + 8 * i + 4 * half < d)   // (d is a multiple of 4: the run lies inside the row or past it)
                    *reinterpret_cast<f32x4*>(orow + (b * 32 + 8 * i) * 4) = o * inv;
            }
    } else {
        const float inv = 1.0f / half_wave_sum(l_run);
        if (q0 + l32 >= N) return;
#pragma unroll
        for (int b = 0; b < OB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 o = {oacc[b][4 * i], oacc[b][4 * i + 1], oacc[b][4 * i + 2], oacc[b][4 * i + 3]};
                if (b * 32 + 8 * i + 4 * half < d) *reinterpret_cast<f32x4*>(orow + (b * 32 + 8 * i) * 4) = o * inv;
            }
    }
}

template <int DVB, int WQ, int WK, int CS = 1>
hipError_t launch_f32_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, int d, float scale,
                        hipStream_t stream)
{
    using C = F32Cfg<DVB, WQ, WK, CS>;
    const uint32_t strips = (uint32_t)((N + C::BM - 1) / C::BM);
    return launch_by_heads(BH, strips * CS, 64 * C::NW, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * d;
        const uint32_t total = (uint32_t)heads * strips * CS, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_f32_kernel<DVB, WQ, WK, CS>), dim3(grid), dim3(64 * C::NW), 0, stream, static_cast<const float*>(Q) + at,
                           static_cast<const float*>(K) + at, static_cast<const float*>(V) + at, static_cast<float*>(O) + at, N, d * 4,
                           fabsf(scale) * kLog2e, scale < 0.0f ? Mma<float>::kSignMask : 0u, strips, total);
        return hipGetLastError();
    });
}

// Key ranges per workgroup.  The time of a launch goes as (waves that the fullest SIMD gets) x (32-key sub-tiles of such
// a wave, one more where partial results are merged: what the merge was measured to cost).  Grids of less than four
// workgroups per compute unit are counted in whole workgroups; beyond that waves without queries or keys only leave
// room for others, and the last round is half full on average.
int key_ranges_f32(int64_t BH, int64_t N, int most)
{
    const int64_t cus = compute_units(), units = BH * ((N + 31) / 32);
    int best = 1;
    double best_cost = 0.0;
    for (int wk = 1; wk <= most; wk *= 2) {
        const int64_t bm = 128 / wk, wgs = BH * ((N + bm - 1) / bm);
        const double waves = wgs >= 4 * cus ? (double)(units * wk) / (4 * cus) + 0.5 : (double)((wgs + cus - 1) / cus);
        const double cost = waves * ((N + 32 * wk - 1) / (32 * wk) + (wk > 1 ? 1 : 0));
        if (wk == 1 || cost < best_cost) { best = wk; best_cost = cost; }
    }
    return best;
}

template <int DVB>
hipError_t launch_f32_ranges(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, int d, float scale,
                             hipStream_t stream)
{
    // at most two query blocks per head: workgroups of as many waves (4096 heads of N = 49, d = 32 with four, two of them
    // idle: 36 -> 30.5 us; of N = 20, d = 16: 22.5 -> 9.0).  d > 128: K and V of 32 keys would leave room for two workgroups on a compute
    // unit, and nothing shares them.
    if constexpr (DVB > 4) {
        if (N <= 32) return launch_attention_short(DType::F32, Q, K, V, O, BH, N, d, scale, stream);
    } else {
        if (N <= 32) return launch_f32_t<DVB, 1, 1>(Q, K, V, O, BH, N, d, scale, stream);
    }
    // Two, three or (d <= 64) five query blocks per head, more heads than compute units, about one block per SIMD (d <= 64 with
    // three or five: two): workgroups of several waves, not all with queries, come to unequal numbers on the compute units; one-wave
    // workgroups do not.  Measured, us, several waves / one: 270 heads of N = 64, d = 32 7.5 / 5.6, 293 of N = 64, d = 128 23.0 / 16.0, 304
    // of N = 68, d = 128 31 / 21, 450 of N = 40, d = 64 12.1 / 9.1, 539 of N = 96, d = 32 14.0 / 11.0, 300 of N = 140, d = 64 38 / 28; beyond:
    // 1000 of N = 40, d = 64 14.9 / 16.4, 600 of N = 64, d = 128 26 / 36, 400 of N = 128, d = 64 24.1 / 24.7; below: 200 of N = 64, d = 128
    // 13.9 / 14.5.
    if constexpr (DVB <= 4) {
        const int64_t blocks = (N + 31) / 32, most = (DVB <= 2 && blocks > 2 ? 8 : 4) * (int64_t)compute_units();
        if ((blocks <= 3 || (DVB <= 2 && blocks == 5)) && BH > compute_units() && BH * blocks <= most)
            return launch_f32_t<DVB, 1, 1>(Q, K, V, O, BH, N, d, scale, stream);
    }
    if (N <= 64) return launch_f32_t<DVB, 2, 1>(Q, K, V, O, BH, N, d, scale, stream);
    // d > 128, few heads: workgroups of one query block that share its columns.  What a launch takes goes as rounds x sub-tiles of a wave x
    // (blocks of columns contracted and multiplied); taken where that is a fifth less.  us, key ranges alone -> columns shared: one head of 1916,
    // d = 208 240 -> 168, two of 674, d = 256 104 -> 58, one of 200, d = 132 28 -> 13, three of 96, d = 144 21 -> 9, one of 4096, d = 192 422 -> 344; by less than
    // that: d = 256 561 -> 571, d = 160 347 -> 387.
    if constexpr (DVB > 4) {
        constexpr int CS = DVB == 8 ? 4 : DVB == 6 ? 3 : DVB, WK = DVB == 8 ? 3 : 4;
        const int64_t cus = compute_units(), blocks = BH * ((N + 31) / 32), pairs = BH * ((N + 63) / 64), quads = BH * ((N + 127) / 128);
        const int64_t shared = (CS * blocks + cus - 1) / cus * ((N + 32 * WK - 1) / (32 * WK) + 1) * (DVB + DVB / CS);
        const int64_t two = (pairs + cus - 1) / cus * ((N + 63) / 64 + 1) * 2 * DVB, one = (quads + cus - 1) / cus * ((N + 31) / 32) * 2 * DVB;
        if (5 * shared < 4 * two && 5 * shared < 4 * one) return launch_f32_t<DVB, 1, WK, CS>(Q, K, V, O, BH, N, d, scale, stream);
    }
    // (d > 128: the K and V tiles of four ranges do not fit the LDS)
    constexpr int most = DVB <= 4 ? 4 : 2;
    const int wk = key_ranges_f32(BH, N, most);
    // No keys to share, and 256-query strips whose waves are more than half busy: the bf16 instruction on operands in three
    // parts (16 heads of N = 4096, d = 128: 998 -> 527 us, eight, exactly half: 519 either way; 300 heads of N = 197, d = 64
    // 52 -> 42; forty of 700, d = 32, 43 % busy: 31 -> 32).
    if constexpr (DVB <= 4) {
        const int64_t cus = compute_units(), rounds = (BH * ((N + 255) / 256) + cus - 1) / cus;
        if (wk == 1 && BH * ((N + 31) / 32) * 2 > rounds * cus * 8 && split_takes_scale(scale))
            return DVB == 1 ? launch_attention_f32_split(Q, K, V, O, BH, N, d, scale, stream) : launch_attention_f32_turns(Q, K, V, O, BH, N, d, scale, stream);
    }
    if constexpr (most == 4)
        if (wk == 4) {
            // One-block workgroups for less than half, a third or a quarter of the compute units: the others share the columns.  us, one head of
            // 4096, d = 128 163 -> 140, d = 64 82 -> 71, of 2048, d = 128 80 -> 59, of 2000, d = 96 63 -> 47, two of 674, d = 128 33 -> 24, one of 300 19.5 -> 14.
            const int64_t cus = compute_units(), blocks = BH * ((N + 31) / 32);
            if constexpr (DVB == 4)
                if (4 * blocks <= cus) return launch_f32_t<DVB, 1, 4, 4>(Q, K, V, O, BH, N, d, scale, stream);
            if constexpr (DVB == 3)
                if (3 * blocks <= cus) return launch_f32_t<DVB, 1, 4, 3>(Q, K, V, O, BH, N, d, scale, stream);
            if constexpr (DVB % 2 == 0)
                if (2 * blocks <= cus) return launch_f32_t<DVB, 1, 4, 2>(Q, K, V, O, BH, N, d, scale, stream);
            return launch_f32_t<DVB, 1, 4>(Q, K, V, O, BH, N, d, scale, stream);
        }
    if (wk == 2) return launch_f32_t<DVB, 2, 2>(Q, K, V, O, BH, N, d, scale, stream);
    return launch_f32_t<DVB, 4, 1>(Q, K, V, O, BH, N, d, scale, stream);
}

}  // namespace

bool attention_f32_supported(int64_t BH, int64_t N, int64_t d)
{
    if (d < 4 || d > 256 || (d % 4) != 0) return false;
    if (N < 1 || N > ((int64_t)1 << 24)) return false;
    return BH * ((N + 31) / 32) <= (int64_t)0x7ffffff0;
}

hipError_t launch_attention_f32(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                float scale, hipStream_t stream)
{
    switch ((int)((d + 31) / 32)) {
    case 1: return launch_f32_ranges<1>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 2: return launch_f32_ranges<2>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 3: return launch_f32_ranges<3>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 4: return launch_f32_ranges<4>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 5: return launch_f32_ranges<5>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 6: return launch_f32_ranges<6>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 7: return launch_f32_ranges<7>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 8: return launch_f32_ranges<8>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
