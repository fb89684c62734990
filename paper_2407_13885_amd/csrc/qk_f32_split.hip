// Fused attention weights  P = softmax(scale * Q K^T)  in fp32 for many strips (d a multiple of 4 up to 128, N a multiple
// of 4): the two sweeps of qk_kernel with the contraction on the bf16 matrix instruction, operands as three bf16 parts
// (split_f32.h).
//
// (Paper: the fused kernel of the section "Fused Matrix Multiply + Scaling + Softmax"; row maxima and sums of the Softmax
// section, Eq. 1, gathered in sweep one, the scores computed again in sweep two, scaled, exponentiated and written.)
//
// What bounds it: with the fp32 instruction the two sweeps filled its pipe (16 heads of N = 2048, d = 64: 110 of 157 us); the
// six bf16 products take 3/8 of its cycles, which brings the contraction near the time that the weights take to
// HBM (268 MB, 42 us).  Eight waves: four query blocks of 32 x two key ranges of one or two
// 32-key sub-tiles per tile.  A thread loads
// 8 elements of a K row, splits them and writes a 16-byte chunk to each of the three planes of the tile, once for 128
// queries.  Weights leave through a staging area of the wave as whole 128-byte pieces of rows.  Measured, 16 heads of N = 2048: d = 64
// 158 -> 119 us (2.4 TB/s), 128 278 -> 199, 32 101 -> 89; what is left: splitting, products and softmax of a tile one after the other
// in all eight waves (matrix pipe 43 % of SIMD cycles, vector ALU 42 %, both 8 %, waves waiting 33 % of their life).
#include "attention_common.h"
#include "launchers.h"
#include "split_f32.h"

namespace attnw {
namespace {

// DVB: 32-column blocks of a row, ceil(d / 32); columns past d are zeros on chip.  Rows past N are read as row N - 1,
// weigh nothing and are not stored.
template <int DVB>
__global__ __launch_bounds__(512)
void qk_f32_split_kernel(const float* __restrict__ Q, const float* __restrict__ K, float* __restrict__ P, int N, int d, float c,
                         float q_sign, uint32_t strips, uint32_t total)
{
    using L = RowLayout<DVB>;
    constexpr int NW = 8, WK = 2;
    constexpr int SUBS = DVB <= 2 ? 2 : 1;        // sub-tiles of a wave per tile (LDS)
    constexpr int BN = 32 * WK * SUBS;
    constexpr int DB = DVB * 64;                  // bytes of a row of a plane
    constexpr int CPR = DVB * 4;                  // 16-byte chunks of it
    constexpr int PLANE = BN * DB;
    constexpr int BUF_BYTES = 3 * PLANE;          // hi, mid, lo
    constexpr int G = DVB * 2;                    // 16-column contraction groups
    constexpr int CHUNKS = BN * CPR;              // chunks of a plane
    constexpr int SLOTS = (CHUNKS + NW * 64 - 1) / (NW * 64);
    constexpr int ST_PITCH = 32 * 4 + 16;         // staged row: 32 weights, padded against bank conflicts
    constexpr int ST_BYTES = 32 * ST_PITCH;

    __shared__ __align__(1024) char lds[2 * BUF_BYTES + NW * ST_BYTES];
    __shared__ float stat_lds[NW * 64];

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int wq = wave / WK, wk = wave % WK;
    const float* Qh = Q + (int64_t)bh * N * d;
    const float* Kh = K + (int64_t)bh * N * d;
    float* Ph = P + (int64_t)bh * N * N;
    const int q0 = strip * 128 + wq * 32;
    char* const stage = lds + 2 * BUF_BYTES + wave * ST_BYTES;

    // (q_sign: a negative scale negates Q)
    const float* const qrow = Qh + (int64_t)min(q0 + l32, N - 1) * d;
    Split8 qf[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int col = g * 16 + half * 8;
        qf[g] = split_row8(load_row8(qrow, col, d), col, d, q_sign * kSplitUp);
    }

    // ---- K tiles: slot s of a tile is its chunk s ---------------------------------------------------------------------------
    // (every workgroup starts its sweeps at another tile: in step, the rows that they write at one moment lie on the
    // same few memory channels)
    const int n_tiles = (N + BN - 1) / BN;
    const int rot = (int)((logical * 7u) % (uint32_t)n_tiles);
    auto tile_at = [&](int j) __attribute__((always_inline)) {   // j-th tile of the two sweeps
        int t = (j >= n_tiles ? j - n_tiles : j) + rot;
        return t >= n_tiles ? t - n_tiles : t;
    };
    Row8 reg[SLOTS];
    auto load = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < SLOTS; ++j)
            if (CHUNKS % (NW * 64) == 0 || (wave + NW * j) * 64 < CHUNKS) {   // (wave-uniform)
                const int s = (wave + NW * j) * 64 + lane;
                const int key = s / CPR;
                reg[j] = load_row8(Kh + (int64_t)min(t * BN + key, N - 1) * d, (s - key * CPR) * 8, d);
            }
    };
    auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < SLOTS; ++j)
            if (CHUNKS % (NW * 64) == 0 || (wave + NW * j) * 64 < CHUNKS) {
                const int s = (wave + NW * j) * 64 + lane;
                const int key = s / CPR, ch = s - key * CPR;
                const Split8 x = split_row8(reg[j], ch * 8, d);
                char* to = lds + buf * BUF_BYTES + key * DB + (ch ^ L::k_chunk(key)) * 16;
                *reinterpret_cast<u32x4*>(to) = x.hi;
                *reinterpret_cast<u32x4*>(to + PLANE) = x.mid;
                *reinterpret_cast<u32x4*>(to + 2 * PLANE) = x.lo;
            }
    };
    constexpr int KPERIOD = L::KPERIOD;
    const char* const krow = lds + (wk * 32 + l32) * DB;
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((2 * g + half) ^ L::k_chunk(l32)) * 16;
    auto scores = [&](int buf, int u) __attribute__((always_inline)) {
        f32x16 s, rest;                           // (two sums: the matrix instructions of one need not wait for each other's results)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = rest[r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const char* k = krow + buf * BUF_BYTES + u * WK * 32 * DB + (g / KPERIOD) * KPERIOD * 32 + koff[g % KPERIOD];
            const Split8 kf = {*reinterpret_cast<const u32x4*>(k), *reinterpret_cast<const u32x4*>(k + PLANE),
                               *reinterpret_cast<const u32x4*>(k + 2 * PLANE)};
            mma_split(s, rest, kf, qf[g]);
        }
        return s + rest;
    };

    const float c_parts = c * kSplitDown;         // for scores of operands in parts
    // running maximum and sum of exponentials over the lane's keys (accumulator r is key key0 + 4 half + 8 (r / 4) + r % 4)
    // In parts scores beyond 2^79 either way (2^127 with the factor of the operands) make the sum NaN: from 2^80 on they are infinite
    // where fp32 holds them, and differences of two of them overflow.
    // (The maximum over no keys is the lowest number there is: scores in parts carry a factor of 2^48, and behind a higher one the
    // exponentials of scores below it come out small, imprecise or zero.)
    float m_run = -0x1.fffffep127f, l_run = 0.0f;
    auto fold = [&](const f32x16& s, float c, int key0, auto partsc) __attribute__((always_inline)) {
        float low = 0.0f;
        if constexpr (decltype(partsc)::value != 0) {
            low = fminf(s[0], s[1]);
#pragma unroll
            for (int r = 2; r < 16; r += 2) low = min3(low, s[r], s[r + 1]);
        }
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        const float mn = fmaxf(m_run, fmaxf(tm, s[15]));       // (keys past the end are copies of key N-1: no new maximum)
        float e[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = fast_exp2((s[r] - mn) * c);
        if (key0 + 32 > N) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + 4 * half + 8 * (r / 4) + (r % 4) >= N) e[r] = 0.0f;
        }
        float sum = e[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) sum += e[r];
        l_run = l_run * fast_exp2((m_run - mn) * c) + sum;
        if (decltype(partsc)::value != 0 && low < -0x1p127f) l_run = __builtin_nanf("");
        m_run = mn;
    };
    auto merge = [&](float m, float l, float c) __attribute__((always_inline)) {   // statistics of other keys of the same query
        const float mn = fmaxf(m_run, m);
        l_run = l_run * fast_exp2((m_run - mn) * c) + l * fast_exp2((m - mn) * c);
        m_run = mn;
    };

    // ---- sweep one: while tile j is computed, tile j + 1 is split into the other buffer and tile j + 2 is under way ----------
    load(tile_at(0));
    store(0);
    load(tile_at(1));
    __syncthreads();
    auto stage_next = [&](int j, int buf) __attribute__((always_inline)) {
        if (j + 1 < 2 * n_tiles) {
            store(buf ^ 1);
            if (j + 2 < 2 * n_tiles) load(tile_at(j + 2));
        }
    };
    for_tiles(0, 0, n_tiles, [&](int j, auto bufc) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        stage_next(j, BUF);
#pragma unroll
        for (int u = 0; u < SUBS; ++u) {
            const int key0 = tile_at(j) * BN + (u * WK + wk) * 32;
            if (q0 < N && key0 < N) fold(scores(BUF, u), c_parts, key0, IC<1>{});
        }
        __syncthreads();
    });
    if (m_run > 0x1p127f) l_run = __builtin_nanf("");
    merge(__shfl_xor(m_run, 32, 64), __shfl_xor(l_run, 32, 64), c_parts);
    if (half == 0) {
        stat_lds[wave * 64 + l32] = m_run;
        stat_lds[wave * 64 + 32 + l32] = l_run;
    }
    __syncthreads();
    merge(stat_lds[(wave ^ 1) * 64 + l32], stat_lds[(wave ^ 1) * 64 + 32 + l32], c_parts);
    // infinities, NaN and overflows: what the parts make of them is not what fp32 does (the end of the kernel deals with them)
    const bool exact = __builtin_amdgcn_ballot_w64(!(l_run > 0.0f && l_run < __builtin_inff())) == 0;

    // ---- sweep two -----------------------------------------------------------------------------------------------------------
    const float bias = fast_log2(l_run);
    const bool rows_full = q0 + 32 <= N, lines = N % 32 == 0;
    float* const out_lane = Ph + (int64_t)(q0 + lane / 8) * N + (lane % 8) * 4;
    auto sweep_two = [&](int j, auto bufc) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        stage_next(j, BUF);
#pragma unroll
        for (int u = 0; u < SUBS; ++u) {
            const int key0 = tile_at(j) * BN + (u * WK + wk) * 32;
            if (!exact || q0 >= N || key0 >= N) continue;
            const f32x16 s = scores(BUF, u);
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                f32x4 p;
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = fast_exp2(__builtin_fmaf(s[4 * r4 + i] - m_run, c_parts, -bias));
                *reinterpret_cast<f32x4*>(stage + l32 * ST_PITCH + (8 * r4 + 4 * half) * 4) = p;
            }
            const bool full = rows_full && key0 + 32 <= N;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(stage + (it * 8 + lane / 8) * ST_PITCH + (lane % 8) * 16);
                f32x4* const to = reinterpret_cast<f32x4*>(out_lane + (int64_t)(it * 8) * N + key0);
                if (full && lines) __builtin_nontemporal_store(v, to);      // whole lines past the caches: K stays in L2
                else if (full || (q0 + it * 8 + lane / 8 < N && key0 + (lane % 8) * 4 < N)) *to = v;
            }
        }
        __syncthreads();
    };
    for_tiles(n_tiles, n_tiles & 1, 2 * n_tiles, sweep_two);
    if (exact || q0 >= N) return;

    // ---- the wave's part of P again on the fp32 instruction, operands straight from memory (rare) ------------------------------
    auto scores_f32 = [&](int key0) __attribute__((always_inline)) {
        const float* kr = Kh + (int64_t)min(key0 + l32, N - 1) * d;
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
        for (int col = 0; col < d; col += 4) {                 // columns col, col + 1, then col + 2, col + 3
            const f32x4 a = *reinterpret_cast<const f32x4*>(kr + col), b = *reinterpret_cast<const f32x4*>(qrow + col) * q_sign;
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? a[1] : a[0], half ? b[1] : b[0], s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? a[3] : a[2], half ? b[3] : b[2], s, 0, 0, 0);
        }
        return s;
    };
    m_run = kNegBig;
    l_run = 0.0f;
    for (int key0 = 0; key0 < N; key0 += 32) fold(scores_f32(key0), c, key0, IC<0>{});
    merge(__shfl_xor(m_run, 32, 64), __shfl_xor(l_run, 32, 64), c);
    const float bias_f32 = fast_log2(l_run);
    for (int key0 = wk * 32; key0 < N; key0 += WK * 32) {
        const f32x16 s = scores_f32(key0);
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            f32x4 p;
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = fast_exp2(__builtin_fmaf(s[4 * r4 + i] - m_run, c, -bias_f32));
            const int key = key0 + 8 * r4 + 4 * half;          // (N is a multiple of 4: a run is inside or outside)
            if (q0 + l32 < N && key < N) *reinterpret_cast<f32x4*>(Ph + (int64_t)(q0 + l32) * N + key) = p;
        }
    }
}

template <int DVB>
hipError_t launch_split_t(const void* Q, const void* K, void* P, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((N + 127) / 128);
    return launch_by_heads(BH, strips, 512, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * d;
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((qk_f32_split_kernel<DVB>), dim3(grid), dim3(512), 0, stream, static_cast<const float*>(Q) + at,
                           static_cast<const float*>(K) + at, static_cast<float*>(P) + first * N * N, N, d, fabsf(scale) * kLog2e,
                           scale < 0.0f ? -1.0f : 1.0f, strips, total);
        return hipGetLastError();
    });
}

}  // namespace

hipError_t launch_qk_f32_split(const void* Q, const void* K, void* P, int64_t BH, int64_t N, int64_t d, float scale, hipStream_t stream)
{
    switch ((int)((d + 31) / 32)) {
    case 1: return launch_split_t<1>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    case 2: return launch_split_t<2>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    case 3: return launch_split_t<3>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    case 4: return launch_split_t<4>(Q, K, P, BH, (int)N, (int)d, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
