// Attention output  O = softmax(scale * Q K^T) V  in bf16 for problems of a few heads: the keys of a query block are
// shared between the waves of a workgroup.
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the product
// with V is what the section "Limitations and future Directions" names as the next thing to fuse.  The
// max-subtracted softmax of the Softmax section, Eq. 1, is applied incrementally as in attention_kernels.hip.)
//
// One head of n = 4096 -- the paper's own problem size -- is 128 blocks of 32 queries.  A workgroup takes one block; its WK
// waves take the 32-key sub-tiles in turn (wave w has sub-tiles w, w + WK, ..), each with a reference exponent, a sum and
// output accumulators of its own, and the partial results are merged through LDS at the end.
//
// What bounds it: every compute unit reads the whole K of its head and its columns of V from the caches, 64 bytes per cycle at best
// (one head of N = 4096, d = 128: 11 us for K and half of V), with little arithmetic per byte; the waves wait 33 % of their life.
// Where the blocks leave compute units idle, several of them share a block's columns (CS below).  No byte is used by two waves, so a
// wave stages its own sub-tiles in an LDS area of its own and no barrier ties the waves together: while one requests and stores, the
// others compute.  K and V lie in LDS as they lie in memory; V is turned by the transposing LDS read.
#include "attention_common.h"
#include "launchers.h"

namespace attnw {
namespace {

// CS: workgroups that share the columns of V and O of a query block
template <int DVB, int WK, int CS>
struct RangesCfg {
    static constexpr int DB = DVB * 64;           // bytes of a row on chip
    static constexpr int CPR = DVB * 4;           // 16-byte chunks of it
    static constexpr int TILE = 32 * DB;          // a wave's sub-tile of K, and of V
    static constexpr int XFERS = TILE / 1024;     // wave-wide transfers of it
    static constexpr int OB = DVB / CS;           // 32-column blocks of V and O
    static constexpr int V_TILE = TILE / CS;
    static constexpr int SLOTS = 2 + OB * 16;     // merge: reference exponent, sum, output accumulators
    static constexpr int MERGE = WK * SLOTS * 256;
    static constexpr int LDS = WK * (TILE + V_TILE) > MERGE ? WK * (TILE + V_TILE) : MERGE;
    static_assert(DVB % CS == 0, "whole column blocks");
    static_assert(LDS <= 160 * 1024, "sub-tiles of all waves");
};

// DVB: 32-column blocks of a row, ceil(d / 32).  HALF: d is an odd multiple of 16 -- the last 16 columns on chip are
// copies of the row's first chunks, left out of the first contraction and not stored by the second.  rb: bytes of a row
// in memory.  Rows past N are read as row N - 1, weigh nothing and are not stored.
// V waits in registers for its place in LDS; K, whose place is free as soon as the scores are made, goes there directly (one head of
// N = 4096, d = 128 27.4 us, K through registers too 29.5; four waves instead of eight 38).
// q_base: the launch covers the queries from that one on.
// Where 32-query workgroups leave half of the compute units idle, CS of them share a block: each makes all scores, but reads and
// multiplies its share of the columns of V only, so that half or a quarter of V passes a compute unit's port.  No exchange between
// them.  (Sums: those of one workgroup of as many waves; d = 192 and 256 take eight and six waves here instead of four, which
// divides the keys differently.)
template <int DVB, bool HALF, int WK, int CS>
__global__ __launch_bounds__(64 * WK)
void attention_ranges_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                             uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t strips, uint32_t total, int q_base)
{
    using C = RangesCfg<DVB, WK, CS>;
    using L = RowLayout<DVB>;
    using LV = RowLayout<DVB / CS>;
    constexpr int OB = C::OB, DBV = OB * 64, CPRV = OB * 4, V_TILE = C::V_TILE, V_XFERS = V_TILE / 1024;
    static_assert(CS == 1 || !HALF, "columns are shared in whole blocks");
    constexpr int DB = C::DB, CPR = C::CPR, TILE = C::TILE, XFERS = C::XFERS;
    constexpr int rb = DB - (HALF ? 32 : 0);
    constexpr int G = rb / 32;                    // 32-byte contraction groups of a row
    static_assert(WK * TILE <= kDirectLds, "reach of direct transfers");

    __shared__ __align__(1024) char lds[C::LDS];

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t block = logical / CS;
    const int col0 = (int)(logical % CS) * DBV;   // this workgroup's first byte of a row of V and O
    const uint32_t bh = block / strips;
    const uint32_t strip = block - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    char* const k_lds = lds + wave * TILE;
    char* const v_lds = lds + WK * TILE + wave * V_TILE;

    const char* Qh = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * rb;
    const char* Kh = reinterpret_cast<const char*>(K) + (int64_t)bh * N * rb;
    const char* Vh = reinterpret_cast<const char*>(V) + (int64_t)bh * N * rb;
    char* Oh = reinterpret_cast<char*>(O) + (int64_t)bh * N * rb;
    const int q0 = q_base + strip * 32;

    // ---- sub-tile transfers: transfer j moves chunks 64 j .. 64 j + 63 of the sub-tile --------------------------------------
    // (a lane's chunk number is its place in LDS; which chunk of the row it reads follows from the swizzle)
    auto offset = [&](int j, int rows, bool v) __attribute__((always_inline)) {   // rows: last valid row of the sub-tile
        const int s = j * 64 + lane;
        const int key = v ? s / CPRV : s / CPR;
        int ch = v ? (s - key * CPRV) ^ (LV::v_block(key) * 4) : (s - key * CPR) ^ L::k_chunk(key);
        if (HALF && ch * 16 >= rb) ch -= rb / 16;
        return (uint32_t)(min(key, rows) * rb + ch * 16);
    };
    uint32_t k_off[XFERS], v_off[V_XFERS];
#pragma unroll
    for (int j = 0; j < XFERS; ++j) k_off[j] = offset(j, 31, false);
#pragma unroll
    for (int j = 0; j < V_XFERS; ++j) v_off[j] = offset(j, 31, true);
    u32x4 vreg[V_XFERS];
    const uint32_t k_base = lds_offset_of(k_lds);
    auto k_load = [&](int t) __attribute__((always_inline)) {
        const char* base = Kh + (int64_t)t * 32 * rb;
        const int rows = N - 1 - t * 32;
#pragma unroll
        for (int j = 0; j < XFERS; ++j)
            dma16_untracked(base, rows >= 31 ? k_off[j] : offset(j, rows, false), k_base + j * 1024);
    };
    auto v_load = [&](int t) __attribute__((always_inline)) {
        const char* base = Vh + (int64_t)t * 32 * rb + col0;
        const int rows = N - 1 - t * 32;
#pragma unroll
        for (int j = 0; j < V_XFERS; ++j)
            vreg[j] = *reinterpret_cast<const u32x4*>(base + (rows >= 31 ? v_off[j] : offset(j, rows, true)));
    };
    const int n_tiles = (N + 31) / 32;
    if (wave < n_tiles) {
        k_load(wave);
        v_load(wave);
    }

    // ---- Q fragments (a negative scale negates Q) -------------------------------------------------------------------
    u32x4 qf[G];
    {
        const char* qrow = Qh + (int64_t)min(q0 + l32, N - 1) * rb + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(qrow + g * 32) ^ sign_flip;
    }

    // ---- per-lane places of the operand fragments ------------------------------------------------------------------------
    constexpr int KPERIOD = L::KPERIOD, VPERIOD = LV::VPERIOD;
    const char* const krow = k_lds + l32 * DB;
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((2 * g + half) ^ L::k_chunk(l32)) * 16;
    const int vkey = 4 * half + ((lane & 15) >> 2);            // a lane's row of the 8-key group that it reads
    const char* const vrow = v_lds + vkey * DBV + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    int voff[VPERIOD];
#pragma unroll
    for (int b = 0; b < VPERIOD; ++b) voff[b] = (b ^ LV::v_block(vkey)) * 64;

    f32x16 oacc[OB];
#pragma unroll
    for (int b = 0; b < OB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
    float mb_run = kNegBig, l_run = 0.0f;
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent

    for (int t = wave; t < n_tiles; t += WK) {
        const bool more = t + WK < n_tiles;
        wait_vmem();                              // K and V of this sub-tile have arrived
#pragma unroll
        for (int j = 0; j < V_XFERS; ++j) *reinterpret_cast<u32x4*>(v_lds + j * 1024 + lane * 16) = vreg[j];
        if (more) v_load(t + WK);
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g)
            Mma<uint16_t>::run(s, *reinterpret_cast<const u32x4*>(krow + (g / KPERIOD) * KPERIOD * 32 + koff[g % KPERIOD]), qf[g]);
        if (more) {
            wait_lds();                           // the K fragments have left their place
            k_load(t + WK);
        }
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        const float m = half_wave_max(fmaxf(tm, s[15]));   // (keys past the end are copies of key N-1: no new maximum)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(m * c > mb_run + kLazy) != 0, 0)) {
            const float mb_new = fmaxf(mb_run, reference_exponent(m, c));
            const float alpha = fast_exp2(mb_run - mb_new);    // exactly 1 for lanes whose exponent stands
            l_run *= alpha;
#pragma unroll
            for (int b = 0; b < OB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[b][r] *= alpha;
            mb_run = mb_new;
        }
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mb_run));
        if (t * 32 + 32 > N) {                    // keys past the end weigh nothing
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (t * 32 + 4 * half + 8 * (r / 4) + (r % 4) >= N) p[r] = 0.0f;
        }
        float sum = p[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) sum += p[r];
        l_run += sum;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            u32x4 pw;
#pragma unroll
            for (int i = 0; i < 4; ++i) pw[i] = pack_bf16x2(p[8 * m + 2 * i], p[8 * m + 2 * i + 1]);
#pragma unroll
            for (int b = 0; b < OB; ++b) {
                const char* v = vrow + 16 * m * DBV + (b / VPERIOD) * VPERIOD * 64 + voff[b % VPERIOD];
                Mma<uint16_t>::run(oacc[b], u32x4_of(lds_read_tr16(v), lds_read_tr16(v + 8 * DBV)), pw);
            }
        }
    }
    __syncthreads();

    // ---- merge the WK partial results of a query block, normalise, round once, store ----------------------------------------
    // (the sub-tiles are free after the barrier.  With M the largest of the WK exponents, partial j counts
    // with the factor 2^(m_j - M): exactly 1 for the largest, 0 for a range without keys)
    constexpr int SLOTS = C::SLOTS;
    float* const part = reinterpret_cast<float*>(lds);
    float* const mine = part + wave * SLOTS * 64 + lane;
    mine[0] = mb_run;
    mine[64] = l_run;
#pragma unroll
    for (int b = 0; b < OB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(2 + b * 16 + r) * 64] = oacc[b][r];
    __syncthreads();
    const float* const grp = part + lane;
    float f[WK], top = grp[0], l_sum = 0.0f;
#pragma unroll
    for (int j = 1; j < WK; ++j) top = fmaxf(top, grp[j * SLOTS * 64]);
#pragma unroll
    for (int j = 0; j < WK; ++j) {
        f[j] = fast_exp2(grp[j * SLOTS * 64] - top);
        l_sum = __builtin_fmaf(f[j], grp[j * SLOTS * 64 + 64], l_sum);
    }
    const float inv = 1.0f / half_wave_sum(l_sum);
    if (q0 + l32 >= N) return;
    // a run is 4 consecutive output columns of the lane's query; wave w takes runs w, w + WK, ..
    char* const orow = Oh + (int64_t)(q0 + l32) * rb + col0 + half * 8;
#pragma unroll
    for (int i = 0; i < OB * 4 / WK + (OB * 4 % WK != 0); ++i) {
        const int run = wave + i * WK;
        if (run * 16 >= (CS == 1 ? rb : DBV)) break;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = 0.0f;
#pragma unroll
            for (int j = 0; j < WK; ++j) o[e] = __builtin_fmaf(f[j], grp[(j * SLOTS + 2 + run * 4 + e) * 64], o[e]);
        }
        const u32x2 w = {pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv)};
        *reinterpret_cast<u32x2*>(orow + run * 16) = w;
    }
}

template <int DVB, bool HALF, int WK, int CS = 1>
hipError_t launch_ranges_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, int q_base, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((N - q_base + 31) / 32);
    return launch_by_heads(BH, strips * CS, 64 * WK, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * (DVB * 32 - (HALF ? 16 : 0));
        const uint32_t total = (uint32_t)heads * strips * CS, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_ranges_kernel<DVB, HALF, WK, CS>), dim3(grid), dim3(64 * WK), 0, stream,
                           static_cast<const uint16_t*>(Q) + at, static_cast<const uint16_t*>(K) + at, static_cast<const uint16_t*>(V) + at,
                           static_cast<uint16_t*>(O) + at, N, fabsf(scale) * kLog2e, scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u, strips,
                           total, q_base);
        return hipGetLastError();
    });
}

template <int DVB, bool HALF>
hipError_t launch_ranges(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, int q_base, hipStream_t stream)
{
    // Waves per block.  One workgroup per compute unit: eight (d > 128: four, the sub-tiles of eight do not fit the LDS), fewer
    // where there are not as many sub-tiles (32 heads of N = 256, d = 128: eight 7.6 us, four 7.1).  More workgroups than
    // that, and a short sweep: two waves, so that the beginning and the merge of one workgroup are covered by the sweep
    // of another (d = 128: 32 heads of N = 512 16.7 -> 13.7, 64 of 256 14.1 -> 9.5, 250 of 80 11.9 -> 7.0; sixteen of
    // 1024 no different, twelve of 2048 50 -> 74).  Four waves up to twice as many workgroups where a compute unit holds two such
    // (d <= 96: 20 heads of N = 512, us, two / four waves: d = 32 7.2 / 5.2, 64 10.0 / 7.8, 96 11.7 / 9.1; 40 of 357, d = 64 8.5 / 7.1; 128
    // of 128 alike; beyond twice: 100 heads of N = 300, d = 64 8.9 / 10.4).
    const int64_t blocks = BH * ((N - q_base + 31) / 32), cus = compute_units();
    // Workgroups per block (CS): what a round of workgroups costs against one of undivided columns, in per cent, times the rounds.  One head
    // of N = 4096, us: d = 64 16.9 -> 15.2, 128 27.7 -> 24.4, 192 57.7 -> 35.1, 256 80 -> 45.7 (their smaller tiles also leave room for eight and six
    // waves instead of four); of 1024: d = 96 8.8 -> 6.9, 128 11.0 -> 8.4, 256 25.0 -> 13.4; of 300: d = 256 13.4 -> 8.5.
    if constexpr (!HALF && (DVB % 2 == 0 || DVB == 3)) {
        auto cost = [&](int cs, int percent) { return (cs * blocks + cus - 1) / cus * percent; };
        if (N > (blocks <= cus ? 256 : 512)) {
            const int64_t whole = cost(1, 100);
            if constexpr (DVB == 8) {
                if (cost(4, 52) < whole && cost(4, 52) <= cost(2, 57)) return launch_ranges_t<DVB, HALF, 8, 4>(Q, K, V, O, BH, N, scale, q_base, stream);
                if (cost(2, 57) < whole) return launch_ranges_t<DVB, HALF, 6, 2>(Q, K, V, O, BH, N, scale, q_base, stream);
            } else if constexpr (DVB == 6) {
                if (cost(2, 61) < whole) return launch_ranges_t<DVB, HALF, 8, 2>(Q, K, V, O, BH, N, scale, q_base, stream);
            } else if constexpr (DVB == 4) {
                if (cost(4, 78) < whole) return launch_ranges_t<DVB, HALF, 8, 4>(Q, K, V, O, BH, N, scale, q_base, stream);
                if (cost(2, 86) < whole) return launch_ranges_t<DVB, HALF, 8, 2>(Q, K, V, O, BH, N, scale, q_base, stream);
            } else {
                if (cost(DVB, 88) < whole) return launch_ranges_t<DVB, HALF, 8, DVB>(Q, K, V, O, BH, N, scale, q_base, stream);
            }
        }
    }
    if (DVB <= 3 && N > 64 && N <= 512 && blocks > cus && blocks <= 2 * cus)
        return launch_ranges_t<DVB, HALF, 4>(Q, K, V, O, BH, N, scale, q_base, stream);
    if (N <= 64 || (blocks > cus && N <= 512)) return launch_ranges_t<DVB, HALF, 2>(Q, K, V, O, BH, N, scale, q_base, stream);
    if (DVB > 4 || N <= 256) return launch_ranges_t<DVB, HALF, 4>(Q, K, V, O, BH, N, scale, q_base, stream);
    return launch_ranges_t<DVB, HALF, DVB <= 4 ? 8 : 4>(Q, K, V, O, BH, N, scale, q_base, stream);
}

}  // namespace

// A round of 32-query workgroups (one per compute unit) against a round of the 256-query workgroups of the kernels that
// give every wave all keys.  N = 4096, us: d = 128 30 a round (one head 27) against 110; d = 64 15 against 75; d = 256
// 80 against 190.  Below 1024 keys a round of the larger workgroups is worth fewer: three rounds, d = 128: 226 heads of N = 85 11.5
// against 6.8, 150 of N = 150 14.0 against 10.2, 100 of N = 200 15.9 against 12.7, 48 of N = 512 24 against 21.6 (d = 80 up to 256
// keys: 6.0 / 5.3, 7.2 / 7.6, 8.1 / 9.0); 100 heads of N = 65, d = 160 (two) 7.9 against 7.0.
bool prefers_attention_ranges(int64_t BH, int64_t N, int64_t d)
{
    const int64_t cus = compute_units();
    const int64_t blocks = (BH * ((N + 31) / 32) + cus - 1) / cus, strips = (BH * ((N + 255) / 256) + cus - 1) / cus;
    if (d <= 64) return blocks <= 4 * strips;
    if (d <= 128) return blocks <= (N >= 1024 || (N <= 256 && d <= 96) ? 3 : 2) * strips;
    return blocks <= (N <= 128 ? 1 : 2) * strips;
}

hipError_t launch_attention_ranges(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                   float scale, int q_base, hipStream_t stream)
{
    switch ((int)(d / 16)) {
    case 1: return launch_ranges<1, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 2: return launch_ranges<1, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 3: return launch_ranges<2, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 4: return launch_ranges<2, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 5: return launch_ranges<3, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 6: return launch_ranges<3, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 7: return launch_ranges<4, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 8: return launch_ranges<4, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 9: return launch_ranges<5, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 10: return launch_ranges<5, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 11: return launch_ranges<6, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 12: return launch_ranges<6, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 13: return launch_ranges<7, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 14: return launch_ranges<7, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 15: return launch_ranges<8, true>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    case 16: return launch_ranges<8, false>(Q, K, V, O, BH, (int)N, scale, q_base, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
