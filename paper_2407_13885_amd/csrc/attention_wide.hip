// Attention output  O = softmax(scale * Q K^T) V  for wide bf16 heads: d a multiple of 16, 128 < d <= 256, any N.
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the product
// with V is what the section "Limitations and future Directions" names as the next thing to fuse.  The
// max-subtracted softmax of the Softmax section, Eq. 1, is applied incrementally as in the kernel for d <= 128.)
//
// What bounds it: the LDS port, as in the kernel for d <= 128 (every matrix instruction takes one 1 KiB operand fragment
// from LDS), with half as much softmax per matrix instruction.  A wave owns 32 queries: 128 accumulators and up to 64
// registers of Q fragments leave no room for a second query block at two waves per SIMD.
//
// A workgroup is WQ query blocks of 32 x WK key ranges; a tile is 32 keys per range.  K and V lie in LDS as they lie in
// memory, chunks swizzled: V is turned by the transposing LDS read (ds_read_b64_tr_b16: 4 keys x 16 columns, a lane gets
// the four keys of its column), so both tiles travel global -> LDS directly, without registers or a scatter.
// Measured, 16 heads of N = 4096, against one wave per workgroup with operands straight from the caches: d = 256 928 ->
// 238 us (1157 TFLOP/s), 192 700 -> 185, 144 633 -> 157; one head of N = 4096, d = 256 301 -> 105.
//   WK = 1, WQ = 8   the problem fills the chip: K and V double buffered (4 x 16 KiB: what the direct transfers can
//                    address), one barrier per tile of 32 keys.
//   WK = 4, WQ = 1   few heads: 32 queries per workgroup, a wave takes one 32-key sub-tile of every 128-key tile; one
//                    buffer each, K lands while V is multiplied, V waits in registers while the scores are made.  The
//                    partial results of the ranges are merged through LDS at the end.
#include "launchers.h"
#include "qk_common.h"

namespace attnw {
namespace {

__device__ __forceinline__ float half_max_w(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
#else
    return x;
#endif
}
__device__ __forceinline__ float half_sum_w(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
#else
    return x;
#endif
}

template <int DVB, int WQ, int WK>
struct WideCfg {
    static constexpr int NW = WQ * WK;
    static constexpr int BM = 32 * WQ;
    static constexpr int BN = 32 * WK;
    static constexpr int DB = DVB * 64;           // bytes of a row on chip
    static constexpr int CPR = DVB * 4;           // 16-byte chunks of it
    static constexpr int TILE = BN * DB;
    static constexpr int XFERS = TILE / 1024;     // wave-wide transfers per tile
    static constexpr int STAGES = WK == 1 ? 2 : 1;
    static constexpr int SLOTS = 2 + DVB * 16;    // merge: reference exponent, sum, output accumulators
    static constexpr int MERGE = WK > 1 ? NW * SLOTS * 256 : 0;
    static constexpr int TILES = 2 * STAGES * TILE;
    static constexpr int LDS = TILES > MERGE ? TILES : MERGE;
};

// Chunk swizzles (applied to the chunk index within a row; involutions that stay inside the row).  K fragments read one
// chunk of 32 consecutive rows: 16 rows have to hit 16 different chunk positions modulo 256 bytes.  The transposing read
// of V takes 64 bytes of four consecutive rows: those four have to lie in different quarters of 256 bytes.
template <int DVB> __device__ __forceinline__ constexpr int k_swz(int key)
{
    return DVB == 8 ? key & 15 : DVB == 6 ? (key >> 1) & 7 : (key >> 2) & 3;
}
template <int DVB> __device__ __forceinline__ constexpr int v_swz(int key)   // in units of 4 chunks
{
    return DVB == 8 ? key & 3 : DVB == 6 ? (key >> 1) & 1 : 0;
}

// DVB: 32-column blocks of a row, ceil(d / 32).  HALF: d is an odd multiple of 16 -- the last 16 columns on chip are
// copies of the row's first chunks, left out of the first contraction and not stored by the second.  rb: bytes of a row
// in memory.  Rows past N are read as row N - 1, weigh nothing and are not stored.
template <int DVB, bool HALF, int WQ, int WK>
__global__ __launch_bounds__(64 * WQ * WK)
void attention_wide_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                           uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t strips, uint32_t total)
{
    using C = WideCfg<DVB, WQ, WK>;
    constexpr int NW = C::NW, DB = C::DB, CPR = C::CPR, BN = C::BN, TILE = C::TILE, XFERS = C::XFERS;
    constexpr int rb = DB - (HALF ? 32 : 0);
    constexpr int G = rb / 32;                    // 32-byte contraction groups of a row
    constexpr bool V_REGS = WK > 1;               // V through registers: its tile lies past what the transfers address
    constexpr int V_CHUNKS = V_REGS ? XFERS / NW : 1;
    static_assert((V_REGS ? TILE : 4 * TILE) <= 65536, "direct transfers address the first 64 KiB of LDS");
    static_assert(!V_REGS || XFERS % NW == 0, "V tile load shape");

    __shared__ __align__(1024) char lds[C::LDS];
    char* const k_lds = lds;
    char* const v_lds = lds + C::STAGES * TILE;

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;
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

    // ---- Q fragments (a negative scale negates Q) -------------------------------------------------------------------
    u32x4 qf[G];
    {
        const char* qrow = Qh + (int64_t)min(q0 + l32, N - 1) * rb + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(qrow + g * 32) ^ sign_flip;
    }

    // ---- tile transfers: transfer i of a tile moves its chunks 64 i .. 64 i + 63, wave w takes i = w, w + NW, .. --------
    // With many transfers per wave a lane's byte offsets within a tile are kept, and worked out anew for the last tile only,
    // where rows past the end exist.
    constexpr int XW = (XFERS + NW - 1) / NW;     // transfers per wave and tile
    const int last_row = N - 1;
    auto offset = [&](int j, int rows, int swz_v) __attribute__((always_inline)) {   // rows: last valid row of the tile
        const int s = (wave + NW * j) * 64 + lane;
        const int key = s / CPR;
        int ch = (s - key * CPR) ^ (swz_v ? v_swz<DVB>(key) * 4 : k_swz<DVB>(key));
        if (HALF && ch * 16 >= rb) ch -= rb / 16;
        return (uint32_t)(min(key, rows) * rb + ch * 16);
    };
    uint32_t k_off[XW], v_off[XW];
#pragma unroll
    for (int j = 0; j < XW; ++j) {
        k_off[j] = offset(j, BN, 0);
        v_off[j] = offset(j, BN, 1);
    }
    // f(j, base, offset) for every transfer j of this wave
    auto transfers = [&](const char* head, int t, const uint32_t* off, int swz_v, auto&& f) __attribute__((always_inline)) {
        const char* base = head + (int64_t)t * BN * rb;
        const bool ragged = WK == 1 || (t + 1) * BN > N;   // (few transfers: three instructions each, and no branch)
#pragma unroll
        for (int j = 0; j < XW; ++j)
            if (XFERS % NW == 0 || wave + NW * j < XFERS) {
                if (ragged) f(j, base, offset(j, last_row - t * BN, swz_v));
                else f(j, base, off[j]);
            }
    };
    const uint32_t k_base = lds_offset_of(k_lds), v_base = lds_offset_of(v_lds);
    auto k_issue = [&](int t, int buf) __attribute__((always_inline)) {
        transfers(Kh, t, k_off, 0, [&](int j, const char* base, uint32_t off) __attribute__((always_inline)) {
            dma16_untracked(base, off, k_base + buf * TILE + (wave + NW * j) * 1024);
        });
    };
    auto v_issue = [&](int t, int buf) __attribute__((always_inline)) {
        transfers(Vh, t, v_off, 1, [&](int j, const char* base, uint32_t off) __attribute__((always_inline)) {
            dma16_untracked(base, off, v_base + buf * TILE + (wave + NW * j) * 1024);
        });
    };
    u32x4 vreg[V_CHUNKS];
    auto v_load = [&](int t) __attribute__((always_inline)) {
        transfers(Vh, t, v_off, 1, [&](int j, const char* base, uint32_t off) __attribute__((always_inline)) {
            if constexpr (V_REGS) vreg[j] = *reinterpret_cast<const u32x4*>(base + off);
        });
    };
    auto v_store = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < V_CHUNKS; ++j) *reinterpret_cast<u32x4*>(v_lds + (wave + NW * j) * 1024 + lane * 16) = vreg[j];
    };

    // ---- per-lane places of the operand fragments ------------------------------------------------------------------------
    const char* const krow = k_lds + (wk * 32 + l32) * DB;
    constexpr int KPERIOD = DVB == 8 ? 8 : DVB == 6 ? 4 : 2;   // groups after which the swizzled low bits of a chunk repeat
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((2 * g + half) ^ k_swz<DVB>(l32)) * 16;
    const int vkey = 4 * half + ((lane & 15) >> 2);            // a lane's row of the 8-key group that it reads
    const char* const vrow = v_lds + (wk * 32 + vkey) * DB + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    constexpr int VPERIOD = DVB == 8 ? 4 : DVB == 6 ? 2 : 1;
    int voff[VPERIOD];
#pragma unroll
    for (int b = 0; b < VPERIOD; ++b) voff[b] = (b ^ v_swz<DVB>(vkey)) * 64;
    auto v_frag = [&](int buf, int b, int m) __attribute__((always_inline)) {
        const char* p = vrow + buf * TILE + 16 * m * DB + (b / VPERIOD) * VPERIOD * 64 + voff[b % VPERIOD];
        return u32x4_of(lds_read_tr16(p), lds_read_tr16(p + 8 * DB));
    };

    f32x16 oacc[DVB];
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
    float mb_run = kNegBig, l_run = 0.0f;
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent

    // the lane's 16 weights of a sub-tile as the operand of the second contraction
    u32x4 pw[2];
    auto weights = [&](int buf, int key0) __attribute__((always_inline)) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g)
            Mma<uint16_t>::run(s, *reinterpret_cast<const u32x4*>(krow + buf * TILE + (g / KPERIOD) * KPERIOD * 32 + koff[g % KPERIOD]), qf[g]);
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        const float mbn = half_max_w(fmaxf(tm, s[15])) * c;    // (keys past the end are copies of key N-1: no new maximum)
        if (__builtin_amdgcn_ballot_w64(mbn > mb_run + kLazy) != 0) {
            const float mb_new = fmaxf(mb_run, mbn);
            const float alpha = fast_exp2(mb_run - mb_new);    // exactly 1 for lanes whose exponent stands
            l_run *= alpha;
#pragma unroll
            for (int b = 0; b < DVB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[b][r] *= alpha;
            mb_run = mb_new;
        }
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mb_run));
        if (key0 + 32 > N) {                      // keys past the end weigh nothing
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + 4 * half + 8 * (r / 4) + (r % 4) >= N) p[r] = 0.0f;
        }
        float sum = p[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) sum += p[r];
        l_run += sum;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) pw[m][i] = pack_bf16x2(p[8 * m + 2 * i], p[8 * m + 2 * i + 1]);
    };
    auto values = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int b = 0; b < DVB; ++b) Mma<uint16_t>::run(oacc[b], v_frag(buf, b, m), pw[m]);
    };

    const int n_tiles = (N + BN - 1) / BN;
    if constexpr (WK == 1) {
        k_issue(0, 0);
        v_issue(0, 0);
        wait_vmem();
        __syncthreads();
        for_tiles(0, 0, n_tiles, [&](int t, auto bufc) __attribute__((always_inline)) {
            constexpr int BUF = decltype(bufc)::value;
            if (t + 1 < n_tiles) {
                k_issue(t + 1, BUF ^ 1);
                v_issue(t + 1, BUF ^ 1);
            }
            if (q0 < N) {                         // (a wave without queries only moves tiles)
                weights(BUF, t * BN);
                values(BUF);
            }
            wait_vmem();
            __syncthreads();
        });
    } else {
        k_issue(0, 0);
        v_load(0);
        for (int t = 0; t < n_tiles; ++t) {
            const int key0 = t * BN + wk * 32;
            const bool active = key0 < N;         // (a wave without keys only moves tiles)
            wait_vmem();                          // K and V of tile t have arrived
            __syncthreads();                      // every wave is past the V tile before it
            v_store();
            if (t + 1 < n_tiles) v_load(t + 1);
            if (active) weights(0, key0);
            __syncthreads();                      // V tile t is stored; every wave is past K tile t
            if (t + 1 < n_tiles) k_issue(t + 1, 0);
            if (active) values(0);
        }
    }

    // ---- normalise, round once, store: a lane owns runs of 4 consecutive output columns of its query ----------------------
    char* const orow = Oh + (int64_t)(q0 + l32) * rb + half * 8;
    auto store_run = [&](int b, int i, float o0, float o1, float o2, float o3) __attribute__((always_inline)) {
        const u32x2 w = {pack_bf16x2(o0, o1), pack_bf16x2(o2, o3)};
        if (!HALF || b * 64 + i * 16 < rb) *reinterpret_cast<u32x2*>(orow + b * 64 + i * 16) = w;
    };
    if constexpr (WK > 1) {
        constexpr int SLOTS = C::SLOTS;
        float* const part = reinterpret_cast<float*>(lds);
        __syncthreads();                          // every wave is past the last V tile
        float* const mine = part + wave * SLOTS * 64 + lane;
        mine[0] = mb_run;
        mine[64] = l_run;
#pragma unroll
        for (int b = 0; b < DVB; ++b)
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
        const float inv = 1.0f / half_sum_w(L);
        if (q0 + l32 >= N) return;
        for (int b = wk; b < DVB; b += WK)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] = 0.0f;
#pragma unroll
                    for (int j = 0; j < WK; ++j) o[e] = __builtin_fmaf(f[j], grp[(j * SLOTS + 2 + b * 16 + 4 * i + e) * 64], o[e]);
                }
                store_run(b, i, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
            }
    } else {
        const float inv = 1.0f / half_sum_w(l_run);
        if (q0 + l32 >= N) return;
#pragma unroll
        for (int b = 0; b < DVB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                store_run(b, i, oacc[b][4 * i] * inv, oacc[b][4 * i + 1] * inv, oacc[b][4 * i + 2] * inv, oacc[b][4 * i + 3] * inv);
    }
}

template <int DVB, bool HALF, int WQ, int WK>
hipError_t launch_wide_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, hipStream_t stream)
{
    using C = WideCfg<DVB, WQ, WK>;
    const uint32_t strips = (uint32_t)((N + C::BM - 1) / C::BM);
    const uint64_t total = (uint64_t)BH * strips;
    const uint32_t grid = (uint32_t)((total + 7) / 8 * 8);
    hipLaunchKernelGGL((attention_wide_kernel<DVB, HALF, WQ, WK>), dim3(grid), dim3(64 * C::NW), 0, stream,
                       static_cast<const uint16_t*>(Q), static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V),
                       static_cast<uint16_t*>(O), N, fabsf(scale) * kLog2e, scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u, strips,
                       (uint32_t)total);
    return hipGetLastError();
}

template <int DVB, bool HALF>
hipError_t launch_wide(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, hipStream_t stream)
{
    // At most two query blocks per head: workgroups of two waves (2000 heads of N = 64, d = 192: 57.5 -> 51 us; 4000 of
    // N = 32: 75 -> 50).  One round of the key ranges (3.3 us per 128-key tile at d = 256) takes half of one round of the
    // 256-query workgroups (1.6 us per 32-key tile): one head of N = 4096 105 against 190 us, four (two rounds) 210 against 188.
    const int64_t cus = compute_units();
    const int64_t wide = (BH * ((N + 255) / 256) + cus - 1) / cus, ranges = (BH * ((N + 31) / 32) + cus - 1) / cus;
    if (N <= 64) return launch_wide_t<DVB, HALF, 2, 1>(Q, K, V, O, BH, N, scale, stream);
    if (ranges < 2 * wide) return launch_wide_t<DVB, HALF, 1, 4>(Q, K, V, O, BH, N, scale, stream);
    return launch_wide_t<DVB, HALF, 8, 1>(Q, K, V, O, BH, N, scale, stream);
}

}  // namespace

bool attention_wide_supported(int64_t BH, int64_t N, int64_t d)
{
    if (d <= 128 || d > 256 || (d % 16) != 0) return false;
    if (N < 1 || N > ((int64_t)1 << 24)) return false;
    return BH * ((N + 31) / 32) <= (int64_t)0x7ffffff0;
}

hipError_t launch_attention_wide(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                 float scale, hipStream_t stream)
{
    switch ((int)(d / 16)) {
    case 9: return launch_wide<5, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 10: return launch_wide<5, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 11: return launch_wide<6, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 12: return launch_wide<6, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 13: return launch_wide<7, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 14: return launch_wide<7, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 15: return launch_wide<8, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 16: return launch_wide<8, false>(Q, K, V, O, BH, (int)N, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
