// Attention output  O = softmax(scale * Q K^T) V  in bf16: d a multiple of 16 up to 256 but 32 and 64, any N.
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the product
// with V is what the section "Limitations and future Directions" names as the next thing to fuse.  The
// max-subtracted softmax of the Softmax section, Eq. 1, is applied incrementally as in attention_kernels.hip.)
//
// What bounds it: the order inside a wave (scores, softmax, output), with the two waves of a SIMD brought into step by the barrier
// of every tile, under the board's power cap.  Counters at d = 128 / 256, of SIMD cycles: matrix pipe 51 / 59 %, vector ALU 46 / 34 %,
// both at once 13 / 8 %; the 1 KiB fragments of the matrix instructions fill about half of what the LDS can deliver.  A wave owns 32
// queries: at d = 256 its 128 accumulators and 64 registers of Q fragments leave no room for a second query block at two
// waves per SIMD.
//
// A workgroup is WQ query blocks of 32; a tile is SUBS x 32 keys.  K and V lie in LDS as they lie in memory, chunks
// swizzled: V is turned by the transposing LDS read (ds_read_b64_tr_b16: 4 keys x 16 columns, a lane gets the four keys of
// its column), so both tiles travel global -> LDS directly, without registers or a scatter.  Double buffered (4 tiles, 64 KiB at
// d = 256), one barrier per tile.  (Problems of a few heads: attention_ranges.hip; of at most 32 keys, d > 128: attention_short.hip.)  (Enough strips of d from 96 on: attention_pipe.hip, attention_turns.hip.)  Measured, 16 heads of N = 4096: d = 256 928 -> 238 us (1157 TFLOP/s), 192 700 -> 185, 144 633 -> 157
// against one wave per workgroup with operands straight from the caches; d = 96 132 -> 106, d = 128 134 -> 130.5, forty
// heads of N = 600, d = 128 26.7 -> 23.6 against 128-key tiles, V scattered transposed and rows padded to 128 columns.
#include "launchers.h"
#include "attention_common.h"

namespace attnw {
namespace {

template <int DVB, int WQ, int SUBS>
struct WideCfg {
    static constexpr int BM = 32 * WQ;
    static constexpr int BN = 32 * SUBS;
    static constexpr int DB = DVB * 64;           // bytes of a row on chip
    static constexpr int CPR = DVB * 4;           // 16-byte chunks of it
    static constexpr int TILE = BN * DB;
    static constexpr int XFERS = TILE / 1024;     // wave-wide transfers per tile
};

// DVB: 32-column blocks of a row, ceil(d / 32).  HALF: d is an odd multiple of 16 -- the last 16 columns on chip are
// copies of the row's first chunks, left out of the first contraction and not stored by the second.  rb: bytes of a row
// in memory.  Rows past N are read as row N - 1, weigh nothing and are not stored.
template <int DVB, bool HALF, int WQ, int SUBS>
__global__ __launch_bounds__(64 * WQ, WQ == 4 ? 2 : 1)
void attention_wide_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                           uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t strips, uint32_t total)
{
    using C = WideCfg<DVB, WQ, SUBS>;
    using L = RowLayout<DVB>;
    constexpr int NW = WQ, DB = C::DB, CPR = C::CPR, BN = C::BN, TILE = C::TILE, XFERS = C::XFERS;
    constexpr int rb = DB - (HALF ? 32 : 0);
    constexpr int G = rb / 32;                    // 32-byte contraction groups of a row
    static_assert(4 * TILE <= kDirectLds, "reach of direct transfers");

    __shared__ __align__(1024) char lds[4 * TILE];
    char* const k_lds = lds;
    char* const v_lds = lds + 2 * TILE;

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;

    const char* Qh = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * rb;
    const char* Kh = reinterpret_cast<const char*>(K) + (int64_t)bh * N * rb;
    const char* Vh = reinterpret_cast<const char*>(V) + (int64_t)bh * N * rb;
    char* Oh = reinterpret_cast<char*>(O) + (int64_t)bh * N * rb;
    const int q0 = strip * C::BM + wave * 32;

    // ---- Q fragments (a negative scale negates Q) -------------------------------------------------------------------
    u32x4 qf[G];
    {
        const char* qrow = Qh + (int64_t)min(q0 + l32, N - 1) * rb + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(qrow + g * 32) ^ sign_flip;
    }

    // ---- tile transfers: transfer i of a tile moves its chunks 64 i .. 64 i + 63, wave w takes i = w, w + NW, .. --------
    constexpr int XW = (XFERS + NW - 1) / NW;     // transfers per wave and tile
    auto offset = [&](int j, int rows, bool v) __attribute__((always_inline)) {   // rows: last valid row of the tile
        const int s = (wave + NW * j) * 64 + lane;
        const int key = s / CPR;
        int ch = (s - key * CPR) ^ (v ? L::v_block(key) * 4 : L::k_chunk(key));
        if (HALF && ch * 16 >= rb) ch -= rb / 16;
        return (uint32_t)(min(key, rows) * rb + ch * 16);
    };
    // (rows past the end exist in the last tile only; to clamp every tile's rows costs three instructions a transfer, a branch
    // around it cost 5 %)
    const uint32_t k_base = lds_offset_of(k_lds), v_base = lds_offset_of(v_lds);
    auto issue = [&](const char* head, uint32_t dst, int t, bool v) __attribute__((always_inline)) {
        const char* base = head + (int64_t)t * BN * rb;
#pragma unroll
        for (int j = 0; j < XW; ++j)
            if (XFERS % NW == 0 || wave + NW * j < XFERS)
                dma16_untracked(base, offset(j, N - 1 - t * BN, v), dst + (wave + NW * j) * 1024);
    };
    auto k_issue = [&](int t, int buf) __attribute__((always_inline)) { issue(Kh, k_base + buf * TILE, t, false); };
    auto v_issue = [&](int t, int buf) __attribute__((always_inline)) { issue(Vh, v_base + buf * TILE, t, true); };

    // ---- per-lane places of the operand fragments ------------------------------------------------------------------------
    const char* const krow = k_lds + l32 * DB;
    constexpr int KPERIOD = L::KPERIOD, VPERIOD = L::VPERIOD;
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((2 * g + half) ^ L::k_chunk(l32)) * 16;
    const int vkey = 4 * half + ((lane & 15) >> 2);            // a lane's row of the 8-key group that it reads
    const char* const vrow = v_lds + vkey * DB + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    int voff[VPERIOD];
#pragma unroll
    for (int b = 0; b < VPERIOD; ++b) voff[b] = (b ^ L::v_block(vkey)) * 64;
    auto v_frag = [&](int buf, int u, int b, int m) __attribute__((always_inline)) {
        const char* p = vrow + buf * TILE + (32 * u + 16 * m) * DB + (b / VPERIOD) * VPERIOD * 64 + voff[b % VPERIOD];
        return u32x4_of(lds_read_tr16(p), lds_read_tr16(p + 8 * DB));
    };

    f32x16 oacc[DVB];
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
    float mb_run = kNegBig, l_run = 0.0f;
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent

    // sub-tile u of the tile in buffer buf
    auto sub_tile = [&](int buf, int u, int key0) __attribute__((always_inline)) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g)
            Mma<uint16_t>::run(s, *reinterpret_cast<const u32x4*>(krow + buf * TILE + u * 32 * DB + (g / KPERIOD) * KPERIOD * 32 + koff[g % KPERIOD]), qf[g]);
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        const float m = half_wave_max(fmaxf(tm, s[15]));    // (keys past the end are copies of key N-1: no new maximum)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(m * c > mb_run + kLazy) != 0, 0)) {
            const float mb_new = fmaxf(mb_run, reference_exponent(m, c));
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
        u32x4 pw[2];                              // the lane's 16 weights as the operand of the second contraction
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) pw[m][i] = pack_bf16x2(p[8 * m + 2 * i], p[8 * m + 2 * i + 1]);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int b = 0; b < DVB; ++b) Mma<uint16_t>::run(oacc[b], v_frag(buf, u, b, m), pw[m]);
    };

    const int n_tiles = (N + BN - 1) / BN;
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
        if (q0 < N) {                             // (a wave without queries only moves tiles)
#pragma unroll
            for (int u = 0; u < SUBS; ++u)
                if (SUBS == 1 || t * BN + u * 32 < N) sub_tile(BUF, u, t * BN + u * 32);
        }
        wait_vmem();
        __syncthreads();
    });

    // ---- normalise, round once, store: a lane owns runs of 4 consecutive output columns of its query ----------------------
    const float inv = 1.0f / half_wave_sum(l_run);
    if (q0 + l32 >= N) return;
    char* const orow = Oh + (int64_t)(q0 + l32) * rb + half * 8;
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x2 w = {pack_bf16x2(oacc[b][4 * i] * inv, oacc[b][4 * i + 1] * inv),
                             pack_bf16x2(oacc[b][4 * i + 2] * inv, oacc[b][4 * i + 3] * inv)};
            if (!HALF || b * 64 + i * 16 < rb) *reinterpret_cast<u32x2*>(orow + b * 64 + i * 16) = w;
        }
}

// Queries 0 .. q_end - 1 of every head.
template <int DVB, bool HALF, int WQ, int SUBS>
hipError_t launch_wide_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, hipStream_t stream, int q_end)
{
    using C = WideCfg<DVB, WQ, SUBS>;
    const uint32_t strips = (uint32_t)((q_end + C::BM - 1) / C::BM);
    return launch_by_heads(BH, strips, 64 * WQ, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * (DVB * 32 - (HALF ? 16 : 0));
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_wide_kernel<DVB, HALF, WQ, SUBS>), dim3(grid), dim3(64 * WQ), 0, stream,
                           static_cast<const uint16_t*>(Q) + at, static_cast<const uint16_t*>(K) + at, static_cast<const uint16_t*>(V) + at,
                           static_cast<uint16_t*>(O) + at, N, fabsf(scale) * kLog2e, scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u, strips,
                           total);
        return hipGetLastError();
    });
}

template <int DVB, bool HALF>
hipError_t launch_wide(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, hipStream_t stream)
{
    // At most two query blocks per head: workgroups of two waves (2000 heads of N = 64, d = 192: 57.5 -> 51 us).  (Up to d = 128 such
    // lengths are the other kernels'.)
    if constexpr (DVB > 4)
        if (N <= 64) return launch_wide_t<DVB, HALF, 2, 1>(Q, K, V, O, BH, N, scale, stream, N);
    // short rows: a tile of four sub-tiles per barrier (16 heads of N = 4096: d = 16 65.5 -> 57 us, 48 79.9 -> 75.0; d = 128 with two:
    // 130.5 -> 132.7)
    constexpr int SUBS = DVB <= 2 ? 4 : 1;
    const int64_t cus = compute_units(), full = N / 256, tail_rows = N - full * 256, eights = (BH * ((N + 255) / 256) + cus - 1) / cus;
    // A last strip of at most 64 queries that would start another round of workgroups spends what ONE of its waves spends on
    // a full strip: it follows as a launch of the kernel for few heads (16 heads of N = 4097, d = 128: 209 -> 170 us).  (From d = 80 only where
    // the full strips are nine tenths of one round or more: 19 heads of N = 3360, d = 256 350 -> 237 us; workgroups of four waves take the
    // others as they are, 2 to 30 % faster over 2000 random shapes, at d = 144 and 160 those too, 14 %.)
    // (The full strips go to attention_turns.hip and attention_pipe.hip here whatever their own rules say: those weigh them against four waves that would take the tail
    // too.  231 to 256 heads of 257 to 320 tokens 0.90 to 0.99 of the time on eight waves here at d of 176 and more, at 96 to 128 0.99 to 1.015; 64 to 128 heads of 513 to
    // 1088 tokens 0.89 to 0.95.)
    const bool one_round = DVB != 5 && BH * full <= cus && 10 * BH * full > 9 * cus;
    if (full >= 1 && tail_rows >= 1 && tail_rows <= 64 && (BH * full + cus - 1) / cus < eights && (DVB <= 2 || one_round)) {
        constexpr int d = DVB * 32 - (HALF ? 16 : 0);
        const hipError_t e = DVB >= 6                         ? launch_attention_turns(Q, K, V, O, BH, N, d, scale, (int)full * 256, stream)
                             : attention_pipe_supported(N, d) ? launch_attention_pipe(8, Q, K, V, O, BH, N, d, scale, (int)full * 256, stream)
                                                              : launch_wide_t<DVB, HALF, 8, SUBS>(Q, K, V, O, BH, N, scale, stream, (int)full * 256);
        return e != hipSuccess ? e : launch_attention_ranges(Q, K, V, O, BH, N, DVB * 32 - (HALF ? 16 : 0), scale, (int)full * 256, stream);
    }
    if (const int waves = attention_pipe_waves(BH, N, DVB * 32 - (HALF ? 16 : 0)))
        return launch_attention_pipe(waves, Q, K, V, O, BH, N, DVB * 32 - (HALF ? 16 : 0), scale, N, stream);
    if (prefers_attention_turns(BH, N, DVB * 32 - (HALF ? 16 : 0)))
        return launch_attention_turns(Q, K, V, O, BH, N, DVB * 32 - (HALF ? 16 : 0), scale, N, stream);
    // d of 80 and more: workgroups of four waves (128 queries), two to a compute unit.  They move K and V twice as often, and where one
    // waits at a tile's barrier the other computes; the rounds of workgroups end in smaller steps.  Workgroups of eight stay where the second 128 queries
    // are few (N of at most 192: 2018 heads of N = 133, d = 96 50 us with four, 43 with eight), and where those of four fill the last round of theirs more than
    // half.  That full they are faster at d of 112 to 160 and up to 1024 tokens only, from the third round on (four / eight waves 0.73 to 0.95); beyond,
    // d = 80, 96 and from 208 1.03 to 1.1 at any number of rounds, 176 and 192 0.98 to 1.06.  Not full 0.88 to 1.0, but d = 96 from the fourth round on (to 1.06)
    // and d of 240 and 256 beyond 4096 tokens (1.02).  us, eight -> four waves: 64 heads of N = 4096, d = 128 622 -> 566, 400 of 512, d = 80 57.4 -> 51.4, 40 of
    // 600, d = 128 23.9 -> 19.1.  (25000 random shapes of N = 200 to 40000.  d = 16 and 48: 2 % at most, many shapes slower.)
    if constexpr (DVB >= 3) {
        const bool half = BH * ((N + 127) / 128) <= (2 * eights - 1) * cus;
        const bool four = N <= 1024 || DVB == 4 || DVB == 5 ? half || eights > 2
                                                            : half && !(DVB == 3 && !HALF && eights > 3) && !(DVB == 8 && N > 4096 && eights > 2);
        if (N > 192 && four) return launch_wide_t<DVB, HALF, 4, SUBS>(Q, K, V, O, BH, N, scale, stream, N);
    }
    return launch_wide_t<DVB, HALF, 8, SUBS>(Q, K, V, O, BH, N, scale, stream, N);
}

}  // namespace

// (d = 32 and 64 have a kernel of their own, whose waves own up to two query blocks)
bool attention_wide_supported(int64_t BH, int64_t N, int64_t d)
{
    if (d < 16 || d > 256 || (d % 16) != 0 || d == 32 || d == 64) return false;
    if (N < 1 || N > ((int64_t)1 << 24)) return false;
    return BH * (d <= 128 ? (N + 255) / 256 : (N + 31) / 32) <= (int64_t)0x7ffffff0;
}

hipError_t launch_attention_wide(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                 float scale, hipStream_t stream)
{
    // one query block per head, nothing that waves could share
    if (d > 128 && N <= 32) return launch_attention_short(DType::BF16, Q, K, V, O, BH, N, d, scale, stream);
    if (prefers_attention_ranges(BH, N, d)) return launch_attention_ranges(Q, K, V, O, BH, N, d, scale, 0, stream);
    switch ((int)(d / 16)) {
    case 1: return launch_wide<1, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 3: return launch_wide<2, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 5: return launch_wide<3, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 6: return launch_wide<3, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 7: return launch_wide<4, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 8: return launch_wide<4, false>(Q, K, V, O, BH, (int)N, scale, stream);
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
