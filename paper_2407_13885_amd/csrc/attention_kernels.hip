// Attention output  O = softmax(scale * Q K^T) V  with the attention weights kept on chip.
//
// The paper's section "Limitations and future Directions" names the product with V as the next thing
// to fuse into its kernel
// (Multi-Head Self-Attention section: Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V).  Once the
// weights are not written, nothing forces two sweeps over the keys: the max-subtracted softmax
// (Softmax section, Eq. 1) is applied incrementally -- a reference exponent that follows the running
// row maximum, a running sum l, and an output accumulator that is rescaled by 2^(old - new) whenever
// the reference moves -- and one sweep over the K and V tiles suffices.
//
// Work split: one workgroup of 8 waves per (head, strip of 8 * QW queries); every wave owns
// QW = 32 * QB queries and walks ALL keys, so no statistics cross waves.  (Problems of a few heads have too few such
// strips for the chip: attention_ranges.hip.)
// Per 128-key tile:
//   K tile  [128 keys][d]      global -> LDS directly, chunk-swizzled as in the weight kernels;
//   V tile  transposed on the way into LDS as Vt[d][128 keys]: the second contraction runs over
//           keys, and a matrix-core operand wants its 8 contraction elements contiguous per lane.
// Per 32-key sub-tile and query block (all on v_mfma_f32_32x32x16_bf16, fp32 accumulate):
//   S^T = K_sub * Q^T          lane (query l32, half h) holds keys 8i + 4h + j of its query;
//   sub-tile max (shared by lanes l, l+32: both feed the same second contraction; long rows: only where the weights'
//   sums call for it), p = 2^(c s - ref),
//   l += sum p (fp32), p rounded to bf16;
//   O^T += Vt_sub * P^T        lane (query l32, half h) holds O[query][8i + 4h + j] per 32-wide block.
// The k-index of the second contraction is a permutation of the keys chosen so that a lane's own
// 8 weights ARE its operand: slot 8h + e  <->  key 16m + 8 (e / 4) + 4h + e % 4.  Vt stores the keys
// of every 16-group in that order (bits 2 and 3 of the key index swapped).
#include "launchers.h"
#include "attention_common.h"

namespace attnw {
namespace {

template <int DB, int QB>
struct AttnCfg {
    static constexpr int D = DB / 2;              // head dimension
    static constexpr int NW = 8;
    static constexpr int QW = 32 * QB;            // queries per wave
    static constexpr int BM = QW * NW;            // queries per workgroup
    static constexpr int BN = 128;                // keys per tile
    static constexpr int G = DB / 32;             // 32-byte contraction groups per K row
    static constexpr int CPR = DB / 16;           // 16-byte chunks per K / V row
    static constexpr int DVB = D / 32;            // 32-wide blocks of the output row
    static constexpr int K_TILE_BYTES = BN * DB;
    static constexpr int K_LOADS = BN * CPR / 64 / NW;
    static constexpr int V_LOADS = 2 * CPR / NW;  // wave-wide loads of 64 keys x one chunk, per wave and tile
    static constexpr int VT_PITCH = BN * 2 + 16;  // bytes of one Vt row (one output column, 128 keys)
    static constexpr int VT_BYTES = D * VT_PITCH;
    static constexpr int RPL = 16 / CPR;          // (4 or 8 chunks per row)
    static constexpr int SWZ_MASK = CPR - 1;
    static constexpr int LDS_TOTAL = 2 * K_TILE_BYTES + 2 * VT_BYTES;
};

// TAIL: N is not a whole number of tiles / strips.  Rows past the end are read as row N-1 (every load
// stays inside the arrays), their weights are forced to 0 and their queries are not stored.
// SUMS: the exponent of the weights follows their sums (kFarSum) and not the maximum of the scores.
template <int DB, int QB, bool TAIL, bool SUMS>
__global__ __launch_bounds__(512)
void attention_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                      uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t strips, uint32_t total)
{
    constexpr int rb = DB;                        // bytes of a row
    using C = AttnCfg<DB, QB>;
    constexpr int NW = C::NW, QW = C::QW, BM = C::BM, BN = C::BN, G = C::G, CPR = C::CPR, DVB = C::DVB;
    constexpr int K_TILE_BYTES = C::K_TILE_BYTES, K_LOADS = C::K_LOADS, V_LOADS = C::V_LOADS;
    constexpr int VT_PITCH = C::VT_PITCH, VT_BYTES = C::VT_BYTES;
    static_assert(2 * K_TILE_BYTES <= kDirectLds, "reach of direct transfers");
    static_assert((2 * CPR) % NW == 0, "V tile load shape");

    __shared__ __align__(1024) char lds[C::LDS_TOTAL];
    char* const k_lds = lds;
    char* const vt_lds = lds + 2 * K_TILE_BYTES;

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;

    const char* Qh = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * rb;
    const char* Kh = reinterpret_cast<const char*>(K) + (int64_t)bh * N * rb;
    const char* Vh = reinterpret_cast<const char*>(V) + (int64_t)bh * N * rb;
    char* Oh = reinterpret_cast<char*>(O) + (int64_t)bh * N * rb;
    const int q0 = strip * BM + wave * QW;

    auto row_in = [&](int r) __attribute__((always_inline)) { return TAIL ? min(r, N - 1) : r; };

    // ---- Q fragments (a negative scale negates Q) ----------------------------------------------------
    u32x4 qf[QB][G];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            qf[qb][g] = *reinterpret_cast<const u32x4*>(Qh + (int64_t)row_in(q0 + qb * 32 + l32) * rb + (2 * g + half) * 16) ^ sign_flip;
        }

    // ---- per-lane constants ----------------------------------------------------------------------------
    // K tile transfer j of this lane: key within the tile (recomputed where a clamp needs it), byte offset in the tile
    // (s = (wave + NW j) 64 + lane is transfer j's chunk of the tile: its chunk within the row, and the bits of its key
    // that the swizzle takes, do not depend on j -- one offset per lane and a constant step per transfer, instead of
    // a 64-bit offset register pair per transfer)
    constexpr int KSTEP = NW * 64 / CPR;          // keys between transfers j and j + 1 of a lane
    static_assert((NW * 64) % CPR == 0 && KSTEP % C::RPL == 0 && (KSTEP / C::RPL) % (C::SWZ_MASK + 1) == 0, "K transfer shape");
    auto k_key = [&](int j) __attribute__((always_inline)) { return (wave * 64 + lane) / CPR + KSTEP * j; };
    int k_off0;
    {
        const int s = wave * 64 + lane;
        const int ch = (s % CPR) ^ ((k_key(0) / C::RPL) & C::SWZ_MASK);
        k_off0 = k_key(0) * rb + ch * 16;
    }
    auto k_off = [&](int j) __attribute__((always_inline)) { return k_off0 + j * KSTEP * rb; };
    const uint32_t k_lds_base = lds_offset_of(k_lds);
    int kfrag_off[G];
    {
        const int swz = (l32 / C::RPL) & C::SWZ_MASK;
#pragma unroll
        for (int g = 0; g < G; ++g) kfrag_off[g] = l32 * DB + (((2 * g + half) ^ swz) * 16);
    }
    // V tile: wave-wide load j covers 64 consecutive keys x one 16-byte chunk (8 output columns); the
    // 8 values go to 8 Vt rows at the key's permuted position (64 lanes -> 128 contiguous bytes per row)
    // (NW is even: the half of the tile is the same for every j, the chunk advances by NW / 2)
    static_assert(NW % 2 == 0, "V load shape");
    const int v_key0 = (wave & 1) * 64 + lane;
    auto v_key = [&](int) __attribute__((always_inline)) { return v_key0; };
    int v_off0, v_ldsoff0;
    {
        const int ch = wave >> 1;
        const int pos = (v_key0 & ~12) | ((v_key0 & 4) << 1) | ((v_key0 & 8) >> 1);   // bits 2 and 3 swapped
        v_off0 = v_key0 * rb + ch * 16;
        v_ldsoff0 = ch * 8 * VT_PITCH + pos * 2;
    }
    auto v_off = [&](int j) __attribute__((always_inline)) { return v_off0 + j * (NW / 2) * 16; };
    auto v_ldsoff = [&](int j) __attribute__((always_inline)) { return v_ldsoff0 + j * (NW / 2) * 8 * VT_PITCH; };
    // Vt fragment of (block dvb, sub-tile u, group m): row dvb*32 + l32, keys u*32 + 16m + 8*half ..
    const int vfrag_off = l32 * VT_PITCH + half * 16;

    const int n_tiles = (N + BN - 1) / BN;
    // rows past the end exist only in the last tile of a TAIL problem: there every row index is clamped
    // (the row a transfer reads moves, its place in LDS does not)
    auto k_issue = [&](int tile, int buf) __attribute__((always_inline)) {
        const char* tile_base = Kh + (int64_t)tile * BN * rb;
        const bool clamp = TAIL && tile == n_tiles - 1;
#pragma unroll
        for (int i = 0; i < K_LOADS; ++i) {
            const char* src = tile_base + k_off(i);
            if (clamp) src -= (int64_t)(tile * BN + k_key(i) - row_in(tile * BN + k_key(i))) * rb;
            dma16_untracked(src, k_lds_base + buf * K_TILE_BYTES + (wave + NW * i) * 1024);
        }
    };
    u32x4 vreg[V_LOADS];
    auto v_load = [&](int tile) __attribute__((always_inline)) {
        const char* tile_base = Vh + (int64_t)tile * BN * rb;
        const bool clamp = TAIL && tile == n_tiles - 1;
#pragma unroll
        for (int j = 0; j < V_LOADS; ++j) {
            const char* src = tile_base + v_off(j);
            if (clamp) src -= (int64_t)(tile * BN + v_key(j) - row_in(tile * BN + v_key(j))) * rb;
            vreg[j] = *reinterpret_cast<const u32x4*>(src);
        }
    };
    auto v_scatter = [&](int buf) __attribute__((always_inline)) {
        char* base = vt_lds + buf * VT_BYTES;
#pragma unroll
        for (int j = 0; j < V_LOADS; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t w = vreg[j][e / 2];
                *reinterpret_cast<uint16_t*>(base + v_ldsoff(j) + e * VT_PITCH) = (uint16_t)((e & 1) ? (w >> 16) : (w & 0xffffu));
            }
    };

    f32x16 oacc[QB][DVB];
    float mb_run[QB], l_run[QB];
    constexpr float kLazy = 8.0f;    // binades the maximum may run ahead of the reference exponent
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        mb_run[qb] = kNegBig; l_run[qb] = 0.0f;
#pragma unroll
        for (int b = 0; b < DVB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[qb][b][r] = 0.0f;
    }

    // one 128-key tile out of buffers `buf`
    // (maskc: the tile runs past N -- only the last tile of a TAIL problem is compiled with the masks)
    auto compute_tile = [&](auto bufc, int t, auto maskc) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        constexpr bool MASK = decltype(maskc)::value != 0;
        const char* kb = k_lds + BUF * K_TILE_BYTES;
        const char* vb = vt_lds + BUF * VT_BYTES + vfrag_off;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            u32x4 kf[G];
#pragma unroll
            for (int g = 0; g < G; ++g) kf[g] = *reinterpret_cast<const u32x4*>(kb + u * 32 * DB + kfrag_off[g]);
            f32x16 s[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[qb][r] = 0.0f;
#pragma unroll
                for (int g = 0; g < G; ++g) Mma<uint16_t>::run(s[qb], kf[g], qf[qb][g]);
            }
            u32x4 vf[DVB][2];
#pragma unroll
            for (int b = 0; b < DVB; ++b)
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    vf[b][m] = *reinterpret_cast<const u32x4*>(vb + b * 32 * VT_PITCH + (u * 32 + 16 * m) * 2);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float p[16];
                // The exponent the weights are taken against (mb_run) follows the running maximum lazily: it moves only when some query
                // of the wave exceeds it by more than kLazy binades (SUMS: when the weights' sums say so).  Until then weights up to
                // 2^kLazy appear, which costs nothing (fp32 sums, and bf16 has the same relative precision at every magnitude),
                // and the 16 * DVB multiplies of the output accumulator - needed at every new maximum otherwise, i.e. in most of
                // the early sub-tiles of a row - become rare.  Lanes whose exponent stands get the factor 2^0 = 1 exactly.
                if constexpr (!SUMS) {
                    // (written out: the compiler schedules this form in 92 registers where it takes 100 with the lambdas of the other branch, 36 -> 33.7 us
                    // for 198 heads of N = 613, d = 32)
                    const float m = half_wave_max(max16(s[qb]));   // shared by the two lanes of a query
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(m * c > mb_run[qb] + kLazy) != 0, 0)) {
                        const float mb_new = fmaxf(mb_run[qb], reference_exponent(m, c));
                        const float alpha = fast_exp2(mb_run[qb] - mb_new);
                        l_run[qb] *= alpha;
#pragma unroll
                        for (int b = 0; b < DVB; ++b)
#pragma unroll
                            for (int r = 0; r < 16; ++r) oacc[qb][b][r] *= alpha;
                        mb_run[qb] = mb_new;
                    }
                    const float mb = mb_run[qb];
#pragma unroll
                    for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[qb][r], c, -mb));
                    if constexpr (MASK) {
                        // keys past the end were read as key N-1 (their scores change no maximum): no weight
                        const int kbase = t * BN + u * 32 + 4 * half;
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (kbase + 8 * (r / 4) + (r % 4) >= N) p[r] = 0.0f;
                    }
                    float sum = p[0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) sum += p[r];
                    l_run[qb] += sum;
                } else {
                    auto weigh = [&](float mb) __attribute__((always_inline)) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[qb][r], c, -mb));
                        if constexpr (MASK) {
                            const int kbase = t * BN + u * 32 + 4 * half;
#pragma unroll
                            for (int r = 0; r < 16; ++r)
                                if (kbase + 8 * (r / 4) + (r % 4) >= N) p[r] = 0.0f;
                        }
                    };
                    auto move = [&](float to) __attribute__((always_inline)) {
                        const float alpha = fast_exp2(mb_run[qb] - to);
                        l_run[qb] *= alpha;
#pragma unroll
                        for (int b = 0; b < DVB; ++b)
#pragma unroll
                            for (int r = 0; r < 16; ++r) oacc[qb][b][r] *= alpha;
                        mb_run[qb] = to;
                    };
                    auto maximum = [&]() __attribute__((always_inline)) { return reference_exponent(half_wave_max(max16(s[qb])), c); };
                    auto total = [&]() __attribute__((always_inline)) {
                        float part[4] = {p[0], p[1], p[2], p[3]};
#pragma unroll
                        for (int r = 4; r < 16; ++r) part[r & 3] += p[r];
                        return (part[0] + part[1]) + (part[2] + part[3]);
                    };
                    if (u == 0 && t == 0) mb_run[qb] = fmaxf(mb_run[qb], maximum());
                    weigh(mb_run[qb]);
                    float sum = total();
                    if (__builtin_amdgcn_ballot_w64(sum > kFarSum) != 0) {
                        if (__builtin_amdgcn_ballot_w64(sum > kOverflow) != 0) {
                            move(fmaxf(mb_run[qb], maximum()));
                            weigh(mb_run[qb]);
                            sum = total();
                        } else {
                            // (one factor, between the exponents as rounded, for these weights and all before them)
                            const float to = mb_run[qb] + far_exponent(p), a = fast_exp2(mb_run[qb] - to);
#pragma unroll
                            for (int r = 0; r < 16; ++r) p[r] *= a;
                            sum *= a;
                            move(to);
                        }
                    }
                    l_run[qb] += sum;
                }
                // a lane's weights of group m are accumulators 8m .. 8m+7: exactly its operand of the second contraction
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    u32x4 pw;
#pragma unroll
                    for (int i = 0; i < 4; ++i) pw[i] = pack_bf16x2(p[8 * m + 2 * i], p[8 * m + 2 * i + 1]);
#pragma unroll
                    for (int b = 0; b < DVB; ++b) Mma<uint16_t>::run(oacc[qb][b], vf[b][m], pw);
                }
            }
        }
    };

    // ---- prologue: tile 0 --------------------------------------------------------------------------------
    k_issue(0, 0);
    v_load(0);
    v_scatter(0);
    wait_vmem();
    __syncthreads();

    // ---- the sweep: while tile t is computed, K tile t+1 lands in the other buffer and V tile t+1 waits in registers
    auto iteration = [&](int t, auto bufc, auto maskc) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        const int nxt = t + 1 < n_tiles ? t + 1 : 0;      // past the end: a valid tile, unused
        k_issue(nxt, BUF ^ 1);
        v_load(nxt);
        // (a wave whose queries all lie past the end -- the last strip of a ragged length -- only moves tiles and meets
        // the barriers: the waves that share its SIMD get the issue slots; measured on 192 heads of N = 577, d = 64:
        // 47.4 -> 43.0 us.  The test stays outside compute_tile -- inside,
        // per query block, it cost the full strips 3-5 %)
        if (!TAIL || q0 < N) compute_tile(bufc, t, maskc);
        v_scatter(BUF ^ 1);
        wait_vmem();
        __syncthreads();
    };
    if constexpr (TAIL) {
        for_tiles(0, 0, n_tiles - 1, [&](int t, auto bufc) __attribute__((always_inline)) { iteration(t, bufc, IC<0>{}); });
        if (((n_tiles - 1) & 1) == 0) iteration(n_tiles - 1, IC<0>{}, IC<1>{});
        else iteration(n_tiles - 1, IC<1>{}, IC<1>{});
    } else {
        for (int t = 0; t < n_tiles; t += 2) {      // N is a multiple of two tiles
            iteration(t, IC<0>{}, IC<0>{});
            iteration(t + 1, IC<1>{}, IC<0>{});
        }
    }

    // ---- normalise, round once, store: a lane owns runs of 4 consecutive output columns of its query -----------
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float inv = 1.0f / half_wave_sum(l_run[qb]);
        if (TAIL && q0 + qb * 32 + l32 >= N) continue;
        char* orow = Oh + (int64_t)(q0 + qb * 32 + l32) * rb + half * 8;
#pragma unroll
        for (int b = 0; b < DVB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                u32x2 w = {pack_bf16x2(oacc[qb][b][4 * i] * inv, oacc[qb][b][4 * i + 1] * inv),
                           pack_bf16x2(oacc[qb][b][4 * i + 2] * inv, oacc[qb][b][4 * i + 3] * inv)};
                *reinterpret_cast<u32x2*>(orow + (b * 32 + 8 * i) * 2) = w;
            }
    }
}

// Queries 0 .. q_end - 1 of every head (q_end < 0: all).
template <int DB, int QB, bool TAIL>
hipError_t launch_attention_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale,
                              hipStream_t stream, int q_end = -1)
{
    using C = AttnCfg<DB, QB>;
    const uint32_t strips = (uint32_t)(((q_end < 0 ? N : q_end) + C::BM - 1) / C::BM);
    const float c = fabsf(scale) * kLog2e;
    const uint32_t flip = scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u;
    auto go = [&](auto kernel) {
        return launch_by_heads(BH, strips, 512, [&](int64_t first, int64_t heads) {
            const int64_t at = first * N * C::D;
            const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(512), 0, stream, static_cast<const uint16_t*>(Q) + at,
                               static_cast<const uint16_t*>(K) + at, static_cast<const uint16_t*>(V) + at, static_cast<uint16_t*>(O) + at, N,
                               c, flip, strips, total);
            return hipGetLastError();
        });
    };
    // A look at the sums costs more where the exponent moves, in the first tiles of a row, and saves in all others.  us, maxima -> sums: 16 heads
    // of N = 4096, d = 32 64.0 -> 59.1, 48 of 4096, d = 64 270 -> 250, 72 of 1120, d = 32 32.3 -> 29.6; rows of every sharpness 276 -> 271 (48 of 4096),
    // 607 -> 585 (8 of 16384); but 200 of 512, d = 64 27.4 -> 28.4, 128 of 2048 in two query blocks a wave 162 -> 171 (one
    // block takes those, prefers_two_blocks).  (Two blocks and ragged ends: registers for the scores and their weights spill.  One block of d = 64
    // without ragged ends: with the maxima two workgroups share a compute unit, and with more workgroups than units that is worth more:
    // 432 of 1280 262 -> 220 us, 61 of 3328 234 -> 225; 50 of 1280, one workgroup a unit, 27.9 with the sums, 29.7 without.)
    if constexpr (QB == 2) return go(attention_kernel<DB, QB, TAIL, !TAIL>);
    else {
        const bool pairs = DB == 128 && !TAIL && BH * strips > compute_units();
        return N >= 1024 && !pairs ? go(attention_kernel<DB, QB, TAIL, true>) : go(attention_kernel<DB, QB, TAIL, false>);
    }
}

// A ragged length whose last strip (256 queries, 512 with two query blocks per wave) holds at most 64 queries, and whose partial strips start another round
// of workgroups on the chip: such a workgroup spends what ONE of its waves spends on a full strip -- the whole sweep
// over the keys -- on a few rows.  The partial strips are left out of the launch and follow as a second one of the kernel
// for few heads, whose waves share the keys of 32 queries.  Measured: 64 heads of N = 2049, d = 64: 146 -> 96 us; 128 heads of
// N = 1025: 74 -> 62 us.
template <int DB, int QB = 1>
hipError_t launch_attention_own_tail(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale,
                                     hipStream_t stream, bool* taken)
{
    constexpr int BM = 256 * QB;
    const int64_t full = N / BM, tail_rows = N - full * BM;
    const int64_t slots = (int64_t)compute_units() * (DB == 64 && QB == 1 ? 2 : 1);   // (co-resident workgroups: registers)
    *taken = full >= 1 && tail_rows >= 1 && tail_rows <= 64 &&
             (BH * full + slots - 1) / slots < (BH * (full + 1) + slots - 1) / slots;
    if (!*taken) return hipSuccess;
    const hipError_t e = launch_attention_t<DB, QB, true>(Q, K, V, O, BH, N, scale, stream, (int)(full * BM));
    if (e != hipSuccess) return e;
    return launch_attention_ranges(Q, K, V, O, BH, N, DB / 2, scale, (int)(full * BM), stream);
}

// d = 64: two query blocks per wave (512-query strips) read K and V half as often, and one block (256) needs half the time per round of
// workgroups.  One workgroup of either kind fits a compute unit, and a round of the first takes 1.8 rounds of the second: two blocks
// where they need at most that share of the rounds.  us, 512 -> 256 queries: 45 heads of N = 2743 (270 strips of 512) 204 -> 121, 33 of 4096 (264)
// 241 -> 208; but 68 of 2888 (408) 195 -> 209, 40 of 3072 (240) 99 -> 113.  Whole lengths below 2560, where one block takes the maxima, two
// workgroups to a unit, and two blocks gained nothing from the sums: always one (794 of 1024 357 -> 268, 128 of 2048 166 -> 160).  (Of 21000 random
// shapes of N = 513 .. 9000 this line comes within 0.3 % of the better of the two, mean; the line "200 strips of 512 or more" within 7 %.)  At
// d = 32 two blocks gain 2 % at best and lose 15 % over the lot: there is one.
bool prefers_two_blocks(int64_t BH, int64_t N)
{
    const int64_t cus = compute_units();
    auto rounds = [&](int64_t BM) {
        const int64_t all = (BH * ((N + BM - 1) / BM) + cus - 1) / cus, whole = (BH * (N / BM) + cus - 1) / cus;
        // (partial strips in a launch of their own, launch_attention_own_tail, weigh as half a workgroup each)
        return N % BM >= 1 && N % BM <= 64 && N > BM && whole < all ? (double)whole + 0.5 * (double)BH / (double)cus : (double)all;
    };
    return N > 512 && !(N % 512 == 0 && N < 2560) && 1.8 * rounds(512) < rounds(256);
}

}  // namespace

bool attention_supported(int64_t BH, int64_t N, int64_t d)
{
    if (d != 32 && d != 64) return false;
    if (N < 1 || N > ((int64_t)1 << 24)) return false;
    return BH * ((N + 255) / 256) <= (int64_t)0x7ffffff0;
}

hipError_t launch_attention(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                            float scale, hipStream_t stream)
{
    if (prefers_attention_ranges(BH, N, d)) return launch_attention_ranges(Q, K, V, O, BH, N, d, scale, 0, stream);
    if (d == 64 ? attention_pipe_64(BH, N) : attention_pipe_32(BH, N)) return launch_attention_pipe(4, Q, K, V, O, BH, N, d, scale, (int)N, stream);
    bool taken;
    if (d == 32) {
        if ((N % 256) == 0) return launch_attention_t<64, 1, false>(Q, K, V, O, BH, (int)N, scale, stream);
        const hipError_t e = launch_attention_own_tail<64>(Q, K, V, O, BH, (int)N, scale, stream, &taken);
        return taken ? e : launch_attention_t<64, 1, true>(Q, K, V, O, BH, (int)N, scale, stream);
    }
    const bool two = prefers_two_blocks(BH, N);
    if ((N % 256) != 0) {   // any length: rows past the end are clamped and masked
        const hipError_t e = two ? launch_attention_own_tail<128, 2>(Q, K, V, O, BH, (int)N, scale, stream, &taken)
                                 : launch_attention_own_tail<128>(Q, K, V, O, BH, (int)N, scale, stream, &taken);
        if (taken) return e;
        return two ? launch_attention_t<128, 2, true>(Q, K, V, O, BH, (int)N, scale, stream)
                   : launch_attention_t<128, 1, true>(Q, K, V, O, BH, (int)N, scale, stream);
    }
    if (two && (N % 512) == 0) return launch_attention_t<128, 2, false>(Q, K, V, O, BH, (int)N, scale, stream);
    return launch_attention_t<128, 1, false>(Q, K, V, O, BH, (int)N, scale, stream);
}

}  // namespace attnw
