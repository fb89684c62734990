// Fused attention weights  P = softmax(scale * Q K^T)  and, from the same tiling,
// the stand-alone scaled-score GEMM of the unfused pair.
//
// The paper's fused kernel (section "Fused Matrix Multiply + Scaling + Softmax")
// leaves a block of scores in each core's SRAM after the matrix multiply, scales
// it, reduces row maxima and row sums across the cores that share a row, and
// writes only the attention weights to DRAM.  On one MI355X compute unit a strip
// of BM query rows times all N keys does not fit on chip for the sizes of
// interest, so this kernel walks the keys twice instead: pass one multiplies a
// K tile (staged in LDS) with the strip's Q fragments (held in registers) on the
// matrix cores and folds the scores into a running row maximum and row sum
// (Softmax section, Eq. 1); pass two recomputes the same scores, turns them into
// weights with one fused multiply-add and one 2^x per element, rounds once and
// streams them to HBM.  Scores never leave the registers.
//
// Work split inside a workgroup of WQ x WK waves: wave (wq, wk) owns QW = 32*QB
// queries (strip rows wq*QW ...) and, of every K tile of BN = 32*SUBS*WK keys,
// the SUBS 32-key sub-tiles wk*SUBS ...; partial row maxima / sums of the WK
// waves that share a query meet once, in LDS, between the passes -- the same
// local-then-global reduction the paper runs across a row of cores.
//
// Orientation: the MFMA computes the TRANSPOSED tile  (K tile) * (Q strip)^T, so
// that a lane's 16 accumulators are 16 keys of ONE query: row reductions stay
// inside the lane (plus one exchange between lanes l and l+32) and every lane
// owns runs of 4 consecutive keys for the store.
#include "launchers.h"
#include "qk_common.h"

#include <cstdlib>
#include <cstring>

namespace attnw {
namespace {

// T      element type (uint16_t = bf16 bits, float)
// DB     padded bytes of one Q/K row held on chip (power of two, >= d * sizeof(T))
// QB     32-query blocks per wave
// WQ,WK  waves along queries / along the keys of a tile
// SUBS   32-key sub-tiles per wave per K tile
// SCORES true: write scale * Q K^T (one pass); false: write the attention weights
// FAST   true: N is a multiple of the strip and of the K tile and rows are exactly
//        DB bytes, so no masking, clamping or store predicate is compiled in
// SPLIT  0: a workgroup sweeps all keys of its strip (both passes).
//        Problems with few strips (one head of a long sequence: the paper's own measurements are
//        on a single head) would leave most compute units idle that way; their keys are cut into
//        `kc_count` ranges of whole tiles, one workgroup per (strip, range), and the two passes
//        become two launches:
//        1: pass one over the workgroup's key range.  The ranges of a row must learn each other's
//           (maximum, sum) and the only memory a call may write is the output: the pair of range
//           k goes into slot k of a small table at the start of the row's piece of EVERY range
//           (kc_count * 8 bytes; a piece is at least two tiles long).
//        2: the workgroup reads, for each of its rows, the table at the start of the row's piece
//           of its OWN range -- nobody else touches that piece during this launch -- folds the
//           pairs into the row's maximum and sum and runs pass two over its range, overwriting
//           the tables with weights.  (The score GEMM needs no statistics: one launch of mode 2.)
// RING   (bf16, ragged lengths; 0 = off, else the bytes of one staging write: 8, 4 or 2.)  A piece of a row as a tile
//        leaves it starts and ends inside memory lines whenever the rows of the output do not start on 64-byte
//        boundaries, and lines written in parts cost a read-modify-write each; rows that do not even start on
//        16-byte boundaries (N not a multiple of 8: odd sequence lengths such as 197, 577, 1025) leave only
//        stores of 8, 4 or 2 bytes per lane.  With RING a wave walks whole tiles (WK = 1) and its staging row is a
//        ring of 16-byte chunks laid out as the row lies in MEMORY: an element goes to the chunk and the position
//        it has there (for rows off the 16-byte boundaries that shifts it by up to 7 elements against the tile,
//        hence the narrower staging writes -- 8 bytes while N is a multiple of 4, 4 while it is even, else 2).
//        After a tile the wave stores, of every row, the 16 chunks that END at the last 64-byte boundary inside
//        what it has computed -- the up to three chunks behind that boundary and the chunk that the next tile
//        completes stay in the ring and leave with the next tile.  Every such store is 16 bytes per lane and
//        covers whole lines.  Chunks that never become whole -- the two ends of a row, which share their chunk
//        with the neighbouring rows, and the place where the rotated sweep of the workgroup started -- are
//        written element by element.
template <typename T, int DB, int QB, int WQ, int WK, int SUBS, bool SCORES, bool FAST, int SPLIT = 0, int RING = 0>
__global__ __launch_bounds__(64 * WQ * WK)
void qk_kernel(const T* __restrict__ Q, const T* __restrict__ K, T* __restrict__ out,
               int N, int d, float c, uint32_t sign_flip, uint32_t strips, uint32_t total_tiles, int kc_count, int q_base)
{
    constexpr int ES = sizeof(T);
    constexpr int EPC = 16 / ES;              // elements per 16-byte chunk
    constexpr int NW = WQ * WK;               // waves per workgroup
    constexpr int QW = 32 * QB;               // queries per wave
    constexpr int BM = QW * WQ;               // queries per workgroup
    constexpr int BN = 32 * SUBS * WK;        // keys per LDS tile
    constexpr int G = DB / 32;                // 32-byte contraction groups per row
    constexpr int CPR = DB / 16;              // chunks per K row in LDS
    constexpr int K_TILE_BYTES = BN * DB;
    constexpr int LOADS = BN * CPR / 64 / NW; // 1-KiB wave loads each wave issues per tile
    constexpr int SEG = 32 * SUBS * ES;       // bytes of one staged row: the wave's keys of one tile
    constexpr int CPS = SEG / 16;             // chunks per staged row
    constexpr int RING_CH = CPS + 5;          // RING: chunks of the ring of a row (a tile, the chunks held back, the chunk it shares with the next)
    constexpr int ST_PITCH = (RING != 0 ? RING_CH * 16 : SEG) + 16;   // padded against bank conflicts
    constexpr int ST_BYTES = QW * ST_PITCH;
    constexpr int RPI = 64 / CPS;             // staged rows one store instruction covers
    constexpr int RPL = CPR >= 16 ? 1 : 16 / CPR;           // K rows per 256-byte LDS line
    constexpr int SWZ_MASK = (CPR >= 16 ? 16 : CPR) - 1;
    static_assert((BN * CPR) % (64 * NW) == 0 && CPS <= 64 && QW % RPI == 0, "tile shape");
    static_assert(RING == 0 || ((RING == 2 || RING == 4 || RING == 8) && !FAST && SPLIT == 0 && WK == 1 && QB == 1 && ES == 2 && CPS % 4 == 0),
                  "ring staging: a wave owns whole tiles of whole lines of 32 rows");

    __shared__ __align__(16) char k_lds0[K_TILE_BYTES];   // the two K tile buffers are separate
    __shared__ __align__(16) char k_lds1[K_TILE_BYTES];   // objects: see dma16
    __shared__ __align__(16) char st_lds[NW * ST_BYTES];
    __shared__ float stat_lds[SCORES ? 2 : NW * QW * 2];

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total_tiles) return;
    uint32_t unit = logical;              // (head, strip) pair; with SPLIT the key range is the fastest index
    int kc = 0;
    if constexpr (SPLIT != 0) {
        kc = (int)(unit % (uint32_t)kc_count);
        unit /= (uint32_t)kc_count;
    }
    const uint32_t bh = unit / strips;
    const uint32_t strip = unit - bh * strips;

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int wq = wave / WK, wk = wave % WK;
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;

    const int cpr_act = FAST ? CPR : d * ES / 16;   // chunks of real data per row
    const int row_bytes = FAST ? DB : d * ES;
    const char* Qh = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * row_bytes;
    const char* Kh = reinterpret_cast<const char*>(K) + (int64_t)bh * N * row_bytes;
    T* out_h = out + (int64_t)bh * N * N;
    // (q_base: the launch covers the queries from there on -- the last, partial strip of a ragged length can be a
    // launch of its own with a workgroup shape that spreads its keys over the waves)
    const int qw0 = q_base + strip * BM + wq * QW;   // first query of this wave
    char* const stage = st_lds + wave * ST_BYTES;

    // ---- Q fragments: registers for the whole kernel --------------------------------
    u32x4 qf[QB][G];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qw0 + qb * 32 + l32;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int cq = 2 * g + half;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (FAST || (q < N && cq < cpr_act))
                v = *reinterpret_cast<const u32x4*>(Qh + (int64_t)q * row_bytes + cq * 16);
            qf[qb][g] = v ^ sign_flip;        // negative scale: softmax(-|c| s) = softmax(|c| (-Q) K^T)
        }
    }

    // ---- K tiles: global memory -> LDS directly, 16 bytes per lane ------------------------
    // A wave-wide load fills 1 KiB of consecutive LDS; LDS slot s holds chunk
    // (key, ch) with s = key * CPR + (ch ^ swizzle(key)), so the swizzle that keeps
    // the MFMA operand reads conflict-free is applied to the global address.
    int key_of[LOADS], goff[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int s = (wave + NW * j) * 64 + lane;
        const int key = s / CPR;
        int ch = (s % CPR) ^ ((key / RPL) & SWZ_MASK);
        ch = ch < cpr_act ? ch : 0;           // padding columns are never read: any valid address
        key_of[j] = key;
        goff[j] = key * row_bytes + ch * 16;
    }
    const int n_tiles_all = (N + BN - 1) / BN;
    // this workgroup's tiles: t0 .. t0 + n_tiles (all of them without SPLIT)
    auto range_begin = [&](int k) __attribute__((always_inline)) { return SPLIT != 0 ? n_tiles_all * k / kc_count : 0; };
    const int t0 = range_begin(kc);
    const int n_tiles = SPLIT != 0 ? range_begin(kc + 1) - t0 : n_tiles_all;
    // Every workgroup starts its sweep over the keys at a different tile and wraps
    // around.  With all workgroups marching in step, the rows they write at one moment
    // sit a whole row pitch apart and land on the same few memory channels; the
    // stagger spreads the store stream over all of them.
    const int rot = (int)((logical * 7u) % (uint32_t)n_tiles);
    auto tile_at = [&](int j) __attribute__((always_inline)) { const int t = j + rot; return t0 + (t >= n_tiles ? t - n_tiles : t); };
    auto k_issue = [&](int tile, auto bufc) __attribute__((always_inline)) {
        char* const k_buf = decltype(bufc)::value == 0 ? k_lds0 : k_lds1;
        const int k0 = tile * BN;
        const char* tile_base = Kh + (int64_t)k0 * row_bytes;
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const char* src = tile_base + goff[j];
            if (!FAST && k0 + BN > N) {       // last tile: keys past the end re-read key N-1 (masked later)
                const int kk = min(k0 + key_of[j], N - 1);
                src = Kh + (int64_t)kk * row_bytes + (goff[j] - key_of[j] * row_bytes);
            }
            dma16(src, k_buf + (wave + NW * j) * 1024);
        }
    };

    // scores of 32-key sub-tile `sub` of the tile in `buf`: acc[qb][r] = q . k for key
    // sub*32 + 8*(r/4) + 4*half + r%4 and query qb*32 + l32
    auto mma_subtile = [&](auto bufc, int sub, f32x16 (&acc)[QB]) {
        const int key = sub * 32 + l32;
        const char* rowp = (decltype(bufc)::value == 0 ? k_lds0 : k_lds1) + key * DB;
        const int swz = (key / RPL) & SWZ_MASK;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[qb][r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            // padding columns of short rows hold a copy of chunk 0 of the key (finite) and meet zero Q
            // fragments: no branch here, the loop stays one block the scheduler can interleave
            const u32x4 a = *reinterpret_cast<const u32x4*>(rowp + (((2 * g + half) ^ swz) * 16));
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) Mma<T>::run(acc[qb], a, qf[qb][g]);
        }
    };

    // move the wave's staged QW x (32*SUBS) block to global memory.  Three paths, chosen per wave and
    // tile (wave-uniform): every row and key of the block exists and rows are 16-byte aligned -> NST
    // unconditional 16-byte stores past the caches (the output is far larger than the K of a head, which
    // then stays in L2); aligned rows at an edge -> the same stores predicated; unaligned rows -> one
    // element per lane, a lane-contiguous run of every staged row.  Returns whether the first path ran:
    // only then is the number of store instructions issued known to the wait that follows.
    const bool wave_has_rows = FAST || qw0 < N;
    const bool vec_ok = FAST || (N % EPC) == 0;
    const bool rows_full = FAST || qw0 + QW <= N;
    // rows that do not start on a 64-byte boundary make every 128-byte piece of a store straddle memory
    // lines: such stores go through L2, which merges the pieces before they reach HBM
    const bool past_caches = FAST || (N * ES) % 64 == 0;
    T* const out_lane = out_h + (int64_t)(qw0 + lane / CPS) * N + (lane % CPS) * EPC;
    auto flush_stage = [&](int kseg0) __attribute__((always_inline)) -> bool {
      if constexpr (RING != 0) {
        return false;                         // (the ring has its own flush below)
      } else {
        const bool full = FAST || (rows_full && vec_ok && kseg0 + 32 * SUBS <= N);
        if (full && past_caches) {
#pragma unroll
            for (int it = 0; it < QW / RPI; ++it) {
                const int row = it * RPI + lane / CPS;
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * ST_PITCH + (lane % CPS) * 16);
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out_lane + (int64_t)(it * RPI) * N + kseg0));
            }
        } else if (full) {
#pragma unroll
            for (int it = 0; it < QW / RPI; ++it) {
                const int row = it * RPI + lane / CPS;
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * ST_PITCH + (lane % CPS) * 16);
                *reinterpret_cast<u32x4*>(out_lane + (int64_t)(it * RPI) * N + kseg0) = v;
            }
        } else if (vec_ok) {
#pragma unroll
            for (int it = 0; it < QW / RPI; ++it) {
                const int row = it * RPI + lane / CPS;
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * ST_PITCH + (lane % CPS) * 16);
                if (qw0 + row < N && kseg0 + (lane % CPS) * EPC < N)
                    *reinterpret_cast<u32x4*>(out_lane + (int64_t)(it * RPI) * N + kseg0) = v;
            }
        } else {
            // rows off the 16-byte boundaries: groups of GB = 8, 4 or sizeof(T) bytes, the largest that the row
            // length is a multiple of (rows then start on multiples of it); a lane-contiguous run of every staged row
            auto store_groups = [&](auto gbc) __attribute__((always_inline)) {
                constexpr int GB = decltype(gbc)::value;          // bytes per lane
                constexpr int EG = GB / ES;                       // elements per lane
                constexpr int LPR = SEG / GB;                     // lanes per staged row
                constexpr int RPE = 64 / LPR;                     // staged rows one instruction covers
                static_assert(LPR <= 64 && QW % RPE == 0, "group store shape");
#pragma unroll 4
                for (int it = 0; it < QW / RPE; ++it) {
                    const int row = it * RPE + lane / LPR;
                    const int e = (lane % LPR) * EG;
                    const char* from = stage + row * ST_PITCH + e * ES;
                    T* to = out_h + (int64_t)(qw0 + row) * N + kseg0 + e;
                    if (qw0 + row < N && kseg0 + e < N) {         // (N is a multiple of EG: a group is inside or outside)
                        if constexpr (GB == 8) *reinterpret_cast<u32x2*>(to) = *reinterpret_cast<const u32x2*>(from);
                        else if constexpr (GB == 4) *reinterpret_cast<uint32_t*>(to) = *reinterpret_cast<const uint32_t*>(from);
                        else *to = *reinterpret_cast<const T*>(from);
                    }
                }
            };
            const int row_bytes_out = N * ES;
            if (row_bytes_out % 8 == 0) store_groups(IC<8>{});
            else if (ES == 2 && row_bytes_out % 4 == 0) store_groups(IC<4>{});
            else store_groups(IC<ES>{});
        }
        return full;
      }
    };
    // RING.  With o(r) = the element index of row r's first element in memory mod 8 and a(r) = its 16-byte chunk
    // index mod 4, element k of the j-th tile of the sweep (tile index t) lies in ring chunk
    // (CPS j + (k + o) / 8) mod RING_CH at position (k + o) % 8.  Window of row r after that tile: the CPS chunks
    // that start a(r) chunks before the chunk of the tile's first element, i.e. on a 64-byte boundary; `tail`: the
    // window after that one, what the tile has left behind -- after the last tile of a row (whose successor in the
    // rotated sweep is tile 0) and at the end of the sweep.  Chunk i of the window starts at row element
    // key0 = BN t + 8 (i - a) - o; available are the elements from BN t on (from the tile before on, if that was the
    // previous one of the sweep) up to the end of the tile or of the row.  A lane takes chunk i = lane % CPS of row
    // lane / CPS of every group of RPI rows.  Returns whether exactly NST unconditional stores were issued.
    int ring_p = 0;                           // ring chunk of the first element of the tile whose values are being staged
    auto ring_flush = [&](int j, bool tail) __attribute__((always_inline)) -> bool {
        const int pj = (CPS * j) % RING_CH;
        const int t = tile_at(j);
        const bool chained = j >= 1 && t >= 1;                 // the tile before in memory was the one before in the sweep
        const bool interior = !tail && chained && rows_full && (t + 1) * BN <= N;   // every chunk of every window is whole
        const int avail_lo = chained ? -(1 << 20) : t * BN;
        const int avail_hi = min(N, (t + 1) * BN);
#pragma unroll
        for (int it = 0; it < QW / RPI; ++it) {
            const int row = it * RPI + lane / CPS;
            const int i = lane % CPS + (tail ? CPS : 0);
            T* const row_ptr = out_h + (int64_t)(qw0 + row) * N;
            const int a = (int)((reinterpret_cast<uintptr_t>(row_ptr) >> 4) & 3);
            const int o = (int)((reinterpret_cast<uintptr_t>(row_ptr) >> 1) & 7);
            int x = pj - a + i;                // -3 .. 2 CPS + RING_CH
            x = x < 0 ? x + RING_CH : x;
            x = x >= RING_CH ? x - RING_CH : x;
            x = x >= RING_CH ? x - RING_CH : x;
            const int key0 = t * BN + (i - a) * EPC - o;
            const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * ST_PITCH + x * 16);
            if (interior) {
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(row_ptr + key0));
            } else if (qw0 + row < N) {
                const int lo = max(0, avail_lo - key0), hi = min(EPC, avail_hi - key0);
                if (lo == 0 && hi == EPC) {
                    *reinterpret_cast<u32x4*>(row_ptr + key0) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < EPC; ++e)
                        if (e >= lo && e < hi) row_ptr[key0 + e] = (T)((e & 1) ? (v[e / 2] >> 16) : (v[e / 2] & 0xffffu));
                }
            }
        }
        return interior;
    };
    // the lane's row (QB = 1): where its 4 consecutive keys of a chunk pair land
    int ring_sel = 0, ring_off = 0;           // s = 4 half + o(r): element s + i of the pair of chunks (B, B + 1)
    if constexpr (RING != 0) {
        const int o = (int)((reinterpret_cast<uintptr_t>(out_h + (int64_t)(qw0 + l32) * N) >> 1) & 7);
        ring_sel = 4 * half + o;
        ring_off = l32 * ST_PITCH;
    }
    auto stage_put4 = [&](int qb, int u, int r4, float v0, float v1, float v2, float v3) __attribute__((always_inline)) {
        char* p = stage + (qb * 32 + l32) * ST_PITCH + (u * 32 + 8 * r4 + 4 * half) * ES;
        if constexpr (RING != 0) {
            int b0 = ring_p + (u * 32 + 8 * r4) * ES / 16;          // wave-uniform: chunk of the pair's first element for o = 0
            b0 = b0 >= RING_CH ? b0 - RING_CH : b0;
            const int b1 = b0 + 1 >= RING_CH ? 0 : b0 + 1;
            const uint32_t w01 = pack_bf16x2(v0, v1), w23 = pack_bf16x2(v2, v3);
            char* const rowp = stage + ring_off;
            auto at = [&](int i) __attribute__((always_inline)) {   // element ring_sel + i
                const int e = ring_sel + i;
                return rowp + (e >= 8 ? b1 : b0) * 16 + (e & 7) * 2;
            };
            if constexpr (RING == 8) {
                *reinterpret_cast<u32x2*>(at(0)) = u32x2{w01, w23};
            } else if constexpr (RING == 4) {
                *reinterpret_cast<uint32_t*>(at(0)) = w01;
                *reinterpret_cast<uint32_t*>(at(2)) = w23;
            } else {
                *reinterpret_cast<uint16_t*>(at(0)) = (uint16_t)(w01 & 0xffffu);
                *reinterpret_cast<uint16_t*>(at(1)) = (uint16_t)(w01 >> 16);
                *reinterpret_cast<uint16_t*>(at(2)) = (uint16_t)(w23 & 0xffffu);
                *reinterpret_cast<uint16_t*>(at(3)) = (uint16_t)(w23 >> 16);
            }
            return;
        }
        if constexpr (ES == 2) {
            u32x2 w = {pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
            *reinterpret_cast<u32x2*>(p) = w;
        } else {
            u32x4 w = {__float_as_uint(v0), __float_as_uint(v1), __float_as_uint(v2), __float_as_uint(v3)};
            *reinterpret_cast<u32x4*>(p) = w;
        }
    };

    // bf16: no exponent is taken against less than about -2^31.  A lane's keys may all be masked through a column of K, and the rounding of their own exponent alone would make their
    // weights infinite (reference_exponent, which two to four more instructions per block would be: 1.04 of the time at d above 128).
    const float least = ES == 2 ? fmaxf(-0x1p31f * __builtin_amdgcn_rcpf(c), kNegBig) : kNegBig;
    float m_run[QB], l_run[QB], bias[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) { m_run[qb] = least; l_run[qb] = 0.0f; bias[qb] = 0.0f; }

    // pass one on the scores of one 32-key sub-tile: running maximum and sum of
    // exponentials (Eq. 1), kept per lane; kbase = first key of this lane's first run
    auto fold_stats = [&](f32x16 (&acc)[QB], int kbase, auto tailc) {
        constexpr bool tail = decltype(tailc)::value != 0;   // this tile holds keys past N
        if constexpr (tail) {
            // (wave-uniform: lane 0's kbase is the sub-tile's first key) a sub-tile wholly past N adds nothing
            if (__builtin_amdgcn_readfirstlane(kbase) >= N) return;
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            if constexpr (tail) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (kbase + 8 * (r / 4) + (r % 4) >= N) acc[qb][r] = kNegBig;
            }
            float tm = max3(acc[qb][0], acc[qb][1], acc[qb][2]);
#pragma unroll
            for (int r = 3; r < 15; r += 2) tm = max3(tm, acc[qb][r], acc[qb][r + 1]);
            tm = fmaxf(tm, acc[qb][15]);
            const float mn = fmaxf(m_run[qb], tm);
            l_run[qb] *= fast_exp2((m_run[qb] - mn) * c);
            m_run[qb] = mn;
            const float mb = mn * c;
            float sum = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                // fp32 results are held to an absolute bound: subtract first so that a
                // large common offset cancels exactly
                float e = (ES == 4) ? fast_exp2((acc[qb][r] - mn) * c) : fast_exp2(__builtin_fmaf(acc[qb][r], c, -mb));
                if constexpr (tail) {
                    if (kbase + 8 * (r / 4) + (r % 4) >= N) e = 0.0f;
                }
                sum += e;
            }
            l_run[qb] += sum;
        }
    };
    // pass two (or the score GEMM) on one sub-tile: final values, rounded, into the staging rows
    auto emit = [&](f32x16 (&acc)[QB], int u) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                float p[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float sc = acc[qb][4 * r4 + i];
                    if constexpr (SCORES) p[i] = sc * c;
                    else if constexpr (ES == 4) p[i] = fast_exp2(__builtin_fmaf(sc - m_run[qb], c, -bias[qb]));
                    else p[i] = fast_exp2(__builtin_fmaf(sc, c, -bias[qb]));   // 2^(c*s - c*m - log2 l)
                }
                stage_put4(qb, u, r4, p[0], p[1], p[2], p[3]);
            }
    };

    // ---- the sweep -------------------------------------------------------------------------
    // The K tiles of both passes form one sequence s = 0 .. S-1 (tile_at(s mod n_tiles),
    // LDS buffer s & 1).  A wave always has two things in flight: the MFMAs of its next
    // sub-tile and the VALU work on the scores of the previous one (two accumulator sets),
    // also across the workgroup barrier that ends a tile -- a wave that issued only
    // MFMAs, or only VALU work, between two barriers would leave the other unit idle.
    //   body(s):  [store the rows staged during s-1]
    //             for u < SUBS-1:  MFMA(s, u+1)  ||  VALU(s, u)
    //             wait for the DMA of tile s+1, barrier, start the DMA of tile s+2
    //             MFMA(s+1, 0)  ||  VALU(s, SUBS-1)
    constexpr int NST = QW / RPI;             // store instructions per flush
    f32x16 acc_a[QB], acc_b[QB];              // accumulator set of sub-tile u of buffer b: (b*SUBS + u) & 1
    auto acc_of = [&](auto slotc) __attribute__((always_inline)) -> f32x16 (&)[QB] {
        if constexpr ((decltype(slotc)::value & 1) == 0) return acc_a; else return acc_b;
    };

    // (maximum, sum) table of query q in the piece of key range k: pairs of floats at the first 4-byte boundary of the
    // piece (accessed as single floats; a piece of an odd-length bf16 row may start 2 bytes before it)
    auto table_of = [&](int q, int k) __attribute__((always_inline)) {
        char* const piece = reinterpret_cast<char*>(out_h) + ((int64_t)q * N + (int64_t)range_begin(k) * BN) * ES;
        return reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(piece) + 3) & ~(uintptr_t)3);
    };
    if constexpr (SPLIT == 2 && !SCORES) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int q = qw0 + qb * 32 + l32;
            float mn = kNegBig, l = 0.0f;
            if (FAST || q < N) {
                const float* tab = table_of(q, kc);
                for (int k = 0; k < kc_count; ++k) {
                    const float pm = tab[2 * k], pl = tab[2 * k + 1];
                    const float mx = fmaxf(mn, pm);
                    l = l * fast_exp2((mn - mx) * c) + pl * fast_exp2((pm - mx) * c);
                    mn = mx;
                }
            } else {
                l = 1.0f;                     // a row past the end: nothing of it is stored
            }
            m_run[qb] = mn;
            bias[qb] = (ES == 4) ? fast_log2(l) : __builtin_fmaf(mn, c, fast_log2(l));
        }
    }

    k_issue(tile_at(0), IC<0>{});
    wait_vmem();       // (mode 2: also the table reads above -- they must be done before anyone stores)
    __syncthreads();
    k_issue(tile_at(1 % n_tiles), IC<1>{});
    mma_subtile(IC<0>{}, wk * SUBS, acc_of(IC<0>{}));

    // Nothing in a body depends on whether a next tile exists: past the end of the sequence
    // the extra DMA re-reads a valid tile and the extra MFMAs chew on stale LDS, both
    // unused -- a branch there would split the block the scheduler interleaves.
    auto body = [&](int j, auto bufc, auto writec, auto flushc, auto tailc) __attribute__((always_inline)) {
        constexpr int B = decltype(bufc)::value;
        constexpr bool WRITE = decltype(writec)::value != 0;   // this tile's results go to memory
        constexpr bool FLUSH = decltype(flushc)::value != 0;   // the previous tile's are still staged
        const int k0 = tile_at(j) * BN;
        bool counted = false;                                  // exactly NST stores were issued by this body
        if constexpr (FLUSH) {
            if constexpr (RING != 0) {
                counted = ring_flush(j - 1, false);
                if (tile_at(j - 1) == n_tiles - 1) {   // the sweep wraps to tile 0: nothing may stay behind
                    ring_flush(j - 1, true);
                    counted = false;
                }
            } else {
                counted = flush_stage(tile_at(j - 1) * BN + wk * SUBS * 32);
            }
        }
        if constexpr (RING != 0) ring_p = (CPS * j) % RING_CH;
        // (a wave whose queries all lie past the end -- the last strip of a ragged length -- only moves K tiles and
        //  meets the barriers: the strip then costs its workgroup a fraction of a full one)
        if (wave_has_rows) {
            static_for<SUBS - 1>([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                mma_subtile(bufc, wk * SUBS + u + 1, acc_of(IC<B * SUBS + u + 1>{}));
                if constexpr (WRITE) emit(acc_of(IC<B * SUBS + u>{}), u);
                else fold_stats(acc_of(IC<B * SUBS + u>{}), k0 + (wk * SUBS + u) * 32 + 4 * half, tailc);
            });
        }
        // The DMA of tile s+1 is older than this body's stores and memory operations
        // retire in order, so the wait can leave the NST stores in flight.
        if constexpr (FAST && FLUSH) {
            wait_vmem_le<NST>();
        } else {
            if (!counted) wait_vmem();
            wait_vmem_le<NST>();
        }
        __syncthreads();
        k_issue(tile_at(j + 2 < n_tiles ? j + 2 : j + 2 - n_tiles), bufc);   // this tile's buffer is free now
        // Pin the transfer here: left alone, the scheduler sinks it to the end of the block,
        // right in front of the wait that needs it, and its whole latency is exposed.
        __builtin_amdgcn_sched_barrier(0);
        if (wave_has_rows) {
            mma_subtile(IC<1 - B>{}, wk * SUBS, acc_of(IC<(1 - B) * SUBS>{}));
            if constexpr (WRITE) emit(acc_of(IC<B * SUBS + SUBS - 1>{}), SUBS - 1);
            else fold_stats(acc_of(IC<B * SUBS + SUBS - 1>{}), k0 + (wk * SUBS + SUBS - 1) * 32 + 4 * half, tailc);
        }
    };
    // pass-one body of tile j: the instantiation with key masks only where the tile runs past N
    auto stats_body = [&](int j, auto bufc) __attribute__((always_inline)) {
        if constexpr (FAST) {
            body(j, bufc, IC<0>{}, IC<0>{}, IC<0>{});
        } else {
            if (tile_at(j) * BN + BN > N) body(j, bufc, IC<0>{}, IC<0>{}, IC<1>{});
            else body(j, bufc, IC<0>{}, IC<0>{}, IC<0>{});
        }
    };

    if constexpr (!SCORES && SPLIT != 2) {
        // ================= pass one =================================================================
        for_tiles(0, 0, n_tiles, stats_body);

        // lanes l and l+32 hold the two halves of each query's keys of this wave; the WK
        // waves that share these queries each saw a different slice of every tile
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mo = __shfl_xor(m_run[qb], 32, 64);
            const float lo = __shfl_xor(l_run[qb], 32, 64);
            const float mn = fmaxf(m_run[qb], mo);
            l_run[qb] = l_run[qb] * fast_exp2((m_run[qb] - mn) * c) + lo * fast_exp2((mo - mn) * c);
            m_run[qb] = mn;
            if (WK > 1 && half == 0) {
                stat_lds[(wave * QW + qb * 32 + l32) * 2] = mn;
                stat_lds[(wave * QW + qb * 32 + l32) * 2 + 1] = l_run[qb];
            }
        }
        if constexpr (WK > 1) __syncthreads();
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float mn = m_run[qb], l = l_run[qb];
            if constexpr (WK > 1) {
#pragma unroll
                for (int o = 1; o < WK; ++o) {
                    const int other = wq * WK + (wk + o) % WK;
                    const float mo = stat_lds[(other * QW + qb * 32 + l32) * 2];
                    const float lo = stat_lds[(other * QW + qb * 32 + l32) * 2 + 1];
                    const float mx = fmaxf(mn, mo);
                    l = l * fast_exp2((mn - mx) * c) + lo * fast_exp2((mo - mx) * c);
                    mn = mx;
                }
            }
            m_run[qb] = mn;
            // bf16: bias = c*m + log2(l) folds max and normaliser into one constant;
            // fp32: the max is subtracted separately, bias = log2(l)
            bias[qb] = (ES == 4) ? fast_log2(l) : __builtin_fmaf(mn, c, fast_log2(l));
            if constexpr (SPLIT == 1) {
                // this range's pair into slot kc of the row's table in every range (one lane per query)
                const int q = qw0 + qb * 32 + l32;
                if (wk == 0 && half == 0 && (FAST || q < N)) {
                    for (int k = 0; k < kc_count; ++k) {
                        float* tab = table_of(q, k);
                        tab[2 * kc] = mn;
                        tab[2 * kc + 1] = l;
                    }
                }
            }
        }
    }
    if constexpr (SPLIT == 1) {
        wait_vmem();       // no K transfer may be in flight when the workgroup's LDS is released
        return;
    }

    // ================= pass two (or the only pass of the score GEMM): compute, round, store ========
    // pass one consumed n_tiles buffers, so the first tile of this pass sits in buffer n_tiles & 1
    const int b0 = (SCORES || SPLIT == 2) ? 0 : (n_tiles & 1);
    if (b0 == 0) body(0, IC<0>{}, IC<1>{}, IC<0>{}, IC<0>{}); else body(0, IC<1>{}, IC<1>{}, IC<0>{}, IC<0>{});
    for_tiles(1, b0 ^ 1, n_tiles, [&](int j, auto bufc) __attribute__((always_inline)) { body(j, bufc, IC<1>{}, IC<1>{}, IC<0>{}); });
    wait_vmem();
    if constexpr (RING != 0) {
        ring_flush(n_tiles - 1, false);
        ring_flush(n_tiles - 1, true);        // the chunks held back behind the last 64-byte boundary
    } else {
        flush_stage(tile_at(n_tiles - 1) * BN + wk * SUBS * 32);
    }
}

// Key ranges per strip for a problem of `units` (head, strip) pairs whose rows have n_tiles K tiles: 1 (no
// split) when the strips alone give at least half of the compute units a workgroup; else enough ranges of
// at least two tiles for about two workgroups per compute unit, at most 16 (the table of a row is
// 8 bytes per range and sits inside the first tile of a piece).
int key_ranges(int64_t units, int n_tiles)
{
    const int64_t cus = compute_units();
    if (2 * units >= cus) return 1;
    int64_t k = (2 * cus + units - 1) / units;
    if (k > n_tiles / 2) k = n_tiles / 2;
    if (k > 16) k = 16;
    return k < 2 ? 1 : (int)k;
}

template <typename T, int DB, int QB, int WQ, int WK, int SUBS, bool FAST, bool SPLITTABLE>
hipError_t launch_variant(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d,
                          float scale, hipStream_t stream, bool allow_split)
{
    constexpr int BM = 32 * QB * WQ, BN = 32 * SUBS * WK;
    constexpr int threads = 64 * WQ * WK;
    const uint32_t strips = (uint32_t)((N + BM - 1) / BM);
    const T* q = static_cast<const T*>(Q);
    const T* k = static_cast<const T*>(K);
    T* o = static_cast<T*>(out);
    const float c = scores_only ? scale : fabsf(scale) * kLog2e;
    const uint32_t flip = (!scores_only && scale < 0.0f) ? Mma<T>::kSignMask : 0u;
    if constexpr (SPLITTABLE) {
        const int kc = allow_split ? key_ranges(BH * strips, (N + BN - 1) / BN) : 1;
        if (kc > 1) {
            const uint64_t total = (uint64_t)BH * strips * kc;
            if (total > 0x7ffffff0u) return hipErrorInvalidValue;
            const uint32_t grid = (uint32_t)((total + 7) / 8 * 8);
            if (scores_only) {
                hipLaunchKernelGGL((qk_kernel<T, DB, QB, WQ, WK, SUBS, true, FAST, 2>), dim3(grid), dim3(threads), 0,
                                   stream, q, k, o, N, d, c, flip, strips, (uint32_t)total, kc, 0);
            } else {
                hipLaunchKernelGGL((qk_kernel<T, DB, QB, WQ, WK, SUBS, false, FAST, 1>), dim3(grid), dim3(threads), 0,
                                   stream, q, k, o, N, d, c, flip, strips, (uint32_t)total, kc, 0);
                hipLaunchKernelGGL((qk_kernel<T, DB, QB, WQ, WK, SUBS, false, FAST, 2>), dim3(grid), dim3(threads), 0,
                                   stream, q, k, o, N, d, c, flip, strips, (uint32_t)total, kc, 0);
            }
            return hipGetLastError();
        }
    }
    return launch_by_heads(BH, strips, threads, [&](int64_t first, int64_t heads) {
        const int64_t in = first * N * d, to = first * N * N;
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        if (scores_only)
            hipLaunchKernelGGL((qk_kernel<T, DB, QB, WQ, WK, SUBS, true, FAST>), dim3(grid), dim3(threads), 0, stream, q + in,
                               k + in, o + to, N, d, c, flip, strips, total, 1, 0);
        else
            hipLaunchKernelGGL((qk_kernel<T, DB, QB, WQ, WK, SUBS, false, FAST>), dim3(grid), dim3(threads), 0, stream, q + in,
                               k + in, o + to, N, d, c, flip, strips, total, 1, 0);
        return hipGetLastError();
    });
}

template <typename T, int DB, int QB, int WQ, int WK, int SUBS, bool SPLITTABLE = false>
hipError_t launch_shape(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d,
                        float scale, hipStream_t stream, bool allow_split = false)
{
    constexpr int BM = 32 * QB * WQ, BN = 32 * SUBS * WK;
    // whole strips, whole K tiles, unpadded rows: the variant without masks and predicates
    if (N % BM == 0 && N % BN == 0 && d * (int)sizeof(T) == DB)
        return launch_variant<T, DB, QB, WQ, WK, SUBS, true, SPLITTABLE>(scores_only, Q, K, out, BH, N, d, scale, stream, allow_split);
    return launch_variant<T, DB, QB, WQ, WK, SUBS, false, SPLITTABLE>(scores_only, Q, K, out, BH, N, d, scale, stream, allow_split);
}

// bf16, ragged lengths: 256-query strips, a wave per 32 queries that walks whole 128-key tiles and stores whole
// memory lines out of a ring laid out as the rows lie in memory (RING in qk_kernel).
template <int DB, int GRAN>
hipError_t launch_ring_t(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d, float scale,
                         hipStream_t stream)
{
    constexpr int WQ = 8, BM = 32 * WQ;
    uint32_t strips = (uint32_t)((N + BM - 1) / BM);
    const uint16_t* q = static_cast<const uint16_t*>(Q);
    const uint16_t* k = static_cast<const uint16_t*>(K);
    uint16_t* o = static_cast<uint16_t*>(out);
    const float c = scores_only ? scale : fabsf(scale) * kLog2e;
    const uint32_t flip = (!scores_only && scale < 0.0f) ? Mma<uint16_t>::kSignMask : 0u;
    // The last strip of a ragged length holds N % BM queries, and a workgroup of this shape spends on it what one of
    // its waves spends on a full strip (the waves without queries only help with the K tiles): about half the
    // time of a full workgroup.  Where those workgroups make the difference between one more round of workgroups
    // on the chip and none (N = 4104, 16 heads: 272 workgroups of 256-query strips on 256 compute units), the last
    // strip becomes a launch of its own: 32-query strips whose keys are spread over the 8 waves of a workgroup.
    // Measured, fused / scores in us, B1 H16 d = 128: N = 4104 296 / 226 -> 251 / 141, 4097 322 / 201 -> 266 / 156, 4100
    // 294 / 175 -> 222 / 139, 8200 929 -> 830 (4072, 16 full strips and nothing else: 203 - 210 / 131); 128 heads of N = 513,
    // d = 32: 53 -> 39.
    const int tail_rows = N % BM;
    const int64_t slots = compute_units();
    const int64_t full = BH * (int64_t)(N / BM);
    const bool own_tail = tail_rows != 0 && tail_rows <= 96 && full > 0 &&
                          (full + slots - 1) / slots < (full + BH + slots - 1) / slots;
    if (own_tail) strips -= 1;
    const uint64_t total = (uint64_t)BH * strips;
    const uint32_t grid = (uint32_t)((total + 7) / 8 * 8);
    if (scores_only)
        hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, WQ, 1, 4, true, false, 0, GRAN>), dim3(grid), dim3(64 * WQ), 0, stream,
                           q, k, o, N, d, c, flip, strips, (uint32_t)total, 1, 0);
    else
        hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, WQ, 1, 4, false, false, 0, GRAN>), dim3(grid), dim3(64 * WQ), 0, stream,
                           q, k, o, N, d, c, flip, strips, (uint32_t)total, 1, 0);
    if (own_tail) {
        // 32-query strips, the 128 keys of a tile over 4 waves; with so few strips their keys are split over workgroups as
        // for problems of a few heads (SPLIT in qk_kernel: statistics through tables in P, then the weights)
        const uint32_t tail_strips = (uint32_t)((tail_rows + 31) / 32);
        const int q_base = (int)strips * BM;
        const int kc = key_ranges((int64_t)BH * tail_strips, (N + 127) / 128);
        const uint64_t tail_total = (uint64_t)BH * tail_strips * kc;
        const uint32_t tail_grid = (uint32_t)((tail_total + 7) / 8 * 8);
        if (kc > 1) {
            if (scores_only) {
                hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, 1, 4, 1, true, false, 2>), dim3(tail_grid), dim3(256), 0, stream,
                                   q, k, o, N, d, c, flip, tail_strips, (uint32_t)tail_total, kc, q_base);
            } else {
                hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, 1, 4, 1, false, false, 1>), dim3(tail_grid), dim3(256), 0, stream,
                                   q, k, o, N, d, c, flip, tail_strips, (uint32_t)tail_total, kc, q_base);
                hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, 1, 4, 1, false, false, 2>), dim3(tail_grid), dim3(256), 0, stream,
                                   q, k, o, N, d, c, flip, tail_strips, (uint32_t)tail_total, kc, q_base);
            }
        } else if (scores_only) {   // (unsplit: the 256 keys of a tile over 8 waves)
            hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, 1, 8, 1, true, false>), dim3(tail_grid), dim3(512), 0, stream,
                               q, k, o, N, d, c, flip, tail_strips, (uint32_t)tail_total, 1, q_base);
        } else {
            hipLaunchKernelGGL((qk_kernel<uint16_t, DB, 1, 1, 8, 1, false, false>), dim3(tail_grid), dim3(512), 0, stream,
                               q, k, o, N, d, c, flip, tail_strips, (uint32_t)tail_total, 1, q_base);
        }
    }
    return hipGetLastError();
}
template <int DB>
hipError_t launch_ring(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d, float scale,
                       hipStream_t stream)
{
    // staging writes as wide as the rows' positions in memory allow (rows start on multiples of 2 N bytes)
    if (N % 4 == 0) return launch_ring_t<DB, 8>(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (N % 2 == 0) return launch_ring_t<DB, 4>(scores_only, Q, K, out, BH, N, d, scale, stream);
    return launch_ring_t<DB, 2>(scores_only, Q, K, out, BH, N, d, scale, stream);
}

constexpr int kWideStrips = 200;                  // from so many wide strips on there is work for every compute unit

template <typename T>
hipError_t launch_qk_t(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d,
                       float scale, hipStream_t stream, bool allow_split)
{
    const int row_bytes = d * (int)sizeof(T);
    constexpr int QB = sizeof(T) == 2 ? 2 : 1;   // fp32 stages twice the bytes per key: half the queries per wave
    // wide strips (4 waves along the queries) when that still gives every compute unit work, also when it
    // does so only with the keys of a strip split over several workgroups (rows of 128 and 256 bytes)
    const int64_t wide_units = BH * ((N + 128 * QB - 1) / (128 * QB));
    const bool big = wide_units >= kWideStrips;
    // (not below 1024 keys: two launches of a few microseconds each cost more than the idle compute units)
    const bool split = allow_split && !big && N >= 1024 && row_bytes > 64 && row_bytes <= 256 &&
                       key_ranges(wide_units, (N + 127) / 128) > 1;
    if constexpr (sizeof(T) == 2) {
        // Ragged lengths with enough 256-query strips for the chip: 8 waves of 32 queries that each walk whole tiles
        // and store whole memory lines out of a ring (RING in qk_kernel).  Measured, general kernel -> this one,
        // fused / scores in us.  B1 H16 d128: N = 2056 223 / 110 -> 88 / 52, 4072 286 / 215 -> 240 / 168, 4097 462 / 322 ->
        // 325 / 201, 4100 398 / 265 -> 294 / 175, 4104 (a 17th strip of 8 rows) 369 / 242 -> 340 / 226, 8168 1069 / 828 ->
        // 929 / 711; 4000 (rows on 64-byte boundaries) 225 / 151 both.  B8 H16 d64: N = 1543 368 / 283 -> 300 / 213,
        // 1544 283 / 230 -> 259 / 169, 1284 209 / 157 -> 181 / 119.  Odd lengths gain earlier, as their alternative is 2-byte stores:
        // 1025 193 / 139 -> 182 / 126, B16 H16 N = 785 208 / 152 -> 179 / 126, but not B16 H12 N = 577 105 / 77 -> 111 / 84.  Up to 1280
        // tokens, though, most calls are on the 32-query strips (prefers_strip); here arrive the odd lengths that it leaves: scores
        // from 704 tokens on whose last round of 256-query strips is nearly full, and d above 96 from 1217 on.
        if (N >= ((N & 1) ? 704 : 1280) && (N % 256) != 0 && row_bytes <= 256 && BH * ((N + 255) / 256) >= 100) {
            if (row_bytes <= 64) return launch_ring<64>(scores_only, Q, K, out, BH, N, d, scale, stream);
            if (row_bytes <= 128) return launch_ring<128>(scores_only, Q, K, out, BH, N, d, scale, stream);
            return launch_ring<256>(scores_only, Q, K, out, BH, N, d, scale, stream);
        }
    }
    if (row_bytes <= 64)
        return big ? launch_shape<T, 64, QB, 4, 2, 2>(scores_only, Q, K, out, BH, N, d, scale, stream)
                   : launch_shape<T, 64, QB, 1, 2, 2>(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (row_bytes <= 128)
        return (big || split) ? launch_shape<T, 128, QB, 4, 2, 2, true>(scores_only, Q, K, out, BH, N, d, scale, stream, split)
                              : launch_shape<T, 128, QB, 1, 2, 2>(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (row_bytes <= 256)
        return (big || split) ? launch_shape<T, 256, QB, 4, 2, 2, true>(scores_only, Q, K, out, BH, N, d, scale, stream, split)
                              : launch_shape<T, 256, QB, 1, 2, 2>(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (row_bytes <= 512) return launch_shape<T, 512, 1, 4, 2, 1>(scores_only, Q, K, out, BH, N, d, scale, stream);
    if constexpr (sizeof(T) == 4)
        return launch_shape<T, 1024, 1, 4, 1, 1>(scores_only, Q, K, out, BH, N, d, scale, stream);
    return hipErrorInvalidValue;   // unreachable: d <= 256 bounds row_bytes
}

// bf16 shapes the persistent kernels take: those the two-pass kernel with split keys serves better.  Measured
// on one head of d = 128 (persistent kernel -> split): N = 2048 37 -> 25 us, 4096 68 -> 37, 8192 130 -> 89,
// 16384 269 -> 223; with 128 strips of 2048 or 4096 keys, and at d = 64 (64-query strips: twice the strips),
// the persistent kernel is as fast or faster.
bool prefers_key_split(int64_t BH, int64_t N, int64_t d)
{
    if (d != 128 || N < 2048 || (N % 2) != 0) return false;
    const int64_t strips = BH * ((N + 127) / 128), cus = compute_units();
    return 4 * strips <= cus || (2 * strips <= cus && N >= 8192);
}

// Problems with less than one 128-query strip per compute unit (one to a few heads: the sizes the paper itself
// measures are single heads) leave the persistent two-sweep kernels without work for most of the chip, and the
// key split above pays for it with two launches.  The kernel that spreads the keys of a strip over a gang of
// workgroups keeps every compute unit busy on them.  Measured, one head, default -> gang: d = 128, N = 1024
// 20.8 -> 14.9 us, 2048 25.4 -> 17.1, 4096 36.5 -> 26.1 (two heads 70 -> 37.5, four 75 -> 58); d = 64, N = 2048
// 18.3 -> 11.2, 4096 32.5 -> 19.0, 8192 60 -> 44; from one strip per compute unit on, and at N = 16384, the
// two-sweep kernels are as fast or faster.
bool prefers_gang(int64_t BH, int64_t N, int64_t d)
{
    if (N < 1024 || N > 8192) return false;
    return BH * (N / 128) < (int64_t)compute_units();
}

// fp32 weights on the two-sweep kernel that splits K once per 128 queries: rows on 16-byte boundaries, d <= 128, strips for at
// least half of the compute units, and where it beats the 32-query strips of the next rule, which need four rounds of workgroups
// for one of these.  Measured, this -> those, us: short sequences (1280 heads of N = 100, d = 64 49 -> 79; 150 of 128 10.5 -> 12.4;
// 375 of 128, d = 32 13.7 -> 17.8) and rows past the 2048 keys that stay in registers (ten heads of 3000, d = 64 167 -> 185, seven
// of 4096, d = 128 376 -> 416) stay; not 15 heads of 2048, d = 64 100 -> 95, 125 of 1024 235 -> 207, 31 of 1024, d = 128 99 -> 87, 160 of
// 200 51 -> 37, and wherever the last round of the larger strips is not full (18 of 1024, d = 64 48 -> 36, 75 of 256 16.8 -> 15.6, four of
// 4096 171 -> 117).
bool prefers_f32_split(int64_t BH, int64_t N, int64_t d)
{
    const int64_t cus = compute_units(), large = BH * ((N + 127) / 128), small = BH * ((N + 31) / 32);
    if (d > 128 || N % 4 != 0 || N < 64 || 2 * large < cus) return false;
    const int64_t rounds = (large + cus - 1) / cus, small_rounds = (small + cus - 1) / cus;
    if (small_rounds < 4 * rounds) return N < (d > 64 ? 192 : d > 32 ? 256 : 512);
    return N > 2048 || N < (d > 64 ? 192 : 512) || d <= 32;
}

// fp32 on 32-query strips whose scores stay in registers, after the rule above: weights of everything but short rows of many short
// sequences, where the general kernel computes whole tiles of 128 queries in few rounds of workgroups.  Measured against that kernel, us:
// two heads of 2976, d = 84 410 -> 61, one of 128, d = 64 8.9 -> 7.4, one of 416, d = 128 69 -> 11.5, nine of 2743, d = 128 420 -> 257, 25 of
// 730, d = 228 219 -> 84, 1969 of 65, d = 64 128 -> 89; not 1969 of 65, d = 8 62 -> 73, 204 of 122, d = 32 12.8 -> 16.2, 740 of 117, d = 20 35 -> 41, 80
// of 358, d = 16 20 -> 24.
// Scores need no second sweep there either, and with short rows that kernel is bound by its stores: from some 500 random shapes of
// each range, us.  d <= 16: 3797 of 108 60 -> 139, 434 of 120 11 -> 21, 637 of 60 10.8 -> 15.4, 85 of 381 14.7 -> 21 (tiles nearly full: not taken), but 204 of
// 131 17.8 -> 16.4, 93 of 1025 59 -> 39 (taken).  d <= 32: 1024 strips of N = 101 to 127 9 -> 13 (not taken), of 131 24 -> 16, of 577 46 -> 26.  d <= 64:
// 1470 of 104, d = 36 56 -> 74 (not taken), 194 of 100, d = 64 30 -> 15.5; one of 2810, d = 48 18.5 -> 32: the general kernel splits
// the keys of a few long rows over workgroups (not taken).  Multiples of 4 whose 128-query strips fill their rounds lose a tenth, 16 of 2048, d = 64
// 88.9 -> 98.0, 64 of 1024 92 -> 105, 128 of 512 52 -> 56 (others gain: 20 of 1024 67 -> 34, 300 of 256 45 -> 41), and are taken all the same for
// errors of 8.3e-8 against 1.45e-7.  Beyond d = 64: four of 996, d = 256 152 -> 33, 93 of 1025, d = 64 241 -> 184; not 93 of 1024, d = 256
// 451 -> 487.  Four columns: the six products are less exact than four of the fp32 instruction (scores of normal vectors 4.10e-8 off
// against 3.97e-8; eight columns 4.02e-8 against 5.4e-8).
bool prefers_f32_strip(bool scores_only, int64_t BH, int64_t N, int64_t d)
{
    if (N * d >= (int64_t)1 << 28) return false;
    const int64_t cus = compute_units(), strips = BH * ((N + 31) / 32), large = BH * ((N + 127) / 128);
    const int64_t rounds = (strips + cus - 1) / cus, large_rounds = (large + cus - 1) / cus;
    const bool wide = large >= kWideStrips;       // the general kernel takes 128 queries per workgroup
    if (!scores_only) {
        if (d <= 16 && N < 128) return strips <= cus;
        if (d > 32 || !wide || 2 * rounds < 7 * large_rounds) return true;
        return d > 16 ? N > 128 : N > 384 || large_rounds > 1;
    }
    if (d < 8) return false;
    if (d > 128) return N % 4 != 0 || N % 128 != 0 || strips <= 4 * cus;
    if (d > 64 || N <= 32) return true;
    // keys of few long rows split over workgroups
    if (2 * strips <= cus && N >= (d <= 16 ? 2048 : d <= 32 ? 1152 : 1536) && (d > 16 || N % 4 == 0)) return false;
    if (strips <= cus) return true;
    if (d <= 32 && N % 4 == 0 && N >= 128 && strips > 2 * cus) return false;
    if (d <= 16) return N > 128 && 10 * rounds < (N <= 160 ? 26 : N <= 384 ? 20 : 30) * large_rounds;
    if (N > 128) return d > 32 || !wide || rounds < 4 * large_rounds;
    if (d > 32) return N <= 96 || !wide || 2 * rounds < 7 * large_rounds;
    return wide ? 10 * rounds < (large_rounds <= 2 ? 20 : 25) * large_rounds : strips <= 2 * cus;
}

// bf16 on 32-query strips, a workgroup each, 129 to 1280 tokens.  Measured, the kernel that would take it otherwise -> this one, fused /
// scores in us:
//   few strips: one head of N = 256, d = 64 5.9 -> 4.5, 384 7.7 -> 5.1, 577 16.3 / 12.5 -> 7.5 / 6.5, 1024 10.2 / 7.3 -> 7.5 / 6.2, d = 128 15.3 /
//     9.8 -> 9.3 / 8.2; 64 heads of 197 6.5 -> 6.4, of 160 4.8 -> 5.2, of 320 8.9 -> 7.7, d = 128 9.4 -> 10.4; 24 of 1024, d = 64 24 -> 18; 12 of 512 5.9
//     -> 6.4, 24 of 512 8.4 -> 7.8; 24 of 1280 30 / 20 -> 33 / 28; 12 of 1024 scores 8.2 -> 9.5
//   many: 192 of 577, d = 64 64 -> 41; 390 of 577, d = 32 108 / 81 -> 66 / 62, d = 64 123 / 102 -> 78 / 71, d = 96 219 / 154 -> 97 / 88, d = 128
//     228 / 165 -> 148 / 132; 130 of 1000, d = 64 151 / 112 -> 77 / 68; 128 of 1025 140 / 110 -> 86 / 82; 97 of 1152 85 / 58 -> 72 / 64; 495 of 512
//     76 / 54 -> 68 / 58; 317 of 640 95 / 67 -> 69 / 62, d = 128 131 / 87 -> 102 / 121; 48 of 1024 26 -> 32, d = 128 97 / 60 -> 101 / 90; 647 of 448,
//     d = 128 169 / 104 -> 125 / 124; 79 of 1279, d = 128 152 / 109 -> 151 / 129
//   the last round of 256-query workgroups nearly full, so that whole tiles waste little (`filled`: 32-query strips per eight of those that the
//     rounds hold), not taken, scores in us: 63 of 852, d = 128 29 -> 38, 127 of 880 54 -> 74, 57 of 1000 33 -> 46, d = 112 31 -> 38, 48 of 1250, d = 64 41 ->
//     49, 102 of 1279 93 -> 111, 73 of 672 16.8 -> 20.1, 51 of 640 10.6 -> 13.3, 69 of 704, d = 32 14.6 -> 16.7; weights 51 of 1279, d = 128 80 -> 93; taken: 102
//     of 1250, d = 96 120 -> 108, 127 of 1000, d = 80 68 -> 66, 190 of 1000, d = 112 (a third round) 153 -> 117
//     the same of multiples of 4: 124 of 860, d = 64 47 -> 58, 116 of 984 54 -> 66, 42 of 1156 30 -> 35, 76 of 620, d = 128 24 -> 29, 42 of 1036 34 -> 43
//   scores of whole 32-query strips, not taken: d = 32 86 of 1248 53 -> 67, 113 of 960 37 -> 44, 38 of 1088 19 -> 23, 40 of 640 8.3 -> 11.3, 24 of 1152 14.9 ->
//     17.6; d = 64 148 of 672 34 -> 46, 226 of 672 50 -> 70; taken: d = 32 26 of 992 16.8 -> 14.0, 58 of 1120 38 -> 31, 129 of 960 (a third round) 50 -> 47, 25 of
//     736 13.3 -> 8.5; d = 64 47 of 672 16.6 -> 14.8, 206 of 608 41 -> 37
bool prefers_strip(bool scores_only, int64_t BH, int64_t N, int64_t d)
{
    const int64_t cus = compute_units(), strips = BH * ((N + 31) / 32);
    if (qk_heads_supported(BH, N, d))             // (against whole rows in a wave: short sequences)
        return strips <= cus || (N > 192 && 2 * strips <= (d > 64 ? 2 : 5) * cus);
    const int64_t large = BH * ((N + 255) / 256), rounds = (large + cus - 1) / cus;
    auto filled = [&](int percent) { return 100 * strips > percent * 8 * cus * rounds; };
    if (scores_only) {
        if (d > 96 && N > 1216) return false;     // (one workgroup to a compute unit)
        if (strips <= cus) return true;
        if (N % 2 != 0) return d <= 32 || N < 704 || rounds > 3 || !filled(93);   // (against the ring)
        const bool whole = N % 32 == 0;
        if (large >= kWideStrips) {
            if (d > 96 && rounds <= 2 && filled(75)) return false;
            if (rounds == 1 && filled(whole ? 70 : 85)) return false;
            if (whole && d > 32 && rounds == 2 && filled(90)) return false;
            if (N % 4 == 0 && (d > 96 ? rounds == 1 && filled(68) : rounds <= 2 && N > 704 && filled(72))) return false;
        }
        if (!whole) return true;
        if (N % 128 == 0 && d >= 32 && strips > (d > 32 ? 3 : 2) * cus) return false;
        if (d <= 32 && N > 800 && rounds <= 2 && filled(rounds == 1 ? 50 : 62)) return false;
        return d <= 64 && (N % 256) != 0 && (d <= 32 || N < 640 || (N < 704 && !filled(50)));
    }
    if (d > 112 && N > 1216 && rounds <= 2 && filled(90)) return false;   // (one workgroup to a compute unit)
    if (N % 256 != 0) return true;
    if (d != 64 && d != 128) return N < 1280 || d > 64;
    // whole tiles of the two-sweep, resident and gang kernels
    if (d == 64 && N == 512) return strips > cus;
    if (d == 64 && N == 768) return true;
    return strips <= (N == 1024 ? 3 : 2) * cus;
}

// bf16 on persistent workgroups with 32-query strips, more than 512 tokens.  From 60000 random shapes of 513 to 8192 tokens, time there /
// time on the kernel that would take the call otherwise, by strips per compute unit (x below):
//   weights, d <= 128, 1281 tokens and more: x up to 1 0.15 to 0.75, to 2 0.26 to 0.8, to 4 0.4 to 0.8, to 5 0.6 to 0.95.  Beyond that rows on
//     16-byte boundaries 0.7 to 1.0 but for last rounds of the others' 256-query workgroups that are nearly full (x of 6 to 8.2 and of 14 to 17: 1.0 to
//     1.26), other rows only from 8.3 to 10.2 (0.73 to 0.99; 6 to 8 and above 12 1.0 to 1.25).  Whole tiles of 256: d = 64 0.84 to 1.4, d = 128 0.74 to
//     0.87 up to 2048 tokens, then 0.8 to 1.3; other d 0.4 to 0.95 up to 5, then to 1.11.  Up to 1280 tokens the one-workgroup-per-strip kernel is faster (1.0 to 3).
//   weights, d > 128: x up to 1 0.3 to 0.6, to 2 0.5 to 0.8, beyond 0.55 to 0.95 but where the 128-query workgroups of the general kernel nearly
//     fill a round (1.0 to 1.42), d above 192 that are not whole pieces of 64 columns, more than 2048 tokens (1.1 to 1.36), and many strips (d <= 192 up to
//     16 to 25 0.66 to 0.97, then to 1.2; d > 192 up to 12 and 1280 tokens 0.83 to 1.0, then to 1.8)
//   scores, against a general kernel that splits the keys of few strips over workgroups.  Odd lengths of 1281 and more 0.13 to 0.9 (beyond 2048
//     tokens with d > 32 and few strips 1.1 to 1.3); d <= 32 0.23 to 0.8, whole blocks of 32 keys up to x of 6 0.59 to 0.95; larger d whole blocks 0.64 to 0.9
//     from 3.1 to 4.6 and 9 to 12, other even lengths 0.65 to 0.98 from 3.2 to 4; else 0.95 to 1.5.  Whole blocks of 513 to 1280 tokens, d > 64, 1.6 to
//     4.5: 0.43 to 0.95.  d > 128: 0.26 to 0.95 up to 2 (d > 192: 1.4, up to 896 tokens 1), odd lengths up to 2.2 and 4 to 6.
// All that ends where K no longer comes from an XCD's L2 (4 MiB): the strips read K again for every 32 queries, once or twice, the other kernels for
// every 128 or 256.  Measured to 148000 tokens and 250 strips per compute unit (17000 random shapes above 8192 tokens or 13 strips per unit), time there /
// time on the other kernel:
//   K of one head: weights up to 8 MiB 0.73 to 1.0, beyond 1.0 to 1.5 (d of 144, 160 and 192 up to 12 MiB 0.76 to 0.95, beyond 1.2 to 1.4); scores, d up to
//     128, up to 6 MiB 0.72 to 0.95, beyond 1.0 to 1.3; d of 144 to 192 up to 12 MiB 0.63 to 0.9.
//   Weights, K of the heads that an XCD's 32 workgroups are in at a time, which goes as x d.  Rows on 16-byte boundaries, d up to 64: x d up to 1280 0.64 to 1.0,
//     beyond 1.05 to 2.1 (128 heads of 1544, d = 64 2.0; d of 16 and 32 up to 2048 tokens never above 1.0); d of 80 to 128 up to 2048 tokens 0.75 to 1.0 up to x of 24, to
//     3072 0.85 to 1.0 up to 19, beyond 0.7 to 0.95 up to 10 (d of 80 and 96 later), then 1.05 to 1.9.  d = 144, 160, 176 and 192, the lines below: on this side
//     0.5 to 0.97, on the other 1.0 to 1.5, earlier where the pieces of K overlap (112, 160, 176); d = 112 beyond 8192 tokens in whole tiles 1.05 to 1.3 from
//     x of 2 to 4, then 0.4 to 0.55 to 5.  Whole blocks, scores, d above 64, beyond 4096 tokens and x of 9: 1.0 to 1.3.
bool stream_keeps_k(bool scores_only, int64_t N, int64_t d, double x)
{
    if (N * d > (d > 128 && (scores_only ? d <= 192 : d != 176 && d <= 192) ? 6 : scores_only && d <= 128 ? 3 : 4) << 20) return false;
    if (scores_only) return d <= 64 || d > 128 || N % 2 != 0 || x <= 9 || N <= 4096;
    if (d > 192 || (d > 128 && N <= 1280)) return true;
    if (d == 144) return x <= (N <= 4096 ? 25 : N <= 16384 ? 15 : 9);
    if (d == 160) return x <= (N <= 2048 ? 25 : N <= 4096 ? 14 : N <= 16384 ? 10 : 5);
    if (d == 176) return N > 16384 ? x <= 2 || (x > 4 && x <= 5) : x <= (N <= 2048 ? 14 : N <= 4096 ? 10 : 9);
    if (d == 192) return x <= (N <= 8192 ? 20 : N <= 16384 ? 15 : 5);
    if (d == 112 && N > 8192 && N % 256 == 0) return x <= 2 || x > 4;
    if (d > 64 && N > 8192) return x <= (d == 112 ? 4 : 5) || (x > 8.2 && x <= 10);
    if (N % 8 != 0 || N % 256 == 0) return true;  // (bounded below)
    if (d <= 64) return x * (double)d <= 1280 || (d <= 32 && N <= 2048);
    if (N <= 3072 || (d <= 96 && N <= 4096)) return x <= (d != 112 && N <= 2048 ? 24 : 19);
    return x <= (d <= 96 ? 12 : 10);
}

bool prefers_stream(bool scores_only, int64_t BH, int64_t N, int64_t d)
{
    if (N <= 512) return false;
    const double x = (double)(BH * ((N + 31) / 32)) / (double)compute_units();
    if (!stream_keeps_k(scores_only, N, d, x)) return false;
    auto within = [&](double lo, double hi) { return x > lo && x <= hi; };
    const bool odd = N % 2 != 0, blocks = N % 32 == 0, tiles = N % 256 == 0;
    if (d > 128) {
        if (scores_only) return within(0, d <= 192 ? 2 : N <= 896 ? 1 : 1.4) || (odd && (within(0, 2.2) || within(4, 6)));
        const int64_t rounds = (BH * ((N + 127) / 128) + compute_units() - 1) / compute_units();
        if (d > 192 && N > 2048) return rounds == 1 ? x <= (d == 256 && N <= 8192 ? 2.1 : 2) : rounds == 2 && d == 256 && within(4, 6);
        if (d > 192) return rounds == 1 ? x <= 2.8 : rounds == 2 ? x <= 6 : rounds == 3 && N <= 1280 && x <= 10;
        if (N > 2048 && rounds <= 2) return x <= 3 * rounds;
        return x <= (N <= 640 ? 16 : N <= 896 ? 20 : 25);
    }
    if (N <= 1280) return scores_only && d > 64 && blocks && !tiles && within(1.6, 4.5);
    if (!scores_only) {
        if (tiles && d == 64) return false;
        if (tiles && d == 128) return N <= 2048 && within(0.25, 6);
        if (tiles) return x <= 5;                 // (d other than 64 and 128)
        if (N % 8 == 0) return !within(6, d <= 32 ? 7.5 : 8.2) && (d <= 32 || !within(14, 17));
        return within(0, d <= 32 ? 6 : 5) || within(8.3, 10.2);
    }
    if (odd && d <= 32) return within(0, 6);
    if (odd) return N <= 2048 ? within(0, 1) || within(1.35, 5) : within(0.9, 1) || within(1.35, 1.95) || within(2, 4.4);
    if (d <= 32) return tiles ? within(0, 4) : blocks ? within(0, 6) : N % 8 == 0 ? within(0, 2) || within(3.1, 4) : within(0, 4);
    if (tiles) return false;
    return blocks ? within(3.1, 4.6) || within(9, 12) : N <= 4096 && within(3.2, 4);
}

}  // namespace

hipError_t launch_qk(DType dt, bool scores_only, const void* Q, const void* K, void* out,
                     int64_t BH, int64_t N, int64_t d, float scale, hipStream_t stream)
{
    if (dt == DType::F32 && !scores_only && prefers_f32_small(BH, N, d)) return launch_qk_f32_small(Q, K, out, BH, N, d, scale, stream);
    if (dt == DType::F32 && !scores_only && prefers_f32_split(BH, N, d) && split_takes_scale(scale))
        return launch_qk_f32_split(Q, K, out, BH, N, d, scale, stream);
    if (dt == DType::F32 && prefers_f32_strip(scores_only, BH, N, d) && split_takes_scale(scale))
        return launch_qk_f32_strip(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (dt == DType::F32) return launch_qk_t<float>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream, true);
    // ATTNW_FUSED_KERNEL=twopass keeps bf16 problems on the two-pass kernel above, =rounds keeps short sequences
    // off the resident kernel (tests and measurements compare the three)
    // (read at every call: the parity tests switch it between calls; one getenv against a launch of microseconds)
    const char* force = getenv("ATTNW_FUSED_KERNEL");
    const bool twopass = force && strcmp(force, "twopass") == 0;
    const bool rounds = force && strcmp(force, "rounds") == 0;
    const bool gang = force && strcmp(force, "gang") == 0;
    const bool tiny = force && strcmp(force, "tiny") == 0;
    const bool heads = force && strcmp(force, "heads") == 0;
    const bool strip = force && strcmp(force, "strip") == 0;
    const bool streamed = force && strcmp(force, "stream") == 0;
    // Very many windows of up to 64 tokens with heads of 16, off the 16-byte boundaries: waves that work alone on a stream of (head, 32
    // queries) pairs.  Against the kernel after the next, us: 12288 heads of N = 49 21.0 / 22.3, 16384 of 33 24.6 / 26.7, 30000 of 13 16.0 / 17.6;
    // not 8192 pairs (4096 of 49 10.4 / 9.2), multiples of 8 (16384 of 56 27.6 / 25.4), scores (16384 of 49 24.9 / 21.9) or heads of 32 (12288 of 49
    // 25.9 / 26.0, 4096 11.6 / 10.2, 12288 of 62 32.9 / 31.3).
    if (qk_tiny_supported(BH, N, d) && (tiny || (!force && !scores_only && N % 8 != 0 && BH * ((N + 31) / 32) >= 16384)))
        return launch_qk_tiny(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (qk_stream_supported(BH, N, d) && (streamed || (!force && prefers_stream(scores_only, BH, N, d))))
        return launch_qk_stream(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (qk_strip_supported(BH, N, d) && (strip || (!force && prefers_strip(scores_only, BH, N, d))))
        return launch_qk_strip(scores_only, Q, K, out, BH, N, d, scale, stream);
    // Up to 384 tokens: whole rows of scores in the registers of a wave, K of the head in LDS.  Measured against the kernels below and
    // those that it replaced, fused / scores in us, 1000 heads: N = 33, d = 64 6.3 / 5.8 -> 5.0 / 4.7, 65 9.6 -> 8.5, 100 16.5 -> 10.4, 128, d = 128
    // 35 -> 17, d = 256 49 -> 37, 129, d = 64 25 / 24 -> 20 / 16, 160 27 / 30 -> 19 / 17, 197 44 / 40 -> 28 / 26 (d = 128 98 / 75 -> 49 / 44),
    // 256 52 -> 41, 257 114 / 93 -> 52 / 43, 304 113 / 82 -> 54 / 46; 200 heads of 371 39 -> 29, of 384 31 -> 23; 20000 of one token 88 -> 15.
    // Not taken: scores in whole tiles of the kernels below (N = 256: 2048 heads of d = 32 50 against 56, d = 128 107 against 114).
    if (qk_heads_supported(BH, N, d) && (heads || (!force && !(scores_only && N == 256))))
        return launch_qk_heads(scores_only, Q, K, out, BH, N, d, scale, stream);
    if (!scores_only && qk_gang_supported(BH, N, d) && (gang || (!force && prefers_gang(BH, N, d))))
        return launch_qk_gang(Q, K, out, BH, N, d, scale, stream);
    if (!twopass && !(!rounds && prefers_key_split(BH, N, d))) {
        if (!scores_only && !rounds && qk_resident_supported(BH, N, d))
            return launch_qk_resident(Q, K, out, BH, N, scale, stream);
        // (scores with 256-byte rows stay on the general kernel: two co-resident workgroups of it stream them faster)
        if (qk_rounds_supported(BH, N, d) && (!scores_only || d == 64))
            return launch_qk_rounds(scores_only, Q, K, out, BH, N, d, scale, stream);
    }
    // (forced onto the two-pass kernel: the plain one, a workgroup per strip)
    return launch_qk_t<uint16_t>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream, !twopass);
}

}  // namespace attnw
