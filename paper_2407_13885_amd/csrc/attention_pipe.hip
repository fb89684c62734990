// Attention output  O = softmax(scale * Q K^T) V  in bf16 for d = 96 to 160 and more than 128 tokens, and for d = 32 and 64: the sweep of attention_wide.hip with
// the steps of neighbouring tiles under way at once.
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; Softmax section, Eq. 1, applied
// incrementally.)
//
// In the time of tile t (32 keys) a wave (32 queries) makes the weights of tile t on the vector unit while the matrix unit makes the output
// of tile t - 1 and the scores of tile t + 1: one matrix instruction, then its share of the exponentials, sums, packs and maxima, so that neither unit
// waits for the other.  A wave alone issues a vector instruction every 7.6 cycles (two waves 3.8): what stands one after the other in a wave is slow even where
// the SIMD's other wave fills the gaps, and with the scores, the softmax and the output of one tile after the other (attention_wide.hip) matrix and
// vector unit worked at the same time in 13 % of the cycles; here in 24 %.
//
// Matrix instructions of 16 x 16 x 32 (mma16): less power per product than 32 x 32 x 16, and these kernels run at the board's power cap.  (They take more issue
// slots, 8 cycles of the vector unit's each: with twice the vector work per product, at d = 64, the 32 x 32 shape is as fast, and this kernel the faster one only where its
// smaller steps count, attention_pipe_64.)
//
// K and V travel global -> LDS directly into rings of four tiles, one barrier for two tiles (one for each: 3 % slower); fragments of K are read a tile ahead.
// 16 heads of N = 4096: d = 96 105 -> 96 us, 128 129 -> 115.5 (1.19 PFLOP/s), 144 154 -> 134, 160 161 -> 140; 8 of 4000, d = 128 91 -> 67;
// two of 32768 965 -> 861 (1.28 PFLOP/s); 40 of 600 18.5 -> 15.1.  Wider heads have no registers for the scores of two tiles.
#include "launchers.h"
#include "attention_common.h"

namespace attnw {
namespace {

// DVB: 32-column blocks of a row, ceil(d / 32).  HALF: d is an odd multiple of 16 -- the last 16 columns on chip are zeros in Q and K
// (written once: no transfer touches them) and left out of the second contraction.  WQ: waves of a workgroup, 32
// queries each.  At least five tiles of 32 keys.  Rows past N are read as row N - 1, weigh nothing and are not stored.
template <int DVB, bool HALF, int WQ>
__global__ __launch_bounds__(64 * WQ, WQ == 4 ? 2 : 1)
void attention_pipe_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                           uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t strips, uint32_t total)
{
    using L = RowLayout<DVB>;
    constexpr int BN = 32, NW = WQ, NBUF = 4;
    constexpr int DB = DVB * 64;                  // bytes of a row on chip
    constexpr int CPR = DVB * 4;                  // 16-byte chunks of it
    constexpr int TILE = BN * DB;
    constexpr int XFERS = TILE / 1024;            // wave-wide transfers per tile
    constexpr int XW = (XFERS + NW - 1) / NW;     // of a wave
    constexpr int rb = DB - (HALF ? 32 : 0);      // bytes of a row in memory
    constexpr int G = DVB;                        // 32-column contraction groups of a row
    constexpr int CB = rb / 32;                   // 16-column blocks
    static_assert(2 * NBUF * TILE <= kDirectLds, "reach of direct transfers");

    __shared__ __align__(1024) char lds[2 * NBUF * TILE];
    char* const k_lds = lds;
    char* const v_lds = lds + NBUF * TILE;

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l16 = lane & 15;
    const int quarter = lane >> 4;

    const char* Qh = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * rb;
    const char* Kh = reinterpret_cast<const char*>(K) + (int64_t)bh * N * rb;
    const char* Vh = reinterpret_cast<const char*>(V) + (int64_t)bh * N * rb;
    char* Oh = reinterpret_cast<char*>(O) + (int64_t)bh * N * rb;
    const int q0 = strip * (32 * WQ) + wave * 32;
    const int n_tiles = (N + BN - 1) / BN;

    // ---- Q fragments of the two blocks of 16 queries (a negative scale negates Q) ------------------------------------------
    u32x4 qf[2][G];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const char* qrow = Qh + (int64_t)min(q0 + 16 * x + l16, N - 1) * rb;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const bool inside = !HALF || g + 1 < G || quarter < 2;
            qf[x][g] = *reinterpret_cast<const u32x4*>(qrow + g * 64 + (inside ? quarter : 0) * 16) ^ sign_flip;
            if (!inside) qf[x][g] = u32x4{0u, 0u, 0u, 0u};
        }
    }

    // ---- tile transfers: transfer i of a tile moves its chunks 64 i .. 64 i + 63, wave w takes i = w, w + NW, ... ----------
    // (Behind the last tile it is transferred again, unused.)
    const uint32_t k_base = lds_offset_of(k_lds), v_base = lds_offset_of(v_lds);
    auto transfer = [&](const char* head, uint32_t dst, int t, int j, bool v) __attribute__((always_inline)) {
        if (XFERS % NW != 0 && wave + NW * j >= XFERS) return;
        t = min(t, n_tiles - 1);
        const int s = (wave + NW * j) * 64 + lane;
        const int key = s / CPR;
        const int ch = (s - key * CPR) ^ (v ? L::v16_block(key) * 2 : L::k_chunk(key));
        if (!HALF || ch * 16 < rb)
            dma16_untracked(head + (int64_t)t * BN * rb, (uint32_t)(min(key, N - 1 - t * BN) * rb + ch * 16), dst + (wave + NW * j) * 1024);
    };
    auto k_issue = [&](int t, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < XW; ++j) transfer(Kh, k_base + buf * TILE, t, j, false);
    };
    auto v_issue = [&](int t, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < XW; ++j) transfer(Vh, v_base + buf * TILE, t, j, true);
    };

    // ---- per-lane places of the operand fragments ------------------------------------------------------------------------
    const char* const krow = k_lds + l16 * DB;
    constexpr int KPERIOD = L::KPERIOD / 2, VPERIOD = L::V16PERIOD;
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((4 * g + quarter) ^ L::k_chunk(l16)) * 16;
    // keys 16 (f % 2) .. + 15 x columns 32 (f / 2) .. + 31 (8 a lane)
    auto k_frag = [&](int buf, int f) __attribute__((always_inline)) {
        const int g = f / 2;
        return *reinterpret_cast<const u32x4*>(krow + buf * TILE + (f % 2) * 16 * DB + (g / KPERIOD) * KPERIOD * 64 + koff[g % KPERIOD]);
    };
    const int vkey = 4 * quarter + (l16 >> 2);    // a lane's row of the 16 keys that it reads
    const char* const vrow = v_lds + vkey * DB + (lane & 3) * 8;
    int voff[VPERIOD];
#pragma unroll
    for (int b = 0; b < VPERIOD; ++b) voff[b] = (b ^ L::v16_block(vkey)) * 32;
    // 16 columns x 32 keys: of a lane keys 4 quarter .. + 3 and 16 more than these, as its weights
    auto v_frag = [&](int buf, int b) __attribute__((always_inline)) {
        const char* p = vrow + buf * TILE + (b / VPERIOD) * VPERIOD * 32 + voff[b % VPERIOD];
        return u32x4_of(lds_read_tr16(p), lds_read_tr16(p + 16 * DB));
    };

    f32x4 oacc[CB][2];                            // columns 16 b + 4 quarter .. + 3 of queries l16, 16 + l16
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int x = 0; x < 2; ++x) oacc[b][x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float mb_run[2], l_run[2];
    constexpr float kLazy = 6.0f;                 // binades the maximum may run ahead of the reference exponent (8: sharp rows 3 % further off)

    struct Scores { f32x4 s[2][2]; };             // keys 16 k + 4 quarter .. + 3, queries 16 x + l16
    struct Weights { u32x4 w[2]; };               // of a lane, as the operand of the second contraction
    constexpr int KF = 2 * G, RV = G == 1 ? 2 : 4;   // fragments of K of a tile; those of V held at a time
    // (From one instruction to the next one operand stays: registers that change cost power.)
    auto scores = [&](int buf) __attribute__((always_inline)) {
        Scores r;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int x = 0; x < 2; ++x) r.s[k][x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int f = 0; f < KF; ++f) {
            const u32x4 kf = k_frag(buf, f);
            const int k = f % 2;
            mma16(r.s[k][k], kf, qf[k][f / 2]);
            mma16(r.s[k][1 - k], kf, qf[1 - k][f / 2]);
        }
        return r;
    };
    auto output = [&](int buf, const Weights& pw) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const u32x4 vf = v_frag(buf, b);
            mma16(oacc[b][b & 1], vf, pw.w[b & 1]);
            mma16(oacc[b][1 - (b & 1)], vf, pw.w[1 - (b & 1)]);
        }
    };
    float p[2][8];                                // the weights of the tile before the one whose scores are s
    auto pack = [&]() __attribute__((always_inline)) {
        Weights pw;
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) pw.w[x][i] = pack_bf16x2(p[x][2 * i], p[x][2 * i + 1]);
        return pw;
    };
    // the largest of a lane's scores of query block x (keys past the end are copies of key N - 1: no new maximum)
    auto largest = [&](const Scores& r, int x) __attribute__((always_inline)) {
        return fmaxf(max3(max3(max3(r.s[0][x][0], r.s[0][x][1], r.s[0][x][2]), r.s[0][x][3], r.s[1][x][0]), r.s[1][x][1], r.s[1][x][2]), r.s[1][x][3]);
    };
    // The exponents move where the largest score of some query is far above (some lane's own is if and only if its query's is); the weights p and
    // all before them follow, of the 16 queries that it is among.
    auto follow = [&](const float (&top)[2]) __attribute__((always_inline)) {
        const float ahead[2] = {__builtin_fmaf(top[0], c, -mb_run[0]), __builtin_fmaf(top[1], c, -mb_run[1])};
        if (__builtin_amdgcn_ballot_w64(fmaxf(ahead[0], ahead[1]) > kLazy) == 0) return;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            if (__builtin_amdgcn_ballot_w64(ahead[x] > kLazy) == 0) continue;
            const float mb_new = fmaxf(mb_run[x], reference_exponent(quarter_wave_max(top[x]), c));
            const float alpha = fast_exp2(mb_run[x] - mb_new);       // exactly 1 for lanes whose exponent stands
            l_run[x] *= alpha;
#pragma unroll
            for (int b = 0; b < CB; ++b) oacc[b][x] *= alpha;
#pragma unroll
            for (int r = 0; r < 8; ++r) p[x][r] *= alpha;
            mb_run[x] = mb_new;
        }
    };

    // ---- One barrier for two tiles: while tiles 2T and 2T + 1 are computed, K of 2T + 4, 2T + 5 and V of 2T + 1, 2T + 2 are on their way; the
    // fragments read are those of K of 2T + 2, 2T + 3 and of V of 2T - 1, 2T. ----------------------------------------------------------
    auto request_pair = [&](int t) __attribute__((always_inline)) {   // t = 2T
        k_issue(t + 4, t & 3);
        k_issue(t + 5, (t + 1) & 3);
        v_issue(t + 1, (t + 1) & 3);
        v_issue(t + 2, (t + 2) & 3);
    };
    auto end_of_pair = [&]() __attribute__((always_inline)) {
        wait_vmem();
        __syncthreads();                          // (and the wave's fragments have left the buffers)
    };
    if constexpr (HALF) {
        for (int i = threadIdx.x; i < NBUF * TILE / 16; i += 64 * NW) *reinterpret_cast<u32x4*>(k_lds + i * 16) = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
    }
    k_issue(0, 0);
    k_issue(1, 1);
    v_issue(0, 0);
    k_issue(2, 2);
    k_issue(3, 3);
    end_of_pair();
    if (q0 >= N) {                                // (a wave without queries only moves tiles)
        __syncthreads();
        request_pair(0);
        for (int t = 1; t < n_tiles - 1; ++t) {
            if (t % 2 == 0) request_pair(t);
            else end_of_pair();
        }
        end_of_pair();
        return;
    }
    Scores s = scores(0), sn = scores(1);
    __syncthreads();
    request_pair(0);
    // The weights of tile 0.  Their exponent is of the largest score of tiles 0 and 1: what a row's largest weight is taken against exactly is not rounded, and
    // in sharp rows that is most of the error.
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        mb_run[x] = fmaxf(kNegBig, reference_exponent(quarter_wave_max(fmaxf(largest(s, x), largest(sn, x))), c));
#pragma unroll
        for (int r = 0; r < 8; ++r) p[x][r] = fast_exp2(__builtin_fmaf(s.s[r / 4][x][r % 4], c, -mb_run[x]));
        l_run[x] = p[x][0];
#pragma unroll
        for (int r = 1; r < 8; ++r) l_run[x] += p[x][r];
    }
    s = sn;
    u32x4 kf[KF], vf[RV];
#pragma unroll
    for (int f = 0; f < KF; ++f) kf[f] = k_frag(2, f);

    // ---- Tile t: its weights, the output of tile t - 1, the scores of tile t + 1 ------------------------------------------------------
    auto tile = [&](int t, auto bufc) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;             // t mod 4
        constexpr int STEPS = 2 * (KF + CB), OPS = 8 + 32 + 16 + 8;
        Weights pw;
        float pn[2][8], sum[2], top[2];
        auto vector_op = [&](auto oc) __attribute__((always_inline)) {
            constexpr int I = decltype(oc)::value;
            if constexpr (I < 8) {
                constexpr int X = I / 4, J = I % 4;
                pw.w[X][J] = pack_bf16x2(p[X][2 * J], p[X][2 * J + 1]);
            } else if constexpr (I < 40) {
                // (f0 f1 e0 f2 e1 .. f15 e14 e15: an exponential does not wait for the product right before it)
                constexpr int J = I - 8;
                constexpr bool EXP = J == 31 || (J >= 2 && J % 2 == 0);
                constexpr int E = J == 31 ? 15 : EXP ? J / 2 - 1 : (J + 1) / 2;
                constexpr int X = E / 8, R = E % 8;
                if constexpr (EXP) pn[X][R] = fast_exp2(pn[X][R]);
                else pn[X][R] = __builtin_fmaf(s.s[R / 4][X][R % 4], c, -mb_run[X]);
            } else if constexpr (I < 56) {
                constexpr int X = (I - 40) % 2, R = (I - 40) / 2;
                if constexpr (R == 0) sum[X] = pn[X][0];
                else sum[X] += pn[X][R];
                if constexpr (R == 7) l_run[X] += sum[X];
            } else {
                constexpr int X = (I - 56) % 2, J = (I - 56) / 2;
                if constexpr (J == 0) top[X] = max3(sn.s[0][X][0], sn.s[0][X][1], sn.s[0][X][2]);
                if constexpr (J == 1) top[X] = max3(top[X], sn.s[0][X][3], sn.s[1][X][0]);
                if constexpr (J == 2) top[X] = max3(top[X], sn.s[1][X][1], sn.s[1][X][2]);
                if constexpr (J == 3) top[X] = fmaxf(top[X], sn.s[1][X][3]);
            }
        };
        static_for<STEPS>([&](auto ic) __attribute__((always_inline)) {
            constexpr int I = decltype(ic)::value, F = I / 2, SECOND = I % 2;
            if constexpr (F < KF) {
                constexpr int GR = F / 2, KB = F % 2, X = SECOND ? 1 - KB : KB;
                if constexpr (GR == 0) sn.s[KB][X] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                mma16(sn.s[KB][X], kf[F], qf[X][GR]);
                if constexpr (SECOND && F >= KF - RV) vf[F - (KF - RV)] = v_frag((BUF + 3) % 4, F - (KF - RV));
            } else {
                constexpr int B = F - KF, X = SECOND ? 1 - B % 2 : B % 2, NEXT = I - 2 * KF;
                mma16(oacc[B][X], vf[B % RV], pw.w[X]);
                if constexpr (SECOND && B + RV < CB) vf[B % RV] = v_frag((BUF + 3) % 4, B + RV);
                if constexpr (NEXT < KF) kf[NEXT] = k_frag((BUF + 2) % 4, NEXT);      // (in the first of these steps: arrived by the end of the tile)
            }
            static_for<(I + 1) * OPS / STEPS - I * OPS / STEPS>([&](auto jc) __attribute__((always_inline)) {
                vector_op(IC<I * OPS / STEPS + decltype(jc)::value>{});
            });
            // (transfers between the steps: a wave that issues them in a row waits 50 cycles for each)
            if constexpr (BUF % 2 == 0 && I % 2 == 0 && I / 2 < 4 * XW) {
                constexpr int J = I / 2 % XW, WHICH = I / 2 / XW;
                if constexpr (WHICH == 0) transfer(Kh, k_base + BUF * TILE, t + 4, J, false);
                if constexpr (WHICH == 1) transfer(Kh, k_base + (BUF + 1) % 4 * TILE, t + 5, J, false);
                if constexpr (WHICH == 2) transfer(Vh, v_base + (BUF + 1) % 4 * TILE, t + 1, J, true);
                if constexpr (WHICH == 3) transfer(Vh, v_base + (BUF + 2) % 4 * TILE, t + 2, J, true);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        static_assert(2 * CB >= KF && 8 * XW <= STEPS);
        s = sn;
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int r = 0; r < 8; ++r) p[x][r] = pn[x][r];
        follow(top);
        if constexpr (BUF % 2 == 1) end_of_pair();
    };
    for (int t = 1;;) {
        if (t >= n_tiles - 1) break;
        tile(t++, IC<1>{});
        if (t >= n_tiles - 1) break;
        tile(t++, IC<2>{});
        if (t >= n_tiles - 1) break;
        tile(t++, IC<3>{});
        if (t >= n_tiles - 1) break;
        tile(t++, IC<0>{});
    }
    end_of_pair();

    // ---- the last two tiles ---------------------------------------------------------------------------------------------------------
    output((n_tiles - 2) & 3, pack());
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        float sum = 0.0f;
#pragma unroll
        for (int r = 0; r < 8; ++r) {             // keys past the end weigh nothing
            const bool past = (n_tiles - 1) * BN + 16 * (r / 4) + 4 * quarter + r % 4 >= N;
            p[x][r] = past ? 0.0f : fast_exp2(__builtin_fmaf(s.s[r / 4][x][r % 4], c, -mb_run[x]));
            sum += p[x][r];
        }
        l_run[x] += sum;
    }
    output((n_tiles - 1) & 3, pack());

    // ---- normalise, round once, store: a lane owns runs of 4 consecutive output columns of its two queries -------------------------
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float inv = 1.0f / quarter_wave_sum(l_run[x]);
        const int q = q0 + 16 * x + l16;
        char* const orow = Oh + (int64_t)q * rb + quarter * 8;
        if (q < N)
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const u32x2 w = {pack_bf16x2(oacc[b][x][0] * inv, oacc[b][x][1] * inv), pack_bf16x2(oacc[b][x][2] * inv, oacc[b][x][3] * inv)};
                *reinterpret_cast<u32x2*>(orow + b * 32) = w;
            }
    }
}

template <int DVB, bool HALF, int WQ>
hipError_t launch_pipe_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, int q_end, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((q_end + 32 * WQ - 1) / (32 * WQ));
    return launch_by_heads(BH, strips, 64 * WQ, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * (DVB * 32 - (HALF ? 16 : 0));
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_pipe_kernel<DVB, HALF, WQ>), dim3(grid), dim3(64 * WQ), 0, stream, static_cast<const uint16_t*>(Q) + at,
                           static_cast<const uint16_t*>(K) + at, static_cast<const uint16_t*>(V) + at, static_cast<uint16_t*>(O) + at, N,
                           fabsf(scale) * kLog2e, scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u, strips, total);
        return hipGetLastError();
    });
}

template <int DVB, bool HALF>
hipError_t launch_pipe_d(int waves, const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, int q_end, hipStream_t stream)
{
    return waves == 4 ? launch_pipe_t<DVB, HALF, 4>(Q, K, V, O, BH, N, scale, q_end, stream)
                      : launch_pipe_t<DVB, HALF, 8>(Q, K, V, O, BH, N, scale, q_end, stream);
}

}  // namespace

bool attention_pipe_supported(int64_t N, int64_t d) { return d >= 96 && d <= 160 && d % 16 == 0 && N > 128; }

// Waves of a workgroup for this shape, 0 where attention_wide_kernel is the faster one.  That one takes 120 to 170 registers: with workgroups of four
// waves three or four of them share a SIMD, which hides as much as the order here does, and one workgroup's first and last tiles hide under another's
// middle.  So it keeps (time here / there, rows alike; rows of every sharpness 0.01 to 0.05 more) d = 80 (1.0 to 1.14), d = 96 from the second round of 256-query strips on
// (1.02 to 1.16), d = 112 from the third (1.0 to 1.07), short rows of few heads (up to 1.1), and of more rounds those of up to 256, 512, 768, then 1024 tokens at d = 128
// (0.99 to 1.16), of up to 1024, then 1536 at 144 and 160 (1.02 to 1.07).  A second round that is less than half
// full is the faster one there too (1.05 to 1.15; d = 128 0.93 to 0.98).  One round: d = 96 0.93 to 0.98, 112 0.92 to 0.97, 128 0.86 to 0.97, 144 0.82 to
// 0.95, 160 0.78 to 0.92; more rounds of long rows 0.90 to 0.99.  (6700 random shapes of 129 to 12000 tokens.)
int attention_pipe_waves(int64_t BH, int64_t N, int64_t d)
{
    if (!attention_pipe_supported(N, d)) return 0;
    const int64_t cus = compute_units(), fours = BH * ((N + 127) / 128), eights = BH * ((N + 255) / 256), rounds = (eights + cus - 1) / cus;
    const int64_t last = (fours + 2 * cus - 1) % (2 * cus) + 1;        // workgroups of four waves in the last round of theirs
    bool take;
    if (rounds == 1) take = N > 352 || 2 * fours > cus;
    else if (d == 96) take = false;
    else if (d == 128) take = N > (rounds == 2 ? 256 : rounds == 3 ? 512 : rounds <= 6 ? 768 : 1024);
    else if (rounds == 2) take = last > cus;
    else take = d != 112 && N > (rounds == 3 ? 1024 : 1536) && rounds <= 12;
    if (!take) return 0;
    // Workgroups of four, two to a compute unit, move K and V twice as often: three hundredths more time a round; a last round of one to a
    // compute unit takes two thirds of that.
    const double cost4 = 1.03 * (double)((fours - last) / (2 * cus)) + (last <= cus ? 0.65 : 1.03);
    return (double)rounds <= cost4 ? 8 : 4;
}

// d = 64: workgroups of four waves against attention_kernel's 256 or 512 queries.  The work of a tile takes as long here, but the rounds end in smaller steps,
// and a ragged end costs a tile of 32 keys instead of one of 128.  So (time here / there; fewer workgroups than half of a round are attention_ranges'
// before this is asked; 323 shapes on both sides of the lines):
//   one round of 256-query strips: ragged rows up to 1056 tokens 0.76 to 0.93, from 1100 on, where the first tiles no longer count, 0.995 to 1.04; whole rows
//     up to 1.07;
//   up to one round of those of four, the strips of 256 queries in a second: 0.72 to 0.93;
//   the second round of those of four at most half full, where two rounds here are as many strips as one there: 0.77 to 0.88; whole rows 0.84 to 1.01, from 8192 on
//     0.97 to 1.03 (left); more than half full: ragged rows up to 1024 tokens 0.7 to 0.93, longer ones 0.91 to 1.09 (left);
//   three rounds and more: ragged rows 0.75 to 0.99, beyond 4096 tokens with the last round more than 0.55 full 0.98 to 1.0 (left); whole ones up to 1.06 beyond 1024
//     tokens (left).
// A last strip of up to 64 queries that follows as a launch of its own there: 1.07 to 1.16 beyond 1024 tokens (left).  us: 275 heads of N = 576 65.9 -> 38.4, 331 of 672
// 76.7 -> 53.0, 134 of 512 0.83 of the time.  (Few heads stay with attention_ranges.hip also because of its waves' references of their own: sharp rows 1.8e-3
// off, here 1.9e-3 to 2.0e-3.)
bool attention_pipe_64(int64_t BH, int64_t N)
{
    const int64_t cus = compute_units(), fours = BH * ((N + 127) / 128), eights = BH * ((N + 255) / 256), last = (fours + 2 * cus - 1) % (2 * cus) + 1;
    const int64_t full = N / 256, tail = N % 256;
    if (N <= 320) return false;
    if (eights <= cus) return tail != 0 && N <= 1056;
    if (fours <= 2 * cus) return true;
    if (N > 1024 && tail >= 1 && tail <= 64 && (BH * full + cus - 1) / cus < (eights + cus - 1) / cus) return false;
    if (fours <= 4 * cus) return tail == 0 ? last <= cus && N < 8192 : N <= 1024 || last <= cus;
    return N <= 1024 || (tail != 0 && (N <= 4096 || 100 * last <= 55 * 2 * cus));
}

// d = 32 (three times the vector work per product): ragged rows of 321 to 1024 tokens alone, 0.64 (285 heads of N = 340 20.1 -> 13.0 us) to 0.94, of 1000 tokens 1.0 to
// 1.02; from 1100 on 1.06 to 1.23, whole rows 0.86 to 1.2.
bool attention_pipe_32(int64_t, int64_t N) { return N > 320 && N <= 1024 && N % 256 != 0; }

hipError_t launch_attention_pipe(int waves, const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d, float scale,
                                 int q_end, hipStream_t stream)
{
    switch ((int)(d / 16)) {
    case 2: return launch_pipe_t<1, false, 4>(Q, K, V, O, BH, (int)N, scale, q_end, stream);   // (attention_pipe_32)
    case 4: return launch_pipe_t<2, false, 4>(Q, K, V, O, BH, (int)N, scale, q_end, stream);   // (attention_pipe_64)
    case 6: return launch_pipe_d<3, false>(waves, Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 7: return launch_pipe_d<4, true>(waves, Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 8: return launch_pipe_d<4, false>(waves, Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 9: return launch_pipe_d<5, true>(waves, Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 10: return launch_pipe_d<5, false>(waves, Q, K, V, O, BH, (int)N, scale, q_end, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
