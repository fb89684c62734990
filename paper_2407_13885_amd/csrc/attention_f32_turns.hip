// Attention output  O = softmax(scale * Q K^T) V  in fp32 for many heads, d a multiple of 4 from 36 to 128, any N: operands as three bf16 parts
// (split_f32.h) as in attention_f32_split.hip, with the two waves of a SIMD taking turns at the matrix unit (as in attention_turns.hip).
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; Softmax section, Eq. 1, applied
// incrementally.)
//
// A tile of 32 keys is two phases of a wave with a barrier after each: the output of the tile before and the scores of this one (192 matrix
// instructions of 16 cycles at d = 128), then the weights and their parts, and the wave's share of a coming tile of K and V, split into LDS
// (some 400 vector instructions).  Waves 4 to 7, the other wave of each SIMD, are one phase behind waves 0 to 3.  With one after the other in all
// waves at once the matrix unit was busy 63 % and both units 8 % of the SIMD cycles; here 82 and 27 %.
//
// What bounds it: the board's power (order of the phases, depth of the fragment ring and priority change the time by less than 1 %; the same code with all
// waves in step is 10 % slower).  Hence mma16, and the operand from LDS stays for two to six instructions.  16 heads of N = 4096, all waves in step on 32 x 32
// x 16 / here: d = 64 320 / 284 us, 96 458 / 397, 128 612 / 508 (1.62 PFLOP/s of bf16 products); error against 64 bits 1.06e-6 / 1.05e-6.  Random
// shapes of d = 36 to 128: 52 of 195 come here, 0.82 to 0.965 of the time.  Up to d = 32 the weights are most of the work: 0.98 on long rows, 1.1 on short ones,
// and attention_f32_split.hip stays.
#include "attention_common.h"
#include "launchers.h"
#include "split_f32.h"

namespace attnw {
namespace {

// DVB: 32-column blocks of a row, ceil(d / 32); columns past d are zeros on chip.  Rows past N are read as row N - 1, weigh
// nothing and are not stored.
template <int DVB>
__global__ __launch_bounds__(512)
void attention_f32_turns_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                                float* __restrict__ O, int N, int d, float c, float q_sign, uint32_t strips, uint32_t total)
{
    using L = RowLayout<DVB>;
    constexpr int NW = 8, BN = 32;
    constexpr int DB = DVB * 64;                  // bytes of a row of a plane
    constexpr int CPR = DVB * 4;                  // 16-byte chunks of it
    constexpr int PLANE = BN * DB;
    constexpr int BUF_BYTES = 6 * PLANE;          // K hi, mid, lo, V hi, mid, lo
    constexpr int G = DVB;                        // 32-column contraction groups
    constexpr int CB = DVB * 2;                   // 16-column blocks
    constexpr int CHUNKS = BN * CPR;              // chunks of a plane: the first CHUNKS slots are K's, as many follow of V
    constexpr int SLOTS = (2 * CHUNKS + NW * 64 - 1) / (NW * 64);
    static_assert(CHUNKS % 64 == 0, "a wave's slots are of one tensor");

    __shared__ __align__(1024) char lds[2 * BUF_BYTES];
    __shared__ int k_large[NW];                   // a wave has brought a |K| beyond kLarge, beyond kHuge (1, 2)

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l16 = lane & 15;
    const int quarter = lane >> 4;
    const float* Qh = Q + (int64_t)bh * N * d;
    const float* Kh = K + (int64_t)bh * N * d;
    const float* Vh = V + (int64_t)bh * N * d;
    float* Oh = O + (int64_t)bh * N * d;
    const int q0 = strip * 32 * NW + wave * 32;

    float q_max = 0.0f;
    Split8 qf[2][G];                              // of queries l16, 16 + l16 (q_sign: a negative scale negates Q)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float* qrow = Qh + (int64_t)min(q0 + 16 * x + l16, N - 1) * d;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int col = g * 32 + quarter * 8;
            const Row8 row = load_row8(qrow, col, d);
            q_max = fmaxf(q_max, largest(row));
            qf[x][g] = split_row8(row, col, d, q_sign * kSplitUp);
        }
    }
    // From 2^80 on, either way, a score in parts is infinite also where fp32 holds it, and one of -infinity leaves no trace in the sums.
    // No score of 128 products gets there while |Q| and |K| stay within 2^20 and 2^52, either of them the larger one; waves whose
    // operands do not start again on the fp32 instruction.  (Six instructions per 32 keys, before
    // the split, and nothing kept but scalar masks.)
    constexpr float kLarge = 0x1p20f, kHuge = 0x1p52f;
    const uint64_t q_large = __builtin_amdgcn_ballot_w64(q_max > kLarge), q_huge = __builtin_amdgcn_ballot_w64(q_max > kHuge);
    uint64_t large = 0, huge = 0;                 // of K

    // ---- tiles: slot s of a tile is chunk s of K or chunk s - CHUNKS of V --------------------------------------------------
    static_assert(CHUNKS <= NW * 64, "all of K in the first slots");
    Row8 reg[SLOTS];                              // of K tile tk, V tile tk - 1
    const int n_tiles = (N + BN - 1) / BN;
    auto load = [&](int tk) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) {
            const int w = wave + NW * j;          // (wave-uniform: which tensor, and whether there is such a slot)
            if ((SLOTS * NW * 64 == 2 * CHUNKS || w * 64 < 2 * CHUNKS)) {
                const bool v = w * 64 >= CHUNKS;
                const int t = tk - (v ? 1 : 0);
                if (t < 0 || t >= n_tiles) continue;
                const int s = (v ? w * 64 - CHUNKS : w * 64) + lane;
                const int key = s / CPR;
                reg[j] = load_row8((v ? Vh : Kh) + (int64_t)min(t * BN + key, N - 1) * d, (s - key * CPR) * 8, d);
            }
        }
    };
    auto store = [&](int tk) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) {
            const int w = wave + NW * j;
            if ((SLOTS * NW * 64 == 2 * CHUNKS || w * 64 < 2 * CHUNKS)) {
                const bool v = w * 64 >= CHUNKS;
                const int t = tk - (v ? 1 : 0);
                if (t < 0 || t >= n_tiles) continue;
                const int s = (v ? w * 64 - CHUNKS : w * 64) + lane;
                const int key = s / CPR, ch = s - key * CPR;
                if (j == 0) {
                    const float k_max = largest(reg[j]);
                    large |= __builtin_amdgcn_ballot_w64(k_max > kLarge);
                    huge |= __builtin_amdgcn_ballot_w64(k_max > kHuge);
                }
                const Split8 x = split_row8(reg[j], ch * 8, d);
                char* to = lds + (t & 1) * BUF_BYTES + (v ? 3 * PLANE : 0) + key * DB + (ch ^ (v ? L::v16_block(key) * 2 : L::k_chunk(key))) * 16;
                *reinterpret_cast<u32x4*>(to) = x.hi;
                *reinterpret_cast<u32x4*>(to + PLANE) = x.mid;
                *reinterpret_cast<u32x4*>(to + 2 * PLANE) = x.lo;
            }
        }
    };

    // ---- per-lane places of the operand fragments ------------------------------------------------------------------------
    const char* const krow = lds + l16 * DB;
    constexpr int KPERIOD = L::KPERIOD / 2, VPERIOD = L::V16PERIOD;
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((4 * g + quarter) ^ L::k_chunk(l16)) * 16;
    const int vkey = 4 * quarter + (l16 >> 2);    // a lane's row of the 16 keys that it reads
    const char* const vrow = lds + 3 * PLANE + vkey * DB + (lane & 3) * 8;
    int voff[VPERIOD];
#pragma unroll
    for (int b = 0; b < VPERIOD; ++b) voff[b] = (b ^ L::v16_block(vkey)) * 32;
    // plane 0, 1, 2: hi, mid, lo; keys 16 (f % 2) .. + 15 x columns 32 (f / 2) .. + 31 (8 a lane)
    auto k_frag = [&](int buf, int f, int plane) __attribute__((always_inline)) {
        const int g = f / 2;
        return *reinterpret_cast<const u32x4*>(krow + buf * BUF_BYTES + plane * PLANE + (f % 2) * 16 * DB + (g / KPERIOD) * KPERIOD * 64 + koff[g % KPERIOD]);
    };
    // 16 columns x 32 keys: of a lane keys 4 quarter .. + 3 and 16 more than these, as its weights
    auto v_frag = [&](int buf, int b, int plane) __attribute__((always_inline)) {
        const char* p = vrow + buf * BUF_BYTES + plane * PLANE + (b / VPERIOD) * VPERIOD * 32 + voff[b % VPERIOD];
        return u32x4_of(lds_read_tr16(p), lds_read_tr16(p + 16 * DB));
    };

    f32x4 oacc[CB][2];                            // columns 16 b + 4 quarter .. + 3 of queries l16, 16 + l16
    float mb_run[2], l_run[2];
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int b = 0; b < CB; ++b) oacc[b][x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            mb_run[x] = kNegBig;
            l_run[x] = 0.0f;
        }
    };
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent
    f32x4 s[2][2];                                // scores of a tile: keys 16 k + 4 quarter .. + 3, queries 16 x + l16
    float p[2][8];                                // its weights
    auto zero_scores = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int x = 0; x < 2; ++x) s[k][x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };

    // weights of 32 keys from their scores; the reference exponent follows the maximum lazily (keys past the end are copies of key N-1: no new
    // maximum)
    auto weights = [&](float c, int key0, bool ragged) __attribute__((always_inline)) {
        float top[2];
#pragma unroll
        for (int x = 0; x < 2; ++x)
            top[x] = fmaxf(max3(max3(max3(s[0][x][0], s[0][x][1], s[0][x][2]), s[0][x][3], s[1][x][0]), s[1][x][1], s[1][x][2]), s[1][x][3]);
        const float ahead[2] = {__builtin_fmaf(top[0], c, -mb_run[0]), __builtin_fmaf(top[1], c, -mb_run[1])};
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(fmaxf(ahead[0], ahead[1]) > kLazy) != 0, 0)) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                if (__builtin_amdgcn_ballot_w64(ahead[x] > kLazy) == 0) continue;
                const float mb_new = fmaxf(mb_run[x], reference_exponent(quarter_wave_max(top[x]), c));
                const float alpha = fast_exp2(mb_run[x] - mb_new);       // exactly 1 for lanes whose exponent stands
                l_run[x] *= alpha;
#pragma unroll
                for (int b = 0; b < CB; ++b) oacc[b][x] *= alpha;
                mb_run[x] = mb_new;
            }
        }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int r = 0; r < 8; ++r) p[x][r] = fast_exp2(__builtin_fmaf(s[r / 4][x][r % 4], c, -mb_run[x]));
        if (ragged) {                             // keys past the end weigh nothing
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if (key0 + 16 * (r / 4) + 4 * quarter + r % 4 >= N) p[x][r] = 0.0f;
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            float sum = p[x][0];
#pragma unroll
            for (int r = 1; r < 8; ++r) sum += p[x][r];
            l_run[x] += sum;
        }
    };

    // ---- the two halves of a tile's work: matrix_phase(t) the output of tile t - 1 and the scores of tile t, vector_phase(t) the weights of tile t ----
    Split8 pw[2];
    constexpr int KF = 2 * G, RING = 4;           // fragments of K of a tile; parts of fragments held at a time
    u32x4 ring[RING];
    auto fragment = [&](int t, auto ic) __attribute__((always_inline)) {      // parts lo, mid, hi of one after another
        constexpr int I = decltype(ic)::value, F = I / 3, PL = 2 - I % 3;
        if constexpr (F < CB) return v_frag((t - 1) & 1, F, PL);
        else return k_frag(t & 1, F - CB, PL);
    };
    auto products = [&](f32x4& a0, f32x4& a1, const u32x4& f, const Split8& b0, const Split8& b1, auto plane) __attribute__((always_inline)) {
        constexpr int PL = decltype(plane)::value;
        if constexpr (PL == 0) { mma16(a0, f, b0.lo); mma16(a1, f, b1.lo); }
        if constexpr (PL <= 1) { mma16(a0, f, b0.mid); mma16(a1, f, b1.mid); }
        mma16(a0, f, b0.hi);
        mma16(a1, f, b1.hi);
    };
    auto step = [&](int t, auto ic, auto lastc) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value, F = I / 3, PL = 2 - I % 3;
        const u32x4 f = ring[I % RING];
        if constexpr (F < CB) {
            products(oacc[F][0], oacc[F][1], f, pw[0], pw[1], IC<PL>{});
        } else {
            constexpr int KB = (F - CB) % 2, GR = (F - CB) / 2;
            if constexpr (GR == 0 && PL == 2) s[KB][0] = s[KB][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            products(s[KB][0], s[KB][1], f, qf[0][GR], qf[1][GR], IC<PL>{});
        }
        if constexpr (I + RING < decltype(lastc)::value) ring[I % RING] = fragment(t, IC<I + RING>{});
        __builtin_amdgcn_sched_barrier(0);
    };
    auto steps = [&](int t, auto firstc, auto lastc) __attribute__((always_inline)) {
        constexpr int FIRST = decltype(firstc)::value, LAST = decltype(lastc)::value;
        static_for<RING>([&](auto ic) __attribute__((always_inline)) { ring[(FIRST + decltype(ic)::value) % RING] = fragment(t, IC<FIRST + decltype(ic)::value>{}); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<LAST - FIRST>([&](auto ic) __attribute__((always_inline)) { step(t, IC<FIRST + decltype(ic)::value>{}, IC<LAST>{}); });
    };
    auto vector_phase = [&](int t, bool ragged) __attribute__((always_inline)) {
        weights(c * kSplitDown, t * BN, ragged);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            float up[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) up[e] = p[x][e] * kSplitUp;
            pw[x] = split8(up);                   // a lane's weights are its operand of the second contraction
        }
    };
    auto turn = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        wait_lds();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // ---- phases: in 2t waves 0 .. 3 multiply for tile t while 4 .. 7 make the weights of t - 1, in 2t + 1 the other way round.  All waves stage K of
    // t + 1 and V of t in their weights' phase of these two (K of t - 1 and V of t - 2, whose places they take, were last read in 2t - 1), and they
    // are first read in 2t + 2. ----
    reset();
    load(0);
    store(0);
    load(1);
    turn();
    const int second = wave >= 4 ? 1 : 0;
    auto stage = [&](int tk) __attribute__((always_inline)) {
        store(tk);
        load(tk + 1);
    };
    if (second) {
        stage(1);
        turn();
    }
    if (q0 < N) {
        steps(0, IC<3 * CB>{}, IC<3 * (CB + KF)>{});
        for (int t = 0; t + 1 < n_tiles; ++t) {
            turn();
            vector_phase(t, false);
            stage(t + 1 + second);
            turn();
            __builtin_amdgcn_s_setprio(1);
            steps(t + 1, IC<0>{}, IC<3 * (CB + KF)>{});
            __builtin_amdgcn_s_setprio(0);
        }
        turn();
        vector_phase(n_tiles - 1, true);
        stage(n_tiles + second);
    } else {                                      // (a wave without queries only moves tiles)
        for (int t = 0; t < n_tiles; ++t) {
            if (t > 0) turn();
            turn();
            stage(t + 1 + second);
        }
    }
    if (lane == 0) k_large[wave] = wave * 64 < CHUNKS ? (large != 0) + (huge != 0) : 0;   // (else its first slots are of V)
    turn();
    if (!second) turn();
    if (q0 >= N) return;
    steps(n_tiles, IC<0>{}, IC<3 * CB>{});

    // ---- infinities, NaN and overflows (rare): what the parts make of them is not what fp32 does.  The wave starts again on
    // the fp32 instruction, operands straight from memory, as many bytes to a lane as the instruction's layouts allow (what bounds it are these
    // loads) ------------------------------------------------------------------------------------------------------------------
    int k_most = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) k_most = max(k_most, k_large[w]);
    float worst = (k_most == 0 ? q_huge : q_large) != 0 || k_most == 2 ? __builtin_inff() : l_run[0];
    worst = __builtin_fmaf(l_run[1], 0.0f, worst);
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r) worst = __builtin_fmaf(oacc[b][x][r], 0.0f, worst);   // NaN if any of them is not finite
    if (__builtin_amdgcn_ballot_w64(!(fabsf(worst) < __builtin_inff())) != 0) {
        reset();
        for (int key0 = 0; key0 < N; key0 += 32) {
            zero_scores();
#pragma unroll
            for (int g = 0; g < G; ++g) {         // 32 columns: of a lane chunks of four, element e of each to instruction e
                f32x4 a[2][2], b[2][2];           // [half of them][keys, queries 16 i + l16]
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int col = g * 32 + h * 16 + quarter * 4;
                        a[h][i] = *reinterpret_cast<const f32x4*>(Kh + (int64_t)min(key0 + 16 * i + l16, N - 1) * d + (col < d ? col : 0));
                        b[h][i] = *reinterpret_cast<const f32x4*>(Qh + (int64_t)min(q0 + 16 * i + l16, N - 1) * d + (col < d ? col : 0));
                        a[h][i] = col < d ? a[h][i] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                        b[h][i] = col < d ? b[h][i] * q_sign : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int k = 0; k < 2; ++k)
#pragma unroll
                            for (int x = 0; x < 2; ++x) s[k][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][k][e], b[h][x][e], s[k][x], 0, 0, 0);
            }
            weights(c, key0, key0 + 32 > N);
#pragma unroll
            for (int r = 0; r < 8; ++r) {         // (columns 32 b + 2 l16, + 1 to the first and the second block of the 32)
                const int key = key0 + 16 * (r / 4) + 4 * quarter + r % 4;
                const float* vr = Vh + (int64_t)min(key, N - 1) * d;
#pragma unroll
                for (int b = 0; b < DVB; ++b) {
                    const f32x2 v = *reinterpret_cast<const f32x2*>(vr + min(b * 32 + 2 * l16, d - 2));
#pragma unroll
                    for (int e = 0; e < 2; ++e)
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                            oacc[2 * b + e][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(key < N ? v[e] : 0.0f, p[x][r], oacc[2 * b + e][x], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const float inv = 1.0f / quarter_wave_sum(l_run[x]);
            const int q = q0 + 16 * x + l16;
            float* const orow = Oh + (int64_t)q * d + quarter * 8;
            if (q < N)
#pragma unroll
                for (int b = 0; b < DVB; ++b)
#pragma unroll
                    for (int r = 0; r < 4; r += 2)
                        if (b * 32 + quarter * 8 + 2 * r < d)
                            *reinterpret_cast<f32x4*>(orow + b * 32 + 2 * r) =
                                f32x4{oacc[2 * b][x][r], oacc[2 * b + 1][x][r], oacc[2 * b][x][r + 1], oacc[2 * b + 1][x][r + 1]} * inv;
        }
        return;
    }

    // ---- normalise and store: a lane owns runs of 4 consecutive output columns of its queries ----------------------
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float inv = 1.0f / quarter_wave_sum(l_run[x]) * kSplitDown;
        const int q = q0 + 16 * x + l16;
        float* const orow = Oh + (int64_t)q * d + quarter * 4;
        if (q < N)
#pragma unroll
            for (int b = 0; b < CB; ++b)
                if (b * 16 + quarter * 4 < d) *reinterpret_cast<f32x4*>(orow + b * 16) = oacc[b][x] * inv;
    }
}

template <int DVB>
hipError_t launch_f32_turns_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((N + 255) / 256);
    return launch_by_heads(BH, strips, 512, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * d;
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_f32_turns_kernel<DVB>), dim3(grid), dim3(512), 0, stream, static_cast<const float*>(Q) + at,
                           static_cast<const float*>(K) + at, static_cast<const float*>(V) + at, static_cast<float*>(O) + at, N, d,
                           fabsf(scale) * kLog2e, scale < 0.0f ? -1.0f : 1.0f, strips, total);
        return hipGetLastError();
    });
}

}  // namespace

hipError_t launch_attention_f32_turns(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                      float scale, hipStream_t stream)
{
    switch ((int)((d + 31) / 32)) {
    case 2: return launch_f32_turns_t<2>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 3: return launch_f32_turns_t<3>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    case 4: return launch_f32_turns_t<4>(Q, K, V, O, BH, (int)N, (int)d, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
