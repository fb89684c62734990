// Attention output  O = softmax(scale * Q K^T) V  in fp32 for many heads (d a multiple of 4 up to 32, any N): both
// contractions on the bf16 matrix instruction, every operand as three bf16 parts (split_f32.h).
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the product
// with V is what the section "Limitations and future Directions" names as the next thing to fuse.  The
// max-subtracted softmax of the Softmax section, Eq. 1, is applied incrementally as in the other kernels.)
//
// What bounds it: the vector ALU (weights and their parts) beside the matrix instruction (12 x 32 cycles per 32 queries, 32 keys and 16 columns of d, where the
// fp32 instruction takes 16 x 64).  Eight waves of 32 queries share a tile of 32 keys: splitting a
// K or V element costs six vector instructions, spread over 256 queries.  A thread loads 8 elements of a row, splits them
// and writes a 16-byte chunk to each of the three planes of the tile; planes lie as rows in memory do, chunks
// swizzled, and V is turned by the transposing LDS read.  Double buffered, one barrier per tile.  (From d = 36 on: attention_f32_turns.hip.)
// Measured, 16 heads of N = 4096, d = 32, against the fp32 instruction: 290 -> 186 us.
#include "attention_common.h"
#include "launchers.h"
#include "split_f32.h"

namespace attnw {
namespace {

// Columns past d are zeros on chip.  Rows past N are read as row N - 1, weigh nothing and are not stored.
__global__ __launch_bounds__(512)
void attention_f32_split_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                                float* __restrict__ O, int N, int d, float c, float q_sign, uint32_t strips, uint32_t total)
{
    using L = RowLayout<1>;
    constexpr int NW = 8, BN = 32;
    constexpr int DB = 64;                        // bytes of a row of a plane: 32 columns
    constexpr int CPR = 4;                        // 16-byte chunks of it
    constexpr int PLANE = BN * DB;
    constexpr int BUF_BYTES = 6 * PLANE;          // K hi, mid, lo, V hi, mid, lo
    constexpr int G = 2;                          // 16-column contraction groups

    __shared__ __align__(1024) char lds[2 * BUF_BYTES];
    __shared__ int k_large[NW];                   // a wave has brought a |K| beyond kLarge, beyond kHuge (1, 2)

    const uint32_t logical = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (logical >= total) return;
    const uint32_t bh = logical / strips;
    const uint32_t strip = logical - bh * strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const float* Qh = Q + (int64_t)bh * N * d;
    const float* Kh = K + (int64_t)bh * N * d;
    const float* Vh = V + (int64_t)bh * N * d;
    float* Oh = O + (int64_t)bh * N * d;
    const int q0 = strip * 32 * NW + wave * 32;

    float q_max = 0.0f;
    Split8 qf[G];                                 // (q_sign: a negative scale negates Q)
    {
        const float* qrow = Qh + (int64_t)min(q0 + l32, N - 1) * d;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int col = g * 16 + half * 8;
            const Row8 row = load_row8(qrow, col, d);
            q_max = fmaxf(q_max, largest(row));
            qf[g] = split_row8(row, col, d, q_sign * kSplitUp);
        }
    }
    // From 2^80 on, either way, a score in parts is infinite also where fp32 holds it, and one of -infinity leaves no trace in the sums.
    // No score of 128 products gets there while |Q| and |K| stay within 2^20 and 2^52, either of them the larger one; waves whose
    // operands do not start again on the fp32 instruction.  (Six instructions per 32 keys, before
    // the split, and nothing kept but scalar masks: 16 heads of N = 4096, d = 32 192.5 us with and without.  The smallest score beside the sums, a vector
    // register and eight instructions: 199.)
    constexpr float kLarge = 0x1p20f, kHuge = 0x1p52f;
    const uint64_t q_large = __builtin_amdgcn_ballot_w64(q_max > kLarge), q_huge = __builtin_amdgcn_ballot_w64(q_max > kHuge);
    uint64_t large = 0, huge = 0;                 // of K

    // ---- tiles: waves 0 and 1 bring the 128 chunks of K, 2 and 3 those of V -------------------------------------------------
    const bool v = wave >= 2;
    const int at = (wave & 1) * 64 + lane, key = at / CPR, ch = at % CPR;
    Row8 reg;
    auto load = [&](int t) __attribute__((always_inline)) {
        if (wave < 4) reg = load_row8((v ? Vh : Kh) + (int64_t)min(t * BN + key, N - 1) * d, ch * 8, d);
    };
    auto store = [&](int buf) __attribute__((always_inline)) {
        if (wave >= 4) return;
        const float k_max = largest(reg);
        large |= __builtin_amdgcn_ballot_w64(k_max > kLarge);
        huge |= __builtin_amdgcn_ballot_w64(k_max > kHuge);
        const Split8 x = split_row8(reg, ch * 8, d);
        char* to = lds + buf * BUF_BYTES + (v ? 3 * PLANE : 0) + key * DB + (ch ^ (v ? L::v_block(key) * 4 : L::k_chunk(key))) * 16;
        *reinterpret_cast<u32x4*>(to) = x.hi;
        *reinterpret_cast<u32x4*>(to + PLANE) = x.mid;
        *reinterpret_cast<u32x4*>(to + 2 * PLANE) = x.lo;
    };

    // ---- per-lane places of the operand fragments ------------------------------------------------------------------------
    const char* const krow = lds + l32 * DB;
    int koff[G];
#pragma unroll
    for (int g = 0; g < G; ++g) koff[g] = ((2 * g + half) ^ L::k_chunk(l32)) * 16;
    const int vkey = 4 * half + ((lane & 15) >> 2);            // a lane's row of the 8-key group that it reads
    const char* const vrow = lds + 3 * PLANE + vkey * DB + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    static_assert(L::KPERIOD == G && L::VPERIOD == 1, "rows of one block: those of V are not swizzled");

    f32x16 oacc;
    float mb_run, l_run;
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[r] = 0.0f;
        mb_run = kNegBig;
        l_run = 0.0f;
    };
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent

    // weights of 32 keys from their scores; the reference exponent follows the maximum lazily
    auto weights = [&](const f32x16& s, float c, int key0, float (&p)[16]) __attribute__((always_inline)) {
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        const float m = half_wave_max(fmaxf(tm, s[15]));   // (keys past the end are copies of key N-1: no new maximum)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(m * c > mb_run + kLazy) != 0, 0)) {
            const float mb_new = fmaxf(mb_run, reference_exponent(m, c));
            const float alpha = fast_exp2(mb_run - mb_new);    // exactly 1 for lanes whose exponent stands
            l_run *= alpha;
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[r] *= alpha;
            mb_run = mb_new;
        }
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
    };

    auto compute = [&](int t, int buf) __attribute__((always_inline)) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const char* k = krow + buf * BUF_BYTES + koff[g];
            const Split8 kf = {*reinterpret_cast<const u32x4*>(k), *reinterpret_cast<const u32x4*>(k + PLANE),
                               *reinterpret_cast<const u32x4*>(k + 2 * PLANE)};
            mma_split(s, kf, qf[g]);
        }
        float p[16];
        weights(s, c * kSplitDown, t * BN, p);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = p[8 * m + e] * kSplitUp;
            const Split8 pw = split8(x);          // a lane's weights of group m are its operand of the second contraction
            const char* v = vrow + buf * BUF_BYTES + 16 * m * DB;
            const Split8 vf = {u32x4_of(lds_read_tr16(v), lds_read_tr16(v + 8 * DB)), u32x4_of(lds_read_tr16(v + PLANE), lds_read_tr16(v + PLANE + 8 * DB)),
                               u32x4_of(lds_read_tr16(v + 2 * PLANE), lds_read_tr16(v + 2 * PLANE + 8 * DB))};
            mma_split(oacc, vf, pw);
        }
    };

    // ---- the sweep: while tile t is computed, tile t + 1 is split into the other buffer and tile t + 2 is under way ----------
    reset();
    const int n_tiles = (N + BN - 1) / BN;
    load(0);
    store(0);
    if (n_tiles > 1) load(1);
    __syncthreads();
    for_tiles(0, 0, n_tiles, [&](int t, auto bufc) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        if (t + 1 < n_tiles) {
            store(BUF ^ 1);
            if (t + 2 < n_tiles) load(t + 2);
        } else if (lane == 0) {
            k_large[wave] = wave < 2 ? (large != 0) + (huge != 0) : 0;   // (else of V)
        }
        if (q0 < N) compute(t, BUF);              // (a wave without queries only moves tiles)
        __syncthreads();
    });
    if (q0 >= N) return;

    // ---- infinities, NaN and overflows (rare): what the parts make of them is not what fp32 does.  The wave starts again on
    // the fp32 instruction, operands straight from memory ---------------------------------------------------------------------
    int k_most = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) k_most = max(k_most, k_large[w]);
    float worst = (k_most == 0 ? q_huge : q_large) != 0 || k_most == 2 ? __builtin_inff() : l_run, down = kSplitDown;
#pragma unroll
    for (int r = 0; r < 16; ++r) worst = __builtin_fmaf(oacc[r], 0.0f, worst);   // NaN if any of them is not finite
    if (__builtin_amdgcn_ballot_w64(!(fabsf(worst) < __builtin_inff())) != 0) {
        reset();
        down = 1.0f;
        const float* qrow = Qh + (int64_t)min(q0 + l32, N - 1) * d;
        for (int key0 = 0; key0 < N; key0 += 32) {
            const float* kr = Kh + (int64_t)min(key0 + l32, N - 1) * d;
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.0f;
            for (int col = 0; col < d; col += 4) {             // columns col, col + 1, then col + 2, col + 3
                const f32x4 a = *reinterpret_cast<const f32x4*>(kr + col), b = *reinterpret_cast<const f32x4*>(qrow + col) * q_sign;
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? a[1] : a[0], half ? b[1] : b[0], s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? a[3] : a[2], half ? b[3] : b[2], s, 0, 0, 0);
            }
            float p[16];
            weights(s, c, key0, p);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = key0 + 4 * half + 8 * (r / 4) + (r % 4);
                const float v = Vh[(int64_t)min(key, N - 1) * d + min(l32, d - 1)];
                oacc = __builtin_amdgcn_mfma_f32_32x32x2f32(key < N ? v : 0.0f, p[r], oacc, 0, 0, 0);
            }
        }
    }

    // ---- normalise and store: a lane owns runs of 4 consecutive output columns of its query ----------------------
    const float inv = 1.0f / half_wave_sum(l_run) * down;
    if (q0 + l32 >= N) return;
    float* const orow = Oh + (int64_t)(q0 + l32) * d + half * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x4 o = {oacc[4 * i], oacc[4 * i + 1], oacc[4 * i + 2], oacc[4 * i + 3]};
        if (8 * i + 4 * half < d) *reinterpret_cast<f32x4*>(orow + 8 * i) = o * inv;
    }
}

}  // namespace

hipError_t launch_attention_f32_split(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                      float scale, hipStream_t stream)
{
    if (d > 32) return hipErrorInvalidValue;
    const uint32_t strips = (uint32_t)((N + 255) / 256);
    return launch_by_heads(BH, strips, 512, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * d;
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL(attention_f32_split_kernel, dim3(grid), dim3(512), 0, stream, static_cast<const float*>(Q) + at,
                           static_cast<const float*>(K) + at, static_cast<const float*>(V) + at, static_cast<float*>(O) + at, (int)N, (int)d,
                           fabsf(scale) * kLog2e, scale < 0.0f ? -1.0f : 1.0f, strips, total);
        return hipGetLastError();
    });
}

}  // namespace attnw
