// Fused attention weights  P = softmax(scale * Q K^T)  and scaled scores in fp32 for any N and any d a multiple of 4 up to 256: the
// contraction on the bf16 matrix instruction, operands as three bf16 parts (split_f32.h), a strip of 32 queries per workgroup.
//
// (Paper: the fused kernel of the section "Fused Matrix Multiply + Scaling + Softmax" keeps a block of scores in a core's
// SRAM from the multiply to the store; here the registers of a compute unit hold 32 queries x 2048 keys.)
//
// Eight waves share the keys of a strip: wave w owns the 32-key blocks w, w + 8, ...  Nothing of K is shared between waves, so
// each brings its own blocks to LDS (32 keys x 32 columns at a time, NSLOT of them under way), splits them on the way from
// there to the matrix instruction, and meets the others only once per strip, at the exchange of row maxima and sums.  The
// exponentials of the first NT blocks of a wave stay in its registers.  They become weights while the next strip is computed:
// step j of a strip first stages block j of the strip before and then fills its registers with block j of this one, so
// that the stores of a strip leave evenly under the arithmetic of the next.  Blocks beyond NT (N > 256 NT) are computed twice, as
// in the two-sweep kernels.
//
// Why 32 queries: a compute unit's registers hold 32 x 2048 scores beside the operands, and one sweep needs half the matrix
// instructions and exponentials of two; a few short heads then also spread over four times the compute units.  Measured, two
// heads of N = 2976, d = 84: 416 us on the fp32 instruction with the keys split over workgroups, 60 here; 16 heads of N = 2048, d = 64 116 us in
// two sweeps over 128-query strips, 105 here (on the same inputs again 101; d = 128 199 -> 162); one head of N = 128, d = 64 8.9 -> 7.7 (5.4).
// What bounds it (16 heads of N = 2048, d = 64): the vector ALU, 53 % of SIMD cycles (per wave and block of 32 keys 382 instructions, some
// 200 of them splitting), with the matrix pipe beside it (25 %, both at once 9 %), and the time that a wave needs to issue its K
// transfers (75 cycles each, a tenth of its life); the waves wait 34 % of theirs.  With NT = 8 the 256 registers are full: two vector and 25
// scalar ones are spilled.  Taken out one at a time: splitting 20 us, stores 11, transfers 6, matrix instructions 4.  Interleaving the
// split of one group with the matrix instructions of the other by hand changed nothing (the two waves of a SIMD do that for each other)
// and spilled.
#include "attention_common.h"
#include "launchers.h"
#include "split_f32.h"

namespace attnw {
namespace {

__device__ __forceinline__ void workgroup_barrier()   // (LDS only: transfers and stores under way stay so)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}
// The number, where the compiler does not know it: what is computed from it stays where it stands (hoisted out of the strip loop,
// the conditions and addresses of every unrolled step spill scalar registers by the hundred).
__device__ __forceinline__ int opaque(int x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(x));
#endif
    return x;
}
template <int N> __device__ __forceinline__ void wait_transfers()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}

// NT: blocks of a wave whose exponentials stay in registers.  NP: the most 32-column panels of a row (2, 4 or 8).  Rows past N are
// read as row N - 1, weigh nothing and are not stored.
template <int NT, int NP, bool SCORES>
__global__ __launch_bounds__(512)
void qk_f32_strip_kernel(const float* __restrict__ Q, const float* __restrict__ K, float* __restrict__ P, int N, int d, float c,
                         float q_sign, uint32_t strips, uint32_t total, uint32_t workers)
{
    constexpr int NW = 8;
    constexpr int NSLOT = NP <= 2 ? 3 : 2;        // panels of a wave under way (LDS)
    constexpr int SLOT = 32 * 128;                // 32 keys x 32 columns
    constexpr int UNIT_OPS = 4;                   // transfers of 1 KiB
    constexpr int ST_BYTES = 32 * 128;            // staged block: 32 rows of 32 weights, 16-byte chunks swizzled by the row
    constexpr int QG = NP * 2;                    // 16-column contraction groups
    constexpr int K_BYTES = NW * NSLOT * SLOT;
    constexpr int Q_BYTES = QG * 3 * 1024;
    constexpr bool OWN_RAW = NP <= 4;             // LDS for the next strip's Q as it comes from memory; with d > 128 the staging areas take it
    constexpr int RAW_BYTES = OWN_RAW ? 4 * NP * 128 : ST_BYTES;   // of a wave: four rows
    __shared__ __align__(1024) char lds[K_BYTES + (OWN_RAW ? NW * RAW_BYTES : 0) + NW * ST_BYTES + Q_BYTES];   // (the transfers' part first)
    __shared__ float stat_lds[SCORES ? 2 : NW * 64];
    static_assert(K_BYTES + NW * RAW_BYTES <= kDirectLds, "transfers go there");

    const uint32_t worker = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (worker >= workers) return;
    const uint32_t first = (uint32_t)((uint64_t)total * worker / workers), last = (uint32_t)((uint64_t)total * (worker + 1) / workers);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int row_bytes = d * 4;
    const int np = (d + 31) / 32;                 // panels of a row
    const int all_blocks = (N + 31) / 32;
    const int nb = (all_blocks - wave + NW - 1) / NW;           // blocks of this wave (0 where N <= 32 wave)
    const int again = SCORES ? 0 : max(0, nb - NT);             // of these computed twice
    const int seq = nb + again;                                 // blocks computed per strip
    // (workgroups start their sweeps at different blocks: in step, the rows that they write at one moment lie on the same few
    // memory channels)
    const int rot = nb > 0 ? (int)((worker * 7u) % (uint32_t)nb) : 0;
    auto key_of = [&](int j) __attribute__((always_inline)) {   // first key of the j-th block of the sequence
        int b = (j < nb ? j : j - nb + NT) + rot;
        b = b >= nb ? b - nb : b;
        return (b * NW + wave) * 32;
    };
    char* const k_lds = lds + wave * (NSLOT * SLOT);
    char* const raw_q = lds + K_BYTES + wave * RAW_BYTES;
    char* const stage = lds + K_BYTES + (OWN_RAW ? NW * RAW_BYTES : 0) + wave * ST_BYTES;
    char* const q_lds = lds + sizeof(lds) - Q_BYTES;
    const uint32_t k_base = __builtin_amdgcn_readfirstlane(lds_offset_of(k_lds));
    const uint32_t raw_base = __builtin_amdgcn_readfirstlane(lds_offset_of(raw_q));

    // ---- K: the panels of the wave's blocks, strip after strip, NSLOT of them under way --------------------------------------
    // Transfer i of a panel brings keys 8 i .. 8 i + 7, lane l the chunk of key l / 8 that belongs at place l % 8 (16-byte chunks
    // swizzled by the key: eight consecutive keys of one chunk lie in different banks).
    const int k_row = lane >> 3, k_chunk = (lane & 7) ^ k_row;
    uint32_t s_strip = first % strips;            // of the panel to request next
    const char* s_head = reinterpret_cast<const char*>(K) + (int64_t)(first / strips) * N * row_bytes;
    uint32_t s_left = last - first;
    int s_j = 0, s_p = 0, s_slot = 0;
    auto request = [&]() __attribute__((always_inline)) {
        const int key0 = key_of(s_j);
        const uint32_t at = k_base + (uint32_t)s_slot * SLOT;
        const bool whole = key0 + 32 <= N && (s_p + 1) * 32 <= d;
        if (whole) {
            const uint32_t off = (uint32_t)(k_row * row_bytes + k_chunk * 16);
            const char* src = s_head + (int64_t)key0 * row_bytes + s_p * 128;
#pragma unroll
            for (int i = 0; i < UNIT_OPS; ++i) dma16_untracked(src + i * 8 * row_bytes, off, at + i * 1024);
        } else {                                  // (chunks past the row's end: its first one, which meets zeros of Q)
            const int col = s_p * 128 + k_chunk * 16;
            const uint32_t off = (uint32_t)(col < row_bytes ? col : 0);
#pragma unroll 1
            for (int i = 0; i < UNIT_OPS; ++i)
                dma16_untracked(s_head, (uint32_t)(min(key0 + 8 * i + k_row, N - 1) * row_bytes) + off, at + i * 1024);
        }
        s_slot = s_slot + 1 == NSLOT ? 0 : s_slot + 1;
        if (++s_p < np) return;
        s_p = 0;
        if (++s_j < seq) return;
        s_j = 0;
        if (s_left > 1) {                         // (behind the last panel the sequence of the last strip comes again, unused)
            --s_left;
            if (++s_strip == strips) {
                s_strip = 0;
                s_head += (int64_t)N * row_bytes;
            }
        }
    };

    // ---- Q: as it lies in memory to LDS (each wave four rows), from there split into the operand layout ------------------------
    // part x of group g: 1 KiB of 16 bytes per lane of the matrix instruction
    const int q_ops = (16 * d + 1023) / 1024;
    auto request_q = [&](uint32_t unit) __attribute__((always_inline)) {
        const uint32_t bh = unit / strips, strip = unit - bh * strips;
        const char* head = reinterpret_cast<const char*>(Q) + (int64_t)bh * N * row_bytes;
        const int end = N * row_bytes - 16;       // (rows past the end: any numbers of the head)
        for (int i = 0; i < q_ops; ++i) {
            const int off = (int)(strip * 32 + wave * 4) * row_bytes + min(i * 1024 + lane * 16, 16 * d - 16);
            dma16_untracked(head, (uint32_t)min(off, end), raw_base + i * 1024);
        }
    };
    auto split_q = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < (NP + 3) / 4; ++i) {
            const int x = i * 64 + lane;          // chunk of 8 columns of the wave's four rows
            const int row = x / (4 * np), ch = x - row * 4 * np;
            if (x >= 16 * np) continue;
            const Row8 r = load_row8(reinterpret_cast<const float*>(raw_q) + row * d, ch * 8, d);
            const Split8 s = split_row8(r, ch * 8, d, q_sign * kSplitUp);
            char* to = q_lds + (ch >> 1) * 3072 + ((ch & 1) * 32 + wave * 4 + row) * 16;
            *reinterpret_cast<u32x4*>(to) = s.hi;
            *reinterpret_cast<u32x4*>(to + 1024) = s.mid;
            *reinterpret_cast<u32x4*>(to + 2048) = s.lo;
        }
    };

    // ---- scores of the next block of the sequence: accumulator r is key key0 + 4 half + 8 (r / 4) + r % 4, query l32 ----------
    // The panel to compute is in registers already (raw); while it is split and multiplied the next one is read from LDS, and the
    // place that it came from is requested again.
    // young: stores that the step before has issued last (0 where their number is not known): they are younger than the transfers
    // that the first panels wait for
    int slot = 0;                                 // of the panel in registers
    const int k_swz = l32 & 7;
    f32x4 raw[2][2];                              // [group][half of its 8 columns]
    auto fetch = [&]() __attribute__((always_inline)) {
        const char* const row = k_lds + slot * SLOT + l32 * 128;
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int x = 0; x < 2; ++x) raw[g][x] = *reinterpret_cast<const f32x4*>(row + ((4 * g + 2 * half + x) ^ k_swz) * 16);
    };
    auto scores = [&](int young) __attribute__((always_inline)) {
        f32x16 s, rest;                           // (two sums: the matrix instructions of one need not wait for each other's results)
        auto panel = [&](int p) __attribute__((always_inline)) {
            wait_lds();                           // the panel has arrived in registers: its place is free
            float x[2][8];
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[g][e] = raw[g][0][e] * kSplitUp;
                    x[g][4 + e] = raw[g][1][e] * kSplitUp;
                }
            request();
            slot = slot + 1 == NSLOT ? 0 : slot + 1;
            if (young == 0 || p >= NSLOT - 1) wait_transfers<UNIT_OPS * (NSLOT - 1)>();
            else if (young == 4) wait_transfers<UNIT_OPS * (NSLOT - 1) + 4>();
            else wait_transfers<UNIT_OPS * (NSLOT - 1) + 16>();
            const char* const q = q_lds + 2 * p * 3072 + lane * 16;
            Split8 qf[2];
#pragma unroll
            for (int g = 0; g < 2; ++g)
                qf[g] = {*reinterpret_cast<const u32x4*>(q + g * 3072), *reinterpret_cast<const u32x4*>(q + g * 3072 + 1024),
                         *reinterpret_cast<const u32x4*>(q + g * 3072 + 2048)};
            fetch();
#pragma unroll
            for (int g = 0; g < 2; ++g) mma_split(s, rest, split8(x[g]), qf[g]);
        };
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = rest[r] = 0.0f;
        panel(0);
        for (int p = 1; p < np; ++p) panel(p);
        return s + rest;
    };

    // ---- the wave's staged 32 x 32 block to P; returns the number of stores if every lane issued them -----------------------------
    const bool vec = N % 4 == 0, lines = N % 32 == 0;
    auto stage_put = [&](int r4, const f32x4& v) __attribute__((always_inline)) {
        *reinterpret_cast<f32x4*>(stage + l32 * 128 + ((2 * r4 + half) ^ k_swz) * 16) = v;
    };
    auto put = [&](const f32x16& v, float f) __attribute__((always_inline)) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) stage_put(r4, f32x4{v[4 * r4] * f, v[4 * r4 + 1] * f, v[4 * r4 + 2] * f, v[4 * r4 + 3] * f});
    };
    auto flush = [&](float* Ph, int q0, int key0) __attribute__((always_inline)) -> int {
        const bool full = q0 + 32 <= N && key0 + 32 <= N;
        if (full && vec) {
            char* const to = reinterpret_cast<char*>(Ph + (int64_t)q0 * N + key0);
            const uint32_t off = (uint32_t)((lane / 8) * N + (lane % 8) * 4) * 4u;
            f32x4 v[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) v[it] = *reinterpret_cast<const f32x4*>(stage + (it * 8 + lane / 8) * 128 + k_chunk * 16);
            if (lines) {                          // whole lines past the caches: K stays in L2
#pragma unroll
                for (int it = 0; it < 4; ++it) __builtin_nontemporal_store(v[it], reinterpret_cast<f32x4*>(to + (int64_t)(it * 8) * N * 4 + off));
            } else {
#pragma unroll
                for (int it = 0; it < 4; ++it) *reinterpret_cast<f32x4*>(to + (int64_t)(it * 8) * N * 4 + off) = v[it];
            }
            return 4;
        }
        if (full) {                               // rows off the 16-byte boundaries
            float* const to = Ph + (int64_t)(q0 + half) * N + key0 + l32;
#pragma unroll 4
            for (int it = 0; it < 16; ++it) {
                const int row = it * 2 + half;
                to[(int64_t)(it * 2) * N] = *reinterpret_cast<const float*>(stage + row * 128 + ((l32 / 4) ^ (row & 7)) * 16 + (l32 % 4) * 4);
            }
            return 16;
        }
        if (key0 + l32 < N) {
            float* const to = Ph + (int64_t)(q0 + half) * N + key0 + l32;
#pragma unroll 1
            for (int row = half; row < min(32, N - q0); row += 2)
                to[(int64_t)(row - half) * N] = *reinterpret_cast<const float*>(stage + row * 128 + ((l32 / 4) ^ (row & 7)) * 16 + (l32 % 4) * 4);
        }
        return 0;
    };

    // ---- the fp32 instruction on operands straight from memory, for what the parts cannot hold (infinities, NaN, overflows) ------
    auto scores_f32 = [&](const float* Qh, const float* Kh, int q0, int key0) __attribute__((always_inline)) {
        const float* kr = Kh + (int64_t)min(key0 + l32, N - 1) * d;
        const float* qr = Qh + (int64_t)min(q0 + l32, N - 1) * d;
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
        for (int col = 0; col < d; col += 4) {                 // columns col, col + 1, then col + 2, col + 3
            const f32x4 a = *reinterpret_cast<const f32x4*>(kr + col), b = *reinterpret_cast<const f32x4*>(qr + col) * q_sign;
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? a[1] : a[0], half ? b[1] : b[0], s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? a[3] : a[2], half ? b[3] : b[2], s, 0, 0, 0);
        }
        return s;
    };

    // Running maximum and sum of exponentials over the lane's keys.  Exponentials refer to the rounded exponent e_run = fl(c max):
    // one rounding each, and factors between references are exactly 1 while the maximum stands.
    const float c_parts = c * kSplitDown;         // for scores of operands in parts
    // In parts a score below -2^80 is -infinity, also where fp32 holds it, and would weigh nothing: it makes the sum NaN (an
    // infinite maximum, or a NaN, does so by itself).
    float m_run, e_run, l_run;
    auto fold = [&](f32x16& s, float c, int key0, auto partsc) __attribute__((always_inline)) {   // the scores become exponentials
        float low = 0.0f;
        if constexpr (decltype(partsc)::value != 0) {
            low = fminf(s[0], s[1]);
#pragma unroll
            for (int r = 2; r < 16; r += 2) low = min3(low, s[r], s[r + 1]);
        }
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        m_run = fmaxf(m_run, fmaxf(tm, s[15]));                // (keys past the end are copies of key N - 1: no new maximum)
        // (In parts as it is: where the keys of a lane are all masked and the rounding makes their weights infinite, the strip starts again.)
        const float en = decltype(partsc)::value != 0 ? m_run * c : fmaxf(e_run, reference_exponent(m_run, c));
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = fast_exp2(__builtin_fmaf(s[r], c, -en));
        if (key0 + 32 > N) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + 4 * half + 8 * (r / 4) + (r % 4) >= N) s[r] = 0.0f;
        }
        float sum = s[0];
        if constexpr (decltype(partsc)::value != 0) sum = __builtin_fmaf(low, 0.0f, sum);
#pragma unroll
        for (int r = 1; r < 16; ++r) sum += s[r];
        l_run = __builtin_fmaf(l_run, fast_exp2(e_run - en), sum);
        e_run = en;
    };
    // The maximum over no keys.  In parts the lowest number there is: scores carry a factor of 2^48, and behind a higher one the
    // exponentials of scores below it come out small, imprecise or zero.
    auto fold_begin = [&](float m, float e) __attribute__((always_inline)) {
        m_run = m;
        e_run = e;
        l_run = 0.0f;
    };
    auto merge_halves = [&]() __attribute__((always_inline)) {   // the keys of the other half-wave
        const float e = __shfl_xor(e_run, 32, 64), l = __shfl_xor(l_run, 32, 64);
        const float en = fmaxf(e_run, e);
        l_run = l_run * fast_exp2(e_run - en) + l * fast_exp2(e - en);
        e_run = en;
    };

    request_q(first);
    if (seq > 0) {
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) request();
    }
    wait_transfers<0>();
    if (seq > 0) {
        fetch();
    }
    split_q();
    workgroup_barrier();

    f32x16 kept[SCORES ? 1 : NT];                 // exponentials of the strip before
    float e_kept[SCORES ? 1 : NT];                // the exponents that they refer to
    float e_row = 0.0f, inv_row = 0.0f;           // the exponent and the inverse sum of the rows of the strip before
    bool pending = false;                         // it still has to be written
    float* P_before = P;
    int q0_before = 0;
    uint32_t bad_first = last, bad_last = 0;      // strips with rows that the parts cannot hold

    for (uint32_t unit = first; unit < last; ++unit) {
        const uint32_t bh = unit / strips, strip = unit - bh * strips;
        const int q0 = strip * 32;
        float* const Ph = P + (int64_t)bh * N * N;
        if constexpr (SCORES) {
            if (OWN_RAW && unit + 1 < last) request_q(unit + 1);
            for (int j = 0; j < nb; ++j) {
                const int key0 = key_of(j);
                f32x16 s = scores(0);
                float bad = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) bad = __builtin_fmaf(s[r], 0.0f, bad);
                float by = c_parts;
                if (__builtin_amdgcn_ballot_w64(bad != 0.0f) != 0) {
                    s = scores_f32(Q + (int64_t)bh * N * d, K + (int64_t)bh * N * d, q0, key0);
                    by = c;
                }
                put(s, by);
                flush(Ph, q0, key0);
            }
            if (!OWN_RAW && unit + 1 < last) {
                wait_lds();
                request_q(unit + 1);
            }
            if (OWN_RAW && seq * np >= NSLOT) wait_transfers<NSLOT * UNIT_OPS>();
            else wait_transfers<0>();
            workgroup_barrier();                  // every wave is done with the strip's Q
            if (unit + 1 < last) split_q();
            workgroup_barrier();
        } else {
            if (OWN_RAW && unit + 1 < last) request_q(unit + 1);
            fold_begin(-0x1.fffffep127f, kNegBig);
            int young = 0;
            static_for<NT>([&](auto tc) __attribute__((always_inline)) {
                constexpr int T = decltype(tc)::value;
                const int j = opaque(T);
                if (j >= nb) return;
                const int key0 = key_of(j);
                if (pending) put(kept[T], fast_exp2(e_kept[T] - e_row) * inv_row);
                kept[T] = scores(young);
                young = pending ? flush(P_before, q0_before, key0) : 0;
                fold(kept[T], c_parts, key0, IC<1>{});
                e_kept[T] = e_run;
            });
            for (int j = NT; j < nb; ++j) {       // blocks whose exponentials do not stay
                const int key0 = key_of(j);
                f32x16 s = scores(0);
                fold(s, c_parts, key0, IC<1>{});
            }
            merge_halves();
            if (half == 0) {
                stat_lds[wave * 64 + l32] = e_run;
                stat_lds[wave * 64 + 32 + l32] = l_run;
            }
            workgroup_barrier();
            e_row = stat_lds[l32];
#pragma unroll
            for (int w = 1; w < NW; ++w) e_row = fmaxf(e_row, stat_lds[w * 64 + l32]);
            float l_row = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) l_row += stat_lds[w * 64 + 32 + l32] * fast_exp2(stat_lds[w * 64 + l32] - e_row);
            inv_row = 1.0f / l_row;
            // (the same in every wave: all see the same statistics)
            const bool exact = __builtin_amdgcn_ballot_w64(!(l_row > 0.0f && l_row < __builtin_inff())) == 0;
            if (!exact) {
                bad_first = min(bad_first, unit);
                bad_last = unit + 1;
            }
            pending = true;
            P_before = Ph;
            q0_before = q0;
            for (int j = nb; j < seq; ++j) {      // the second time
                const int key0 = key_of(j);
                f32x16 s = scores(0);
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = fast_exp2(__builtin_fmaf(s[r], c_parts, -e_row));
                put(s, inv_row);
                flush(Ph, q0, key0);
            }
            if (all_blocks > NT * NW) workgroup_barrier();      // every wave is done with the strip's Q
            if (unit + 1 < last) {
                if (!OWN_RAW) {
                    wait_lds();
                    request_q(unit + 1);
                }
                // (requested at the start of the strip: the transfers of the first NSLOT panels after it are younger)
                if (OWN_RAW && seq * np >= NSLOT) wait_transfers<NSLOT * UNIT_OPS>();
                else wait_transfers<0>();
                split_q();
            }
            workgroup_barrier();
        }
    }
    wait_transfers<0>();                          // (no transfer may be under way when the LDS of the workgroup is given back)
    if constexpr (!SCORES) {
        static_for<NT>([&](auto tc) __attribute__((always_inline)) {
            constexpr int T = decltype(tc)::value;
            const int j = opaque(T);
            if (j >= nb) return;
            put(kept[T], fast_exp2(e_kept[T] - e_row) * inv_row);
            flush(P_before, q0_before, key_of(j));
        });
        if (bad_first < bad_last) wait_transfers<0>();
        // Strips with infinities, NaN or overflows (and what lies between them) again on the fp32 instruction: rare.
        for (uint32_t unit = bad_first; unit < bad_last; ++unit) {
            const uint32_t bh = unit / strips;
            const int q0 = (int)(unit - bh * strips) * 32;
            const float* const Qh = Q + (int64_t)bh * N * d;
            const float* const Kh = K + (int64_t)bh * N * d;
            float* const Ph = P + (int64_t)bh * N * N;
            fold_begin(kNegBig, kNegBig * c);
            for (int key0 = 0; key0 < N; key0 += 32) {
                f32x16 s = scores_f32(Qh, Kh, q0, key0);
                fold(s, c, key0, IC<0>{});
            }
            merge_halves();
            const float inv = 1.0f / l_run;
            for (int j = 0; j < nb; ++j) {
                const int key0 = key_of(j);
                const f32x16 s = scores_f32(Qh, Kh, q0, key0);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = key0 + 4 * half + 8 * (r / 4) + (r % 4);
                    if (q0 + l32 < N && key < N) Ph[(int64_t)(q0 + l32) * N + key] = fast_exp2(__builtin_fmaf(s[r], c, -e_run)) * inv;
                }
            }
        }
    }
}

template <int NT, int NP, bool SCORES>
hipError_t launch_strip_t(const void* Q, const void* K, void* P, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((N + 31) / 32);
    const uint32_t total = (uint32_t)BH * strips;
    const uint32_t workers = total < (uint32_t)compute_units() ? total : (uint32_t)compute_units();
    hipLaunchKernelGGL((qk_f32_strip_kernel<NT, NP, SCORES>), dim3((workers + 7) / 8 * 8), dim3(512), 0, stream, static_cast<const float*>(Q),
                       static_cast<const float*>(K), static_cast<float*>(P), N, d, SCORES ? scale : fabsf(scale) * kLog2e,
                       !SCORES && scale < 0.0f ? -1.0f : 1.0f, strips, total, workers);
    return hipGetLastError();
}

template <int NP>
hipError_t launch_strip_p(bool scores_only, const void* Q, const void* K, void* P, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    if (scores_only) return launch_strip_t<1, NP, true>(Q, K, P, BH, N, d, scale, stream);
    if (N <= 256) return launch_strip_t<1, NP, false>(Q, K, P, BH, N, d, scale, stream);
    if (N <= 512) return launch_strip_t<2, NP, false>(Q, K, P, BH, N, d, scale, stream);
    if (N <= 1024) return launch_strip_t<4, NP, false>(Q, K, P, BH, N, d, scale, stream);
    return launch_strip_t<8, NP, false>(Q, K, P, BH, N, d, scale, stream);
}

}  // namespace

hipError_t launch_qk_f32_strip(bool scores_only, const void* Q, const void* K, void* P, int64_t BH, int64_t N, int64_t d, float scale,
                               hipStream_t stream)
{
    if (d <= 64) return launch_strip_p<2>(scores_only, Q, K, P, BH, (int)N, (int)d, scale, stream);
    return d <= 128 ? launch_strip_p<4>(scores_only, Q, K, P, BH, (int)N, (int)d, scale, stream)
                    : launch_strip_p<8>(scores_only, Q, K, P, BH, (int)N, (int)d, scale, stream);
}

}  // namespace attnw
