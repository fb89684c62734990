// Fused attention weights  P = softmax(scale * Q K^T)  and scaled scores, bf16, more than 512 keys of any number: persistent workgroups of
// one per compute unit, a strip of 32 queries at a time, its keys shared between the waves.
//
// (Paper: the fused kernel of the section "Fused Matrix Multiply + Scaling + Softmax": the scores stay where the matrix multiply left
// them, the cores of a row exchange local maxima and sums, only then are the weights formed and written.)
//
// A step is a window of 32 keys per wave.  Nothing of K is used by two waves, so each brings its own blocks to LDS by direct transfers, a
// stream that runs on from strip to strip.  Windows whose exponentials find room in registers (d > 64; above that many, and everywhere at
// d <= 64, where 16 waves hide more than the room of eight would save) are contracted once, the others for the statistics and again for
// the weights.  Vector work goes between the matrix instructions of the next block: while a held window of the next strip is contracted, that
// of the last strip leaves its registers.  The statistics (Softmax section, Eq. 1) are taken per lane against a reference exponent that
// moves only when a block's weights sum to more than 2^16, so that no maximum stands between a contraction and its exponentials.  The 32
// rows of a window are staged [query][key] and stored a step later; rows off the 16-byte boundaries are shifted on the way from LDS into
// aligned chunks, the elements of the chunks at a window's ends following one by one.  One barrier per step.
//
// Measured, us, kernel before -> this one: 8 heads of N = 1659, d = 128 76 -> 37, 6 of 1833, d = 64 61 -> 30, 2 of 7066, d = 32 220 -> 76, one of 8078,
// d = 128 112 -> 70, of 7381, d = 208 317 -> 122, 24 of 1312, d = 256 90 -> 62; over 3190 random shapes of 513 to 30000 tokens that come here 0.58 of the time
// (1950 of scores 0.53).  What bounds it: waits, 38 to 46 % of a wave's life, of the 2 or 4 waves per SIMD that a step's barrier keeps together, and the
// vector ALU, 53 % busy at d = 32, 28 to 47 % at d of 64 to 256 (2 heads of 7072, d = 32: 149 issue slots per block of 32 x 32, of which 128 are Eq. 1
// and its second pass); at d = 128 also K, which every strip reads again (a quarter of the time goes with its transfers left out).
#include "launchers.h"
#include "attention_common.h"

namespace attnw {
namespace {

// G: 16-element steps of the contraction (d = 16 G)
template <int G> struct StreamCfg {
    // Waves: 16 where that leaves a wave enough registers for the contraction (2 heads of N = 7066, d = 32 76 against 91 us, d = 96 159 against 149).
    static constexpr int NW = G <= 4 ? 16 : 8;
    static constexpr int WINDOW = 32 * NW;                      // keys of a window: a block of 32 per wave
    static constexpr int PITCH = WINDOW * 2 + 16, STAGED = 32 * PITCH;   // bytes of a staged row, of a staged window
    static constexpr int NP = NW == 16 ? (G + 1) / 2 : (G + 3) / 4;   // a block of 32 keys travels in NP pieces of ..
    static constexpr int PW = (G + NP - 1) / NP;                // .. PW contraction steps (the last one overlaps its neighbour)
    static constexpr int NS = NW == 16 ? 2 : NP == 3 || NP == 1 ? 3 : 2;                  // pieces that a wave holds in LDS
    static constexpr int SLOT = PW * 1024;
    static constexpr int RING = NS * SLOT;
    // windows whose exponentials stay in registers (one more spills; some 60 scalars spill with any)
    static constexpr int held(bool whole) { return NW == 16 ? 0 : (G <= 6 ? 7 : G <= 10 ? 6 : G <= 14 ? 5 : 4) - (whole ? 0 : 1); }
    static constexpr int QBUF = NW * RING, STAGE = QBUF + NP * SLOT, STAT = STAGE + 2 * STAGED, LDS = STAT + NW * 32 * 8;
    static_assert(LDS <= 160 * 1024 && STAGE <= kDirectLds, "LDS of a workgroup, reach of direct transfers");
    static constexpr int piece_col(int p) { return p * PW < G - PW ? p * PW : G - PW; }
};

__device__ __forceinline__ void lds_barrier()     // (transfers and stores under way stay so)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}
// The number, where the compiler does not know it: what is computed from it stays where it stands (hoisted out of the strip loop, the
// windows' places spilled several hundred scalars)
__device__ __forceinline__ int opaque(int x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(x));
#endif
    return x;
}

// WHOLE: N a multiple of 8, every row of P on a 16-byte boundary.  SCORES: write scale * Q K^T instead of the weights; c is the scale.
template <int G, bool WHOLE, bool SCORES>
__global__ __launch_bounds__(64 * StreamCfg<G>::NW, StreamCfg<G>::NW / 4)
void qk_stream_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, uint16_t* __restrict__ out, int N, float c,
                      uint32_t sign_flip, uint32_t strips_per_head, uint32_t per_worker, uint32_t extra)
{
    using C = StreamCfg<G>;
    constexpr int RB = 32 * G, NP = C::NP, PW = C::PW, NS = C::NS, SLOT = C::SLOT, T = SCORES ? 0 : C::held(WHOLE);
    constexpr int kWaves = C::NW, kWindow = C::WINDOW, kPitch = C::PITCH, kStage = C::STAGED;
    constexpr int ROWB = 32 * PW, CPR = 2 * PW;
    // chunk XOR row / RPL stays inside the row and puts the 16 rows that a fragment read serves at a time on different banks
    constexpr int P2 = PW == 4 ? 8 : PW == 2 ? 4 : 2, RPL = 16 / P2;
    constexpr int FLUSH = 4;                      // the item before which the window staged a step ago is stored
    // shares of a step's vector work: one per matrix instruction, PRE while a piece's fragments arrive
    constexpr int PRE = 2, CHUNKS = (NP - 1) * (PW + PRE) + PRE + G - (NP - 1) * PW;
    extern __shared__ __align__(4096) char lds[];
    f32x2* const stat = reinterpret_cast<f32x2*>(lds + C::STAT);

    const uint32_t id = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    const uint32_t s_begin = id * per_worker + (id < extra ? id : extra);
    const uint32_t s_end = s_begin + per_worker + (id < extra ? 1u : 0u);
    if (s_begin == s_end) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;

    const int n_win = (N + kWindow - 1) / kWindow;
    const int held = n_win < T ? n_win : T;       // windows in registers; the others are computed twice
    const int twice = n_win - held;
    const int rot = (int)(id * 5u % (uint32_t)n_win);   // every workgroup starts its sweeps elsewhere
    auto window = [&](int t) __attribute__((always_inline)) { const int w = t + rot; return w >= n_win ? w - n_win : w; };
    auto next_window = [&](int w) __attribute__((always_inline)) { return w + 1 == n_win ? 0 : w + 1; };

    // ---- the stream of K blocks: per strip the windows computed twice, those held, the former again ----
    // places of a wave-wide transfer's chunks in 32 rows of K from row `first` on, rows past `last` being row `last` again
    auto place = [&](int j, int first, int last) __attribute__((always_inline)) {
        const int s = j * 64 + lane, row = s / CPR;
        return (uint32_t)(min(first + row, last) * RB + (((s % CPR) ^ ((row / RPL) & (P2 - 1))) * 16) - j * 1024);
    };
    // the PW transfers of a piece: transfer j's place is 1 KiB further on in LDS, hence in memory too (- j * 1024 above; never negative:
    // 1 KiB in front of transfer j are rows of their own, or chunks of a row, at 32 bytes a row and more)
    auto transfer = [&](const char* base, const uint32_t (&at)[PW], uint32_t dst) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (PW == 4)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5\n\tglobal_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                         "global_load_lds_dwordx4 %3, %5 offset:2048\n\tglobal_load_lds_dwordx4 %4, %5 offset:3072"
                         ::"s"(dst), "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "s"(base) : "memory", "m0");
        else if constexpr (PW == 3)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\tglobal_load_lds_dwordx4 %2, %4 offset:1024\n\t"
                         "global_load_lds_dwordx4 %3, %4 offset:2048"
                         ::"s"(dst), "v"(at[0]), "v"(at[1]), "v"(at[2]), "s"(base) : "memory", "m0");
        else if constexpr (PW == 2)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024"
                         ::"s"(dst), "v"(at[0]), "v"(at[1]), "s"(base) : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"::"s"(dst), "v"(at[0]), "s"(base) : "memory", "m0");
#endif
    };
    const uint32_t lds0 = lds_offset_of(lds), ring = lds0 + (uint32_t)(wave * C::RING);
    const int steps = SCORES ? n_win : n_win + twice;
    uint32_t at_strip = s_begin, at_in_head = s_begin % strips_per_head;
    const char* at_head = reinterpret_cast<const char*>(K) + (int64_t)(s_begin / strips_per_head) * N * RB;
    int at_step = 0, at_window = window(twice > 0 ? held : 0);
    const char* at_base = nullptr;                // rows of the block
    uint32_t off[PW];
    bool at_end = true;                           // off[] belongs to a block that ends past N
    auto locate = [&]() __attribute__((always_inline)) {
        const int first = (at_window * kWaves + wave) * 32;
        const bool end = first + 32 > N;
        at_base = at_head + (end ? 0 : (int64_t)first * RB);
        if (end || at_end) {
#pragma unroll
            for (int j = 0; j < PW; ++j) off[j] = end ? place(j, first, N - 1) : place(j, 0, 31);
            at_end = end;
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
        at_window = next_window(at_window);
        if (++at_step == steps) {
            at_step = 0;
            at_window = window(twice > 0 ? held : 0);
            if (at_strip + 1 < s_end) {           // (after the last strip its blocks again, so that the counts of the waits hold)
                ++at_strip;
                if (++at_in_head == strips_per_head) {
                    at_in_head = 0;
                    at_head += (int64_t)N * RB;
                }
            }
        }
        locate();
    };
    locate();
    static_for<NS>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i > 0 && i % NP == 0) advance();
        transfer(at_base + C::piece_col(i % NP) * 32, off, ring + i * SLOT);
    });

    // ---- fragments: lanes 0..31 carry the even 16-byte chunk of each 32-byte group, lanes 32..63 the odd one ----
    int frag_off[PW];
#pragma unroll
    for (int g = 0; g < PW; ++g) frag_off[g] = l32 * ROWB + (((2 * g + half) ^ ((l32 / RPL) & (P2 - 1))) * 16);
    u32x4 qf[G];
    {
        const uint32_t h = s_begin / strips_per_head;
        const int q0 = (int)at_in_head * 32;
        const char* const p = reinterpret_cast<const char*>(Q) + ((int64_t)h * N + min(q0 + l32, N - 1)) * RB + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(p + g * 32) ^ sign_flip;
    }
    // Q of a later strip: to LDS by all waves, from there some steps later
    auto bring_q = [&](uint32_t strip) __attribute__((always_inline)) {
        const uint32_t h = strip / strips_per_head;
        const int q0 = (int)(strip - h * strips_per_head) * 32;
        const char* const head = reinterpret_cast<const char*>(Q) + (int64_t)h * N * RB;
        for (int p = wave; p < NP; p += kWaves) {
            uint32_t at[PW];
#pragma unroll
            for (int j = 0; j < PW; ++j) at[j] = place(j, q0, N - 1);
            transfer(head + (p * PW < G - PW ? p * PW : G - PW) * 32, at, __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(C::QBUF + p * SLOT)));
        }
    };
    auto take_q = [&]() __attribute__((always_inline)) {
        static_for<G>([&](auto gc) __attribute__((always_inline)) {
            constexpr int g = decltype(gc)::value, p = g / PW;
            qf[g] = *reinterpret_cast<const u32x4*>(lds + C::QBUF + p * SLOT + frag_off[g - C::piece_col(p)]) ^ sign_flip;
        });
    };

    // Scores of the next block of the stream: acc[r] = q . k for key 8 (r / 4) + 4 half + r % 4 of the block and query l32; work(chunk)
    // is the vector work beside the waits and the matrix instructions.
    f32x16 acc;
    int at_slot = 0;                              // the slot of the next piece
    auto contract = [&](auto&& work) __attribute__((always_inline)) {
        static_for<NP>([&](auto pc) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value, first = C::piece_col(p);
            constexpr int count = (p + 1) * PW < G ? PW : G - p * PW;
            constexpr int q = (p + NS) % NP;
            wait_vmem_le<(NS - 1) * PW>();        // (stores among the younger operations make it wait for more)
            asm volatile("" ::: "memory");
            const int slot = NP % NS != 0 ? at_slot : (p % NS) * SLOT;
            const char* const blk = lds + wave * C::RING + slot;
            u32x4 kf[count];
#pragma unroll
            for (int g = 0; g < count; ++g) kf[g] = *reinterpret_cast<const u32x4*>(blk + frag_off[p * PW + g - first]);
            __builtin_amdgcn_sched_barrier(0);
            work(IC<p * (PW + PRE)>{}, IC<p * (PW + PRE) + PRE>{});
            wait_lds();                           // the fragments have left the slot
            asm volatile("" ::: "memory");
            if constexpr (q == 0) advance();
            transfer(at_base + C::piece_col(q) * 32, off, __builtin_amdgcn_readfirstlane(ring + (uint32_t)slot));
            if constexpr (p == 0) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
            }
            if constexpr (NP % NS != 0) at_slot = at_slot + SLOT == C::RING ? 0 : at_slot + SLOT;
            static_for<count>([&](auto gc) __attribute__((always_inline)) {
                constexpr int g = decltype(gc)::value, at = p * (PW + PRE) + PRE + g;
                __builtin_amdgcn_sched_barrier(0);
                Mma<uint16_t>::run(acc, kf[g], qf[p * PW + g]);
                work(IC<at>{}, IC<at + 1>{});
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto nothing = [](auto, auto) __attribute__((always_inline)) {};
    // items [0, M) of vector work spread over the shares of a step
    auto spread = [&](auto mc, auto&& item) __attribute__((always_inline)) {
        return [&](auto c0, auto c1) __attribute__((always_inline)) {
            constexpr int M = decltype(mc)::value, i0 = decltype(c0)::value * M / CHUNKS;
            constexpr int i1 = decltype(c1)::value >= CHUNKS ? M : decltype(c1)::value * M / CHUNKS;
            static_for<i1 - i0>([&](auto ic) __attribute__((always_inline)) { item(IC<i0 + decltype(ic)::value>{}); });
        };
    };

    // ---- the way out: a window of 32 rows staged [query][key], stored a step later as aligned 16-byte chunks ----
    int buf = 0;
    char* const stage_at = lds + C::STAGE + l32 * kPitch + (wave * 32 + 4 * half) * 2;
    auto stage_run = [&](int r4, uint32_t w01, uint32_t w23) __attribute__((always_inline)) {
        *reinterpret_cast<u32x2*>(stage_at + buf + r4 * 16) = u32x2{w01, w23};
    };
    char* strip_out = nullptr;                    // the strip in P, its rows, its first element mod 8
    int rows = 0, strip_o = 0;
    char* pend_dst = nullptr;                     // the staged window: its place in P ..
    int pend = 0, pend_rows = 0, pend_len = 0, pend_o = 0;   // .. (pend: 0 none, 1 cut off at the end of rows or columns, 2 whole)
    auto staged = [&](int wi) __attribute__((always_inline)) {
        pend_dst = strip_out + (int64_t)wi * (kWindow * 2);
        pend_len = N - wi * kWindow;
        pend = rows == 32 && pend_len >= kWindow ? 2 : 1;
        pend_rows = rows;
        pend_o = strip_o;
        buf ^= kStage;
    };
    // two rows of a window per store with eight waves, one with 16
    const int chunk = kWaves == 8 ? l32 : lane;
    auto store_row = [&](int i) __attribute__((always_inline)) { return kWaves == 8 ? 4 * wave + 2 * i + half : 2 * wave + i; };
    u32x4 fl[2];
    uint32_t fl4[2];
    uint16_t edge = 0;
    // (unaligned rows) the chunks of a row start o elements in front of the window; those wholly inside it are put together from the
    // staged words, the elements of the others follow one by one
    auto chunk_key = [&](int i) __attribute__((always_inline)) { return chunk * 8 - ((pend_o + store_row(i) * N) & 7); };
    const int edge_row = kWaves == 8 ? 4 * wave + (lane >> 4) : lane < 32 ? 2 * wave + (lane >> 4) : 32;
    auto edge_key = [&](int row) __attribute__((always_inline)) {
        const int o = (pend_o + row * N) & 7, i = lane & 15;
        const int len = min(pend_len, kWindow);
        const int k = i < 8 ? (o != 0 ? i - o : -1) : ((o + len) & ~7) - o + i - 8;
        return row < pend_rows && k < len ? k : -1;
    };
    auto flush_read = [&](bool settle = false) __attribute__((always_inline)) {
        if (settle) wait_vmem();
        lds_barrier();
        const char* const src = lds + C::STAGE + (buf ^ kStage);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const char* const row = src + store_row(i) * kPitch;
            if constexpr (WHOLE) {
                fl[i] = *reinterpret_cast<const u32x4*>(row + chunk * 16);
            } else {
                const uint32_t* const w = reinterpret_cast<const uint32_t*>(row + ((max(chunk_key(i), 0) * 2) & ~3));
#pragma unroll
                for (int e = 0; e < 4; ++e) fl[i][e] = w[e];
                fl4[i] = w[4];
            }
        }
        if constexpr (!WHOLE) {
            const int row = edge_row;
            edge = *reinterpret_cast<const uint16_t*>(src + min(row, 31) * kPitch + max(edge_key(row), 0) * 2);
        }
    };
    auto flush_store = [&]() __attribute__((always_inline)) {
        if (pend == 0) return;
        if (WHOLE && pend == 2) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                __builtin_nontemporal_store(fl[i], reinterpret_cast<u32x4*>(pend_dst + (uint32_t)(store_row(i) * N * 2 + chunk * 16)));
        } else if (WHOLE) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = store_row(i);
                if (row < pend_rows && chunk * 8 < pend_len)
                    __builtin_nontemporal_store(fl[i], reinterpret_cast<u32x4*>(pend_dst + (uint32_t)(row * N * 2 + chunk * 16)));
            }
        } else {
            const int len = min(pend_len, kWindow);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = store_row(i), k = chunk_key(i);
                if (row < pend_rows && k >= 0 && k + 8 <= len) {
                    const uint32_t sh = (uint32_t)(k & 1) * 16u;
                    u32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_alignbit(e < 3 ? fl[i][e + 1] : fl4[i], fl[i][e], sh);
                    *reinterpret_cast<u32x4*>(pend_dst + (uint32_t)(row * N + k) * 2u) = v;
                }
            }
            const int row = edge_row, k = edge_key(row);
            if (k >= 0) *reinterpret_cast<uint16_t*>(pend_dst + (uint32_t)(row * N + k) * 2u) = edge;
        }
        pend = 0;
    };

    // ---- statistics of the strip (Eq. 1), per lane against a reference exponent that follows the maximum from afar ----
    constexpr float kFar = 65536.0f;              // a block whose weights sum to more moves the reference
    float ref = kNegBig, l = 0.0f, f = 0.0f, bias = 0.0f;
    float arg[16], s4[4];
    auto acc_max = [&]() __attribute__((always_inline)) {
        float m = max3(acc[0], acc[1], acc[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) m = max3(m, acc[r], acc[r + 1]);
        return fmaxf(reference_exponent(fmaxf(m, acc[15]), c), kNegBig);
    };
    // the reference moves by m; rescale(a): the strip's exponentials so far take the factor a
    // (in two factors: v_exp_f32 gives 0 below 2^-126, and these may be as large as 2^16)
    auto lower = [&](float m, auto&& rescale) __attribute__((always_inline)) {
        const float m1 = fminf(m, 64.0f);
#pragma unroll 1
        for (int i = 0; i < 2; ++i) {
            const float a = fast_exp2(i == 0 ? -m1 : m1 - m);
            l *= a;
            rescale(a);
        }
    };
    // Exponents of the block's weights against the reference; the first block sets it.  While it lies far below 0 it follows the maximum itself: exponents against
    // that of masked keys (-1e9 through a column of K) keep too few bits to move it by them.
    constexpr float kLow = -1024.0f;
    auto arguments = [&](int key0, auto&& rescale) __attribute__((always_inline)) {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(ref < kLow) != 0, 0)) {
            const float to = ref < kLow ? fmaxf(ref, acc_max()) : ref;
            if (__builtin_amdgcn_ballot_w64(to > ref) != 0) lower(to - ref, rescale);
            ref = to;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) arg[r] = __builtin_fmaf(acc[r], c, -ref);
        if (key0 + 32 > N) {                      // keys past N do not count
#pragma unroll
            for (int r = 0; r < 16; ++r) arg[r] = key0 + 8 * (r / 4) + 4 * half + (r % 4) < N ? arg[r] : -__builtin_inff();
        }
    };
    auto weigh = [&](float (&e)[16], auto rc) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        e[r] = fast_exp2(arg[r]);
        if constexpr (r < 4) s4[r] = e[r];
        else s4[r & 3] += e[r];
    };
    // after all 16: into the sum; rescale(a): the strip's exponentials before these take the factor a
    auto count = [&](float (&e)[16], auto&& rescale) __attribute__((always_inline)) {
        float s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(s > kFar) != 0, 0)) {
            float m = arg[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) m = fmaxf(m, arg[r]);
            // by so much the reference moves, as rounded: blocks after this one are taken against ref itself
            const float to = ref + fmaxf(m, 0.0f);
            m = to - ref;
            ref = to;
            lower(m, rescale);
#pragma unroll
            for (int r = 0; r < 16; ++r) arg[r] -= m;
            static_for<16>([&](auto rc) __attribute__((always_inline)) { weigh(e, rc); });
            s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        }
        l += s;
    };
    // the two halves of a query's keys, then the waves: the paper's local-then-global reduction across a row of cores
    auto publish = [&]() __attribute__((always_inline)) {
        const float ro = __shfl_xor(ref, 32, 64), lo = __shfl_xor(l, 32, 64);
        const float mw = fmaxf(ref, ro);
        if (half == 0) stat[wave * 32 + l32] = f32x2{mw, l * fast_exp2(ref - mw) + lo * fast_exp2(ro - mw)};
    };
    float X[T > 0 ? T : 1][16];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) X[t][r] = 0.0f;
    auto fold = [&]() __attribute__((always_inline)) {
        float m = kNegBig, sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) m = fmaxf(m, stat[w * 32 + l32][0]);
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const f32x2 s = stat[w * 32 + l32];
            sum += s[1] * fast_exp2(s[0] - m);
        }
        bias = m + fast_log2(sum);
        float d = ref - m;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(d < -100.0f) != 0, 0)) {   // a factor near the smallest number: in two steps
            const float d1 = fmaxf(d, -60.0f), a = fast_exp2(d1);
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) X[t][r] *= a;
            d -= d1;
        }
        f = fast_exp2(d) * __builtin_amdgcn_rcpf(sum);
        ref = kNegBig;
        l = 0.0f;
    };

    contract(nothing);                            // the first block
    for (uint32_t strip = s_begin;; ++strip) {
        const bool cur = strip < s_end;
        if (strip > s_begin) {
            const uint32_t h = (strip - 1) / strips_per_head;
            const int q0 = (int)(strip - 1 - h * strips_per_head) * 32;
            // (a window of the strip before may still be staged: it keeps its own place)
            const int64_t e0 = ((int64_t)h * N + q0) * N;
            strip_out = reinterpret_cast<char*>(out) + e0 * 2;
            strip_o = (int)(e0 & 7);
            rows = min(32, N - q0);
            int wi = window(held);
            for (int j = 0; j < twice; ++j, wi = next_window(wi)) {
                // (scores of two windows: Q of the next strip is under way since the step before; else the waits for K cover it)
                flush_read(SCORES && j == 1 && n_win == 2);
                if (!SCORES && j == 0) fold();
                if (SCORES && j == 0 && cur) bring_q(strip);
                if (j + 1 == twice && cur) take_q();
                float p[16];
                uint32_t pk[8];
#pragma unroll
                for (int r = 0; r < 16; ++r) arg[r] = SCORES ? acc[r] * c : __builtin_fmaf(acc[r], c, -bias);
                contract(spread(IC<16>{}, [&](auto ic) __attribute__((always_inline)) {
                    constexpr int r = decltype(ic)::value;
                    if constexpr (r == FLUSH) flush_store();
                    p[r] = SCORES ? arg[r] : fast_exp2(arg[r]);
                    if constexpr (r % 2 == 1) pk[r / 2] = pack_bf16x2(p[r - 1], p[r]);
                    if constexpr (r % 4 == 3) stage_run(r / 4, pk[r / 2 - 1], pk[r / 2]);
                }));
                staged(wi);
            }
        }
        if constexpr (SCORES) {
            if (!cur) break;
            continue;
        }
        if (cur && twice > 0) {
            if (pend != 0) {
                flush_read();
                flush_store();
            }
            if (strip + 1 < s_end) bring_q(strip + 1);   // (behind a barrier that every wave reached after it took the last one)
            int wi = window(opaque(held));
            for (int j = 0; j < twice; ++j, wi = next_window(wi)) {
                arguments((wi * kWaves + wave) * 32, [](float) __attribute__((always_inline)) {});
                float e[16];
                contract(spread(IC<16>{}, [&](auto ic) __attribute__((always_inline)) { weigh(e, ic); }));
                count(e, [](float) __attribute__((always_inline)) {});
            }
        }
        int wi = rot;
        static_for<T>([&](auto tc) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value;
            if (t < held) {
                flush_read();
                if (t == 0 && twice == 0) {
                    if (strip > s_begin) fold();
                    if (strip + 1 < s_end) bring_q(strip + 1);
                }
                if (cur) {
                    if (twice == 0 && t + 1 == held && strip + 1 < s_end) take_q();
                    const auto rescale = [&](float a) __attribute__((always_inline)) {
#pragma unroll
                        for (int u = 0; u < t; ++u)
#pragma unroll
                            for (int r = 0; r < 16; ++r) X[u][r] *= a;
                    };
                    arguments((wi * kWaves + wave) * 32, rescale);
                    uint32_t pk[8];
                    contract(spread(IC<24>{}, [&](auto ic) __attribute__((always_inline)) {
                        constexpr int i = decltype(ic)::value;
                        if constexpr (i == FLUSH) flush_store();
                        if constexpr (i < 8) {
                            pk[i] = pack_bf16x2(X[t][2 * i] * f, X[t][2 * i + 1] * f);
                            if constexpr (i % 2 == 1) stage_run(i / 2, pk[i - 1], pk[i]);
                        } else {
                            weigh(X[t], IC<i - 8>{});
                        }
                    }));
                    count(X[t], rescale);
                } else {
                    flush_store();
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        stage_run(r4, pack_bf16x2(X[t][4 * r4] * f, X[t][4 * r4 + 1] * f), pack_bf16x2(X[t][4 * r4 + 2] * f, X[t][4 * r4 + 3] * f));
                }
                if (strip > s_begin) staged(wi);
                wi = next_window(opaque(wi));
            }
        });
        if (!cur) break;
        publish();
    }
    flush_read();
    flush_store();
    wait_vmem();                                  // no transfer may be under way when the workgroup's LDS is released
}

template <int G>
hipError_t launch_stream_t(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, float scale, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((N + 31) / 32);
    const uint32_t total = (uint32_t)BH * strips, cus = (uint32_t)compute_units();
    const uint32_t grid = ((total < cus ? total : cus) + 7) / 8 * 8;
    const float c = scores_only ? scale : fabsf(scale) * kLog2e;
    const uint32_t flip = (!scores_only && scale < 0.0f) ? Mma<uint16_t>::kSignMask : 0u;
    const uint16_t* const q = static_cast<const uint16_t*>(Q);
    const uint16_t* const k = static_cast<const uint16_t*>(K);
    uint16_t* const p = static_cast<uint16_t*>(out);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * StreamCfg<G>::NW), StreamCfg<G>::LDS, stream, q, k, p, N, c, flip, strips, total / grid, total % grid);
    };
    if (scores_only) N % 8 == 0 ? go(qk_stream_kernel<G, true, true>) : go(qk_stream_kernel<G, false, true>);
    else N % 8 == 0 ? go(qk_stream_kernel<G, true, false>) : go(qk_stream_kernel<G, false, false>);
    return hipGetLastError();
}

}  // namespace

// (offsets into 32 rows of P and into a head of K are 32 bits; Q of the next strip travels over three steps)
bool qk_stream_supported(int64_t BH, int64_t N, int64_t d)
{
    return N > 512 && N <= (1 << 22) && d >= 16 && d <= 256 && d % 16 == 0 && BH * ((N + 31) / 32) <= (int64_t)0x7ffffff0;
}

hipError_t launch_qk_stream(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                            hipStream_t stream)
{
    switch ((int)(d / 16)) {
#define ATTNW_STREAM(g) case g: return launch_stream_t<g>(scores_only, Q, K, out, BH, (int)N, scale, stream);
    ATTNW_STREAM(1) ATTNW_STREAM(2) ATTNW_STREAM(3) ATTNW_STREAM(4) ATTNW_STREAM(5) ATTNW_STREAM(6) ATTNW_STREAM(7) ATTNW_STREAM(8)
    ATTNW_STREAM(9) ATTNW_STREAM(10) ATTNW_STREAM(11) ATTNW_STREAM(12) ATTNW_STREAM(13) ATTNW_STREAM(14) ATTNW_STREAM(15) ATTNW_STREAM(16)
#undef ATTNW_STREAM
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
