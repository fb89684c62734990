// Attention output  O = softmax(scale * Q K^T) V  in bf16 for d = 176 to 256: the sweep of attention_wide.hip with the two waves of a SIMD
// taking turns at the matrix unit.
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; Softmax section, Eq. 1, applied
// incrementally.)
//
// A wave (32 queries) owns up to 128 accumulators and 64 registers of Q: no room for the scores of two tiles, which attention_pipe.hip interleaves.
// Here a tile (32 keys) is two phases of a wave with a barrier after each: the output of the tile before and the scores of this one (matrix
// unit, 64 instructions of 16 cycles at d = 256), then its softmax (vector unit).  Waves 4 to 7, the other wave of each SIMD, are one phase behind
// waves 0 to 3, so that one multiplies while the other makes its weights.  In step (both in the same phase) the same code takes 221 us where it takes
// 207.5 (16 heads of N = 4096, d = 256); without the matrix phase's priority 212.
//
// What bounds it: the matrix phase under the board's power cap (matrix unit busy 68 % of SIMD cycles, both units 23 %, waves waiting 19 %; attention_wide.hip
// 59, 8 and 52 %).  Its fragments come from LDS four instruction pairs ahead (six ahead: 2 % slower at d = 176, spilled at 256).  mma16 for less power per
// product, as in attention_pipe.hip.  Below d = 176 a vector phase is longer than a matrix phase (a wave alone issues a vector instruction every 7.6
// cycles) and attention_pipe.hip is the faster one (d = 128 116.6 / 122.7 us, 160 146.9 / 147.9).
// 16 heads of N = 4096, attention_wide.hip / here: d = 176 172 / 153 us, 192 179 / 161, 240 225 / 197, 256 232 / 204 (1.35 PFLOP/s).
#include "launchers.h"
#include "attention_common.h"

namespace attnw {
namespace {

// DVB: 32-column blocks of a row, ceil(d / 32).  HALF: d is an odd multiple of 16 -- the last 16 columns on chip are zeros in Q and K
// (written once: no transfer touches them) and left out of the second contraction.  Rows past N are read as row N - 1, weigh nothing and are not stored.
template <int DVB, bool HALF>
__global__ __launch_bounds__(512, 1)
void attention_turns_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                            uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t strips, uint32_t total)
{
    using L = RowLayout<DVB>;
    constexpr int BN = 32, WQ = 8, NW = WQ, NBUF = 4;   // rings of four tiles
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
    constexpr float kLazy = 7.0f;                 // binades the maximum may run ahead of the reference exponent

    // ---- the two halves of a tile's work ---------------------------------------------------------------------------------------
    f32x4 s[2][2];                                // scores of a tile: keys 16 k + 4 quarter .. + 3, queries 16 x + l16
    u32x4 pw[2];                                  // weights of a tile, a lane's operand of the second contraction
    constexpr int KF = 2 * G, RING = 4;           // fragments of K of a tile; fragments held at a time
    u32x4 ring[RING];
    // fragment i of tile t's matrix phase: V of tile t - 1, then K of tile t
    auto fragment = [&](int t, auto ic) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value;
        if constexpr (I < CB) return v_frag((t - 1) & 3, I);
        else return k_frag(t & 3, I - CB);
    };
    auto step = [&](int t, auto ic, auto lastc) __attribute__((always_inline)) {
        constexpr int I = decltype(ic)::value;
        const u32x4 f = ring[I % RING];
        if constexpr (I < CB) {
            mma16(oacc[I][I & 1], f, pw[I & 1]);
            mma16(oacc[I][1 - (I & 1)], f, pw[1 - (I & 1)]);
        } else {
            constexpr int F = I - CB, KB = F % 2, GR = F / 2;
            if constexpr (GR == 0) s[KB][0] = s[KB][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            mma16(s[KB][KB], f, qf[KB][GR]);
            mma16(s[KB][1 - KB], f, qf[1 - KB][GR]);
        }
        if constexpr (I + RING < decltype(lastc)::value) ring[I % RING] = fragment(t, IC<I + RING>{});
        __builtin_amdgcn_sched_barrier(0);
    };
    auto prefetch_v = [&](int t) __attribute__((always_inline)) {
        static_for<RING>([&](auto ic) __attribute__((always_inline)) { ring[decltype(ic)::value] = fragment(t, ic); });
    };
    auto matrix_phase = [&](int t) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
        static_for<CB + KF>([&](auto ic) __attribute__((always_inline)) { step(t, ic, IC<CB + KF>{}); });
        __builtin_amdgcn_s_setprio(0);
    };
    auto scores = [&]() __attribute__((always_inline)) {          // tile 0
        static_for<RING>([&](auto ic) __attribute__((always_inline)) { ring[(CB + decltype(ic)::value) % RING] = fragment(0, IC<CB + decltype(ic)::value>{}); });
        static_for<KF>([&](auto ic) __attribute__((always_inline)) { step(0, IC<CB + decltype(ic)::value>{}, IC<CB + KF>{}); });
    };
    auto output = [&](int t) __attribute__((always_inline)) {     // of tile t - 1, the last
        static_for<CB>([&](auto ic) __attribute__((always_inline)) { step(t, ic, IC<CB>{}); });
    };
    auto vector_phase = [&](int t, auto lastc) __attribute__((always_inline)) {
        float top[2], p[2][8];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            top[x] = fmaxf(max3(max3(max3(s[0][x][0], s[0][x][1], s[0][x][2]), s[0][x][3], s[1][x][0]), s[1][x][1], s[1][x][2]), s[1][x][3]);
        }
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
        if constexpr (decltype(lastc)::value) {   // keys past the end weigh nothing
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if (t * BN + 16 * (r / 4) + 4 * quarter + r % 4 >= N) p[x][r] = 0.0f;
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            float sum = p[x][0];
#pragma unroll
            for (int r = 1; r < 8; ++r) sum += p[x][r];
            l_run[x] += sum;
#pragma unroll
            for (int i = 0; i < 4; ++i) pw[x][i] = pack_bf16x2(p[x][2 * i], p[x][2 * i + 1]);
        }
    };

    // ---- phases: in 2t waves 0 .. 3 multiply for tile t while 4 .. 7 make the weights of t - 1, in 2t + 1 the other way round.  Requests belong to the
    // weights' phases, K three tiles and V two tiles ahead of phase 2t for all waves: K of t - 1 and V of t - 2, whose places they take, were
    // last read in phase 2t - 1, and what request(t) brings is read from phase 2t + 5 on (V, into the ring).  A wave's request(t - 1) has arrived when it ends
    // phase 2t + 1. -------------------------------------------------------------------------------------------------------------------
    auto request = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < XW; ++j) transfer(Kh, k_base + ((t + 3) & 3) * TILE, t + 3, j, false);
#pragma unroll
        for (int j = 0; j < XW; ++j) transfer(Vh, v_base + ((t + 2) & 3) * TILE, t + 2, j, true);
    };
    const bool fewer = XFERS % NW != 0 && wave >= XFERS % NW;
    auto wait_but = [&](auto pc) __attribute__((always_inline)) {  // all transfers but those of the last P requests
        constexpr int P = decltype(pc)::value;
        if (fewer) wait_vmem_le<P * 2 * (XW - 1)>();
        else wait_vmem_le<P * 2 * XW>();
    };
    auto turn = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (HALF) {
        for (int i = threadIdx.x; i < NBUF * TILE / 16; i += 64 * NW) *reinterpret_cast<u32x4*>(k_lds + i * 16) = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) { mb_run[x] = kNegBig; l_run[x] = 0.0f; }
#pragma unroll
    for (int j = 0; j < XW; ++j) transfer(Kh, k_base, 0, j, false);
    request(-2);
    request(-1);
    wait_but(IC<1>{});
    turn();
    const bool second = wave >= 4;
    if (q0 >= N) {
        if (second) { request(0); turn(); }
        for (int t = 0; t < n_tiles; ++t) {
            if (second) wait_but(IC<1>{});
            turn();
            request(t + second);
            if (!second) wait_but(IC<1>{});
            turn();
        }
        if (!second) turn();
        wait_vmem();
        return;
    }
    if (second) { request(0); turn(); }
    auto vector_turn = [&](int t, auto lastc) __attribute__((always_inline)) {
        if (second) wait_but(IC<1>{});
        turn();
        request(t + second);
        vector_phase(t, lastc);
        prefetch_v(t + 1);
        if (!second) wait_but(IC<1>{});
        turn();
    };
    scores();
    for (int t = 0; t + 1 < n_tiles; ++t) {
        vector_turn(t, IC<0>{});
        matrix_phase(t + 1);
    }
    vector_turn(n_tiles - 1, IC<1>{});
    output(n_tiles);
    if (!second) turn();
    wait_vmem();

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

template <int DVB, bool HALF>
hipError_t launch_turns_t(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, int q_end, hipStream_t stream)
{
    const uint32_t strips = (uint32_t)((q_end + 255) / 256);
    return launch_by_heads(BH, strips, 512, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * (DVB * 32 - (HALF ? 16 : 0));
        const uint32_t total = (uint32_t)heads * strips, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_turns_kernel<DVB, HALF>), dim3(grid), dim3(512), 0, stream, static_cast<const uint16_t*>(Q) + at,
                           static_cast<const uint16_t*>(K) + at, static_cast<const uint16_t*>(V) + at, static_cast<uint16_t*>(O) + at, N,
                           fabsf(scale) * kLog2e, scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u, strips, total);
        return hipGetLastError();
    });
}

}  // namespace

// Whether the waves take turns for this shape.  A round of 256-query strips here against one of the workgroups of four waves in attention_wide.hip, two of which share
// a compute unit and whose rounds end in smaller steps; a last round of theirs with one to a compute unit takes 0.7 of a full one.  What a round takes here (theirs is 1):
// rows alike 0.85 (d of 240 and 256) to 0.94, of 512 tokens and fewer 0.01 to 0.05 more (the first and the last of twelve to sixteen tiles count), rows of every
// sharpness 0.02 to 0.07 more (exponents move in more of the tiles, and the wave whose turn at the matrix unit comes after waits), d = 192 0.02 more than its neighbours
// (measured, the reason is not known).  The lines leave what is then the slower one for rows of both kinds together: of 2100 random shapes of 385 to 3500 tokens those
// taken are rows alike 0.91 (d of 240 and 256) to 0.94 of the time, 1.012 at most, of every sharpness 0.94 to 0.99, 30 of 445 above 1.04 (to 1.09).
bool prefers_attention_turns(int64_t BH, int64_t N, int64_t d)
{
    if (d < 176 || d > 256 || d % 16 != 0 || N <= 384) return false;
    const int64_t cus = compute_units(), fours = BH * ((N + 127) / 128), eights = BH * ((N + 255) / 256);
    const int64_t last = (fours + 2 * cus - 1) % (2 * cus) + 1;
    const double round = d >= 240 ? (N > 512 ? 0.85 : 0.88) : d == 192 ? 0.94 + 48.0 / (double)N : 0.917 + 38.0 / (double)N;
    return round * (double)((eights + cus - 1) / cus) <= (double)((fours - last) / (2 * cus)) + (last <= cus ? 0.71 : 1.0);
}

hipError_t launch_attention_turns(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d, float scale,
                                  int q_end, hipStream_t stream)
{
    switch ((int)(d / 16)) {
    case 11: return launch_turns_t<6, true>(Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 12: return launch_turns_t<6, false>(Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 13: return launch_turns_t<7, true>(Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 14: return launch_turns_t<7, false>(Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 15: return launch_turns_t<8, true>(Q, K, V, O, BH, (int)N, scale, q_end, stream);
    case 16: return launch_turns_t<8, false>(Q, K, V, O, BH, (int)N, scale, q_end, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
