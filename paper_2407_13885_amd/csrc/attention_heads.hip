// Attention output  O = softmax(scale * Q K^T) V  in bf16 for sequences whose K and V fit the LDS of a compute unit (d up to 128).
//
// (Paper: Multi-Head Self-Attention section, Attention(Q, K, V) = softmax(Q K^T / sqrt(d_k)) V; the max-subtracted softmax of the
// Softmax section, Eq. 1, is applied incrementally as in attention_kernels.hip.)
//
// A workgroup brings the K and V of a head to LDS by direct transfers, as they lie in memory, and meets at one barrier; each of its waves
// then walks all keys for 32 queries of its own.  Without tiles to wait for the waves of a SIMD drift apart, and one's softmax is
// the other's matrix instructions; V is turned by the transposing LDS read.
//
// Measured, 7267 heads of N = 129, d = 64: 122 us (480 MB of Q, K, V and O, 3.9 TB/s; 255 with tiles shared by 256-query workgroups), 7324 of
// 128 105 (163 with operands gathered by every wave for itself), 1953 of 400 168 (233).  What bounds it: short of N = 128 the traffic of Q, K, V
// and O, beyond the vector ALU between the two matrix instructions of a wave (softmax of 32 x 32 scores: about 150 instructions against
// 4 + 4 of the matrix at d = 64), and the time that a workgroup alone on its compute unit waits for K and V.
#include "attention_common.h"
#include "launchers.h"

namespace attnw {
namespace {

constexpr int kAttnHeadsLds = 160 * 1024;
template <int DVB> constexpr int kAttnHeadsWaves = DVB <= 2 ? 16 : 10;   // (128 and 168 registers)

// DVB: 32-column blocks of a row, ceil(d / 32).  HALF: d is an odd multiple of 16 -- the last 16 columns on chip are copies of the
// row's first chunks, left out of the first contraction and not stored by the second.  Rows past N are read as row N - 1, weigh
// nothing and are not stored.
template <int DVB, bool HALF>
__global__ __launch_bounds__(64 * kAttnHeadsWaves<DVB>)
void attention_heads_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                            uint16_t* __restrict__ O, int N, float c, uint32_t sign_flip, uint32_t groups, uint32_t total)
{
    using L = RowLayout<DVB>;
    constexpr int DB = DVB * 64, CPR = DVB * 4;   // bytes and 16-byte chunks of a row on chip
    constexpr int rb = DB - (HALF ? 32 : 0);      // bytes of a row in memory
    constexpr int G = rb / 32;                    // 32-byte contraction groups of a row
    constexpr int TILE = 32 * DB;
    extern __shared__ __align__(1024) char lds[];

    const uint32_t id = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (id >= total) return;
    const uint32_t bh = id / groups;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int n_tiles = (N + 31) / 32;
    const int64_t at = (int64_t)bh * N * rb;
    const int q0 = ((int)(id - bh * groups) * nw + wave) * 32;

    // ---- K, then V of the head: transfer j moves chunks 64 j .. 64 j + 63 of the two together ----
    {
        const int per = n_tiles * (TILE / 1024);  // transfers of K, and of V
        for (int j = wave; j < 2 * per; j += nw) {
            const bool v = j >= per;              // (wave-uniform)
            const int s = (v ? j - per : j) * 64 + lane;
            const int key = s / CPR;
            int ch = (s - key * CPR) ^ (v ? L::v_block(key) * 4 : L::k_chunk(key));
            if (HALF && ch * 16 >= rb) ch -= rb / 16;
            const char* const src = reinterpret_cast<const char*>(v ? V : K) + at + (int64_t)min(key, N - 1) * rb + ch * 16;
            if ((j + 1) * 1024 <= kDirectLds) dma16(src, lds + j * 1024);
            else *reinterpret_cast<u32x4*>(lds + j * 1024 + lane * 16) = *reinterpret_cast<const u32x4*>(src);
        }
    }
    u32x4 qf[G];                                  // (a negative scale negates Q)
    {
        const char* const qrow = reinterpret_cast<const char*>(Q) + at + (int64_t)min(q0 + l32, N - 1) * rb + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(qrow + g * 32) ^ sign_flip;
    }
    wait_vmem();
    __syncthreads();
    if (q0 >= N) return;                          // (no barrier follows)

    // ---- per-lane places of the operand fragments ----
    constexpr int KPERIOD = L::KPERIOD, VPERIOD = L::VPERIOD;
    const char* krow = lds + l32 * DB;
    int koff[KPERIOD];
#pragma unroll
    for (int g = 0; g < KPERIOD; ++g) koff[g] = ((2 * g + half) ^ L::k_chunk(l32)) * 16;
    const int vkey = 4 * half + ((lane & 15) >> 2);            // a lane's row of the 8-key group that it reads
    const char* vrow = lds + n_tiles * TILE + vkey * DB + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    int voff[VPERIOD];
#pragma unroll
    for (int b = 0; b < VPERIOD; ++b) voff[b] = (b ^ L::v_block(vkey)) * 64;

    f32x16 oacc[DVB];
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
    float mb_run = kNegBig, l_run = 0.0f;
    constexpr float kLazy = 8.0f;                 // binades the maximum may run ahead of the reference exponent

    for (int t = 0; t < n_tiles; ++t, krow += TILE, vrow += TILE) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g)
            Mma<uint16_t>::run(s, *reinterpret_cast<const u32x4*>(krow + (g / KPERIOD) * KPERIOD * 32 + koff[g % KPERIOD]), qf[g]);
        float tm = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) tm = max3(tm, s[r], s[r + 1]);
        const float m = half_wave_max(fmaxf(tm, s[15]));   // (keys past the end are copies of key N-1: no new maximum)
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
        if (t * 32 + 32 > N) {                    // keys past the end weigh nothing
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (t * 32 + 4 * half + 8 * (r / 4) + (r % 4) >= N) p[r] = 0.0f;
        }
        float sum[2] = {p[0], p[1]};
#pragma unroll
        for (int r = 2; r < 16; ++r) sum[r & 1] += p[r];
        l_run += sum[0] + sum[1];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            u32x4 pw;
#pragma unroll
            for (int i = 0; i < 4; ++i) pw[i] = pack_bf16x2(p[8 * m + 2 * i], p[8 * m + 2 * i + 1]);
#pragma unroll
            for (int b = 0; b < DVB; ++b) {
                const char* v = vrow + 16 * m * DB + (b / VPERIOD) * VPERIOD * 64 + voff[b % VPERIOD];
                Mma<uint16_t>::run(oacc[b], u32x4_of(lds_read_tr16(v), lds_read_tr16(v + 8 * DB)), pw);
            }
        }
    }

    const float inv = 1.0f / half_wave_sum(l_run);
    if (q0 + l32 >= N) return;
    // a run is 4 consecutive output columns of the lane's query
    char* const orow = reinterpret_cast<char*>(O) + at + (int64_t)(q0 + l32) * rb + half * 8;
#pragma unroll
    for (int run = 0; run < rb / 16; ++run) {
        const f32x16& a = oacc[run / 4];
        const int r = (run % 4) * 4;
        *reinterpret_cast<u32x2*>(orow + run * 16) = u32x2{pack_bf16x2(a[r] * inv, a[r + 1] * inv), pack_bf16x2(a[r + 2] * inv, a[r + 3] * inv)};
    }
}

template <int DVB, bool HALF>
hipError_t launch_heads(const void* Q, const void* K, const void* V, void* O, int64_t BH, int N, float scale, hipStream_t stream)
{
    const int blocks = (N + 31) / 32;             // of queries, and of keys
    const uint32_t groups = (uint32_t)((blocks + kAttnHeadsWaves<DVB> - 1) / kAttnHeadsWaves<DVB>);
    const uint32_t nw = ((uint32_t)blocks + groups - 1) / groups;
    const size_t lds = (size_t)blocks * 2 * 32 * DVB * 64;
    return launch_by_heads(BH, groups, 64 * nw, [&](int64_t first, int64_t heads) {
        const int64_t at = first * N * (DVB * 32 - (HALF ? 16 : 0));
        const uint32_t total = (uint32_t)heads * groups, grid = (total + 7) / 8 * 8;
        hipLaunchKernelGGL((attention_heads_kernel<DVB, HALF>), dim3(grid), dim3(64 * nw), lds, stream,
                           static_cast<const uint16_t*>(Q) + at, static_cast<const uint16_t*>(K) + at, static_cast<const uint16_t*>(V) + at,
                           static_cast<uint16_t*>(O) + at, N, fabsf(scale) * kLog2e, scale < 0.0f ? Mma<uint16_t>::kSignMask : 0u, groups,
                           total);
        return hipGetLastError();
    });
}

}  // namespace

bool attention_heads_supported(int64_t BH, int64_t N, int64_t d)
{
    if (N < 1 || N > 2048 || d < 16 || d > 128 || d % 16 != 0 || BH > (int64_t)0x0fffffff) return false;
    return (N + 31) / 32 * 2 * 32 * ((d + 31) / 32) * 64 <= kAttnHeadsLds;
}

// Against the kernel that would take it otherwise, us: d = 64 9375 heads of N = 100 146 -> 111, 7324 of 128 163 -> 105, 7267 of 129 255 -> 122, 4758 of
// 197 188 -> 130, 4000 of 240 187 -> 138, 3662 of 256 126 -> 130, 3647 of 257 255 -> 159, 1953 of 400 227 -> 166, 1192 of 512 136 -> 137; d = 32 18750 of 100 129 -> 110,
// 9517 of 197 172 -> 138, 7295 of 257 236 -> 163, 3906 of 400 227 -> 175, 2384 of 512 141 -> 149, 1877 of 577 182 -> 168; d = 128 14204 of 33 238 ->
// 120, 7324 of 64 141 -> 108, 4687 of 100 137 -> 121, 3633 of 129 145 -> 151, 1823 of 257 201 -> 166; d = 96 9765 of 64 113 -> 108, 4844 of 129 115 ->
// 118, 2034 of 320 178 -> 154, 1412 of 384 131 -> 179; d = 16 and 48 of 64 142 -> 103, 112 -> 101, of 197 216 -> 221, 136 -> 143.  Fewer heads: 200 of
// 129, d = 64 7.6 both, of 197 11.5 -> 9.8, of 320, d = 32 9.8 -> 11.0, 300
// of 192, d = 32 6.7 -> 8.3, 200 of 64, d = 128 6.4 -> 7.0.  d = 64 beyond 256 tokens is one workgroup to a compute unit: not where the 256-query
// strips make one round (102 of 480 16.0 -> 19.5, 114 of 450 16.2 -> 19.8, 110 of 415 16.4 -> 18.5; 153 of 400 taken), nor the few heads of a second
// round (263 of 288 18.8 -> 21.3, 320 of 288 20.9 -> 23.2, 257 of 336 24.6 -> 28.4; taken 345 of 288 and 310 of 310, 0.69 times).  d = 32 of 256: 755 15.3 -> 18.1,
// 1648 34 -> 39.
bool prefers_attention_heads(int64_t BH, int64_t N, int64_t d)
{
    const int64_t cus = compute_units(), blocks = BH * ((N + 31) / 32);
    if (2 * blocks < 11 * cus || (d == 32 && BH < 2 * cus)) return false;
    if (d == 64 && N > 256 && 2 * BH <= cus) return false;
    if (d == 64 && N > 256 && N <= 352 && BH > cus && 20 * BH < (N <= 288 ? 27 : 23) * cus) return false;
    if (d == 64) return N > 64 && N <= 480 && N % 256 != 0;    // (256: the tiled kernel's workgroups are full)
    if (d == 32) return N > 64 && N != 256 && (N <= 448 || (N <= 608 && N % 32 != 0));
    if (d <= 48) return N > 32 && N <= 64;
    if (d <= 96) return N > 32 && (N <= 64 || (N > 256 && N <= 320));
    return N > 32 && (N <= 112 || N > 256);
}

hipError_t launch_attention_heads(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d, float scale,
                                  hipStream_t stream)
{
    switch ((int)(d / 16)) {
    case 1: return launch_heads<1, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 2: return launch_heads<1, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 3: return launch_heads<2, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 4: return launch_heads<2, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 5: return launch_heads<3, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 6: return launch_heads<3, false>(Q, K, V, O, BH, (int)N, scale, stream);
    case 7: return launch_heads<4, true>(Q, K, V, O, BH, (int)N, scale, stream);
    case 8: return launch_heads<4, false>(Q, K, V, O, BH, (int)N, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
