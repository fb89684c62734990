// Fused attention weights  P = softmax(scale * Q K^T)  and scaled scores, bf16, a strip of 32 queries per workgroup, up to 1280 keys:
// the keys shared between its waves, the scores in their registers, the strip staged as it lies in memory.
//
// (Paper: the fused kernel of the section "Fused Matrix Multiply + Scaling + Softmax": the scores stay where the matrix multiply left
// them, the cores of a row exchange local maxima and sums, only then are the weights formed and written.)
//
// Wave w owns a run of 32-key blocks.  Nothing of K is used by two waves, so each brings its own blocks to LDS by direct transfers,
// two ahead, and no barrier ties them together until every score is made.  Softmax section, Eq. 1, against the wave's own maximum; one
// exchange of (reference exponent, sum) through LDS.  The area of the K blocks then becomes the way out: the 32 rows of a strip are
// one contiguous piece of P, staged as they lie in memory (N a multiple of 16: row by row with 16 bytes between) and stored as aligned
// 16-byte chunks, consecutive lanes consecutive chunks, whatever N is.  Two barriers per strip; a workgroup ends with its stores, and
// the others of the compute unit are at other phases.
//
// Measured, 192 heads of N = 577, d = 64: 64 -> 41 us (128 MB of P), 160 of 900 142 -> 76, scores of 128 of 1025 110 -> 82; one head of 577
// 16.3 -> 7.5.  Before, a strip's keys were tiles shared by a workgroup that swept them twice (or, up to 608 keys, by persistent workgroups of
// one per compute unit).  What bounds it: the phases of a strip one after the other (K two blocks ahead, exponentials, staging, stores) with
// two to four workgroups on a compute unit to fill each other's, two from N = 600 with eight waves on; every strip brings the K of its
// head again (131 KB at N = 1024, d = 64, for 64 KiB of P), which is why whole tiles of 128 queries stay elsewhere.  Above 1216 keys
// LDS holds one workgroup.
#include "launchers.h"
#include "qk_common.h"

namespace attnw {
namespace {

constexpr int kStripMaxWaves = 8;
constexpr int kStripDump = 48;                    // elements where a wave's keys past its last go (32 + a run of 4)

inline __host__ __device__ int strip_pitch(int N) { return N % 16 == 0 ? N + 8 : N; }
inline __host__ __device__ int strip_area(int N) { return ((32 * strip_pitch(N) + 8) * 2 + 15) / 16 * 16; }

// NT: 32-key blocks of a wave at most; G: 16-element steps of the contraction (d = 16 G: a row padded to fewer instantiations would
// bring an infinity in K to zeros of Q, NaN for a key that weighs nothing); NSLOT: blocks of K a wave holds in LDS
// SCORES: write scale * Q K^T instead of the weights; c is then the scale itself
template <int NT, int G, int NSLOT, bool SCORES>
__global__ __launch_bounds__(64 * kStripMaxWaves, 4)
void qk_strip_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, uint16_t* __restrict__ out, int N, float c,
                     uint32_t sign_flip, uint32_t strips_per_head, uint32_t total_strips)
{
    constexpr int DB = 32 * G, CPR = 2 * G;       // bytes and 16-byte chunks of a row
    // chunk XOR row / RPL stays inside the row and puts the 16 rows that a fragment read serves at a time on different banks
    constexpr int P2 = G % 8 == 0 ? 16 : G % 4 == 0 ? 8 : G % 2 == 0 ? 4 : 2;
    constexpr int RPL = 16 / P2, SWZ_MASK = P2 - 1;
    constexpr int SLOT = 32 * DB;
    extern __shared__ __align__(1024) char lds[];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;

    const uint32_t id = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (id >= total_strips) return;
    const uint32_t h = id / strips_per_head;
    const int q0 = (int)(id - h * strips_per_head) * 32;

    // this wave's blocks of keys
    const int n_blocks = (N + 31) / 32;
    const int b0 = wave * n_blocks / nw;
    const int cnt = (wave + 1) * n_blocks / nw - b0;
    const int key0 = b0 * 32, key_end = min(N, (b0 + cnt) * 32);

    const char* const Kh = reinterpret_cast<const char*>(K) + (int64_t)h * N * DB;
    const uint32_t ring = lds_offset_of(lds) + (uint32_t)(wave * NSLOT * SLOT);
    // block t -> its slot (chunks XOR-swizzled by the row; rows past N are row N - 1 again)
    auto bring = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int s = j * 64 + lane;
            const int row = s / CPR;
            const int chunk = (s % CPR) ^ ((row / RPL) & SWZ_MASK);
            dma16_untracked(Kh + (int64_t)min(key0 + t * 32 + row, N - 1) * DB + chunk * 16,
                            __builtin_amdgcn_readfirstlane(ring + (uint32_t)((t % NSLOT) * SLOT + j * 1024)));
        }
    };
    u32x4 qf[G];
    {
        const char* const p = reinterpret_cast<const char*>(Q) + ((int64_t)h * N + min(q0 + l32, N - 1)) * DB + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(p + g * 32) ^ sign_flip;
    }
#pragma unroll
    for (int t = 0; t < NSLOT; ++t)
        if (t < cnt) bring(t);

    // ---- scores: X[t][r] = q . k for key key0 + 32 t + 8 (r / 4) + 4 half + r % 4 and query q0 + l32 ----
    f32x16 X[NT];
    {
        int frag_off[G];
#pragma unroll
        for (int g = 0; g < G; ++g) frag_off[g] = l32 * DB + (((2 * g + half) ^ ((l32 / RPL) & SWZ_MASK)) * 16);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int r = 0; r < 16; ++r) X[t][r] = 0.0f;
            if (t < cnt) {                        // (wave-uniform)
                // block t has landed: at most the transfers of the blocks after it are outstanding
                if (NSLOT > 1 && t + 1 < cnt) wait_vmem_le<(NSLOT > 1 ? G : 0)>();
                else wait_vmem();
                asm volatile("" ::: "memory");
                const char* const blk = lds + (wave * NSLOT + t % NSLOT) * SLOT;
#pragma unroll
                for (int g = 0; g < G; ++g) Mma<uint16_t>::run(X[t], *reinterpret_cast<const u32x4*>(blk + frag_off[g]), qf[g]);
                if (t + NSLOT < NT && t + NSLOT < cnt) {
                    wait_lds();                   // its fragments have left the slot
                    bring(t + NSLOT);
                }
            }
        }
    }

    // ---- exponentials in place against the wave's own maximum, statistics of the row over the waves (Eq. 1) ----
    float inv = c;                                // SCORES: the scale
    if constexpr (!SCORES) {
        // (keys past N carry the score of key N - 1, whose K row they loaded: the maximum is not theirs alone)
        float m = kNegBig;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t < cnt) {
#pragma unroll
                for (int r = 0; r < 16; r += 2) m = max3(m, X[t][r], X[t][r + 1]);
            }
        }
        m = fmaxf(m, __shfl_xor(m, 32, 64));      // lanes l and l + 32 hold the two halves of a query's keys
        const float mb = reference_exponent(m, c);
        float ls[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // four chains of additions instead of one
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t < cnt) {
                const int kp = key0 + t * 32;
#pragma unroll
                for (int r = 0; r < 16; ++r) X[t][r] = fast_exp2(__builtin_fmaf(X[t][r], c, -mb));
                if (kp + 32 > N) {                // (wave-uniform) keys past N do not count
#pragma unroll
                    for (int r = 0; r < 16; ++r) X[t][r] = kp + 8 * (r / 4) + 4 * half + (r % 4) < N ? X[t][r] : 0.0f;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) ls[r & 3] += X[t][r];
            }
        }
        float l = (ls[0] + ls[1]) + (ls[2] + ls[3]);
        l += __shfl_xor(l, 32, 64);
        // (reference exponent, sum) of every wave and query, behind everything else in LDS
        const int area = strip_area(N) + nw * 2 * kStripDump, rings = nw * NSLOT * SLOT;
        f32x2* const stat = reinterpret_cast<f32x2*>(lds + (area > rings ? area : rings));
        if (half == 0) stat[wave * 32 + l32] = f32x2{mb, l};
        __syncthreads();                          // statistics published, every wave past its K
        float mbg = mb;
        for (int w = 0; w < nw; ++w) mbg = fmaxf(mbg, stat[w * 32 + l32][0]);
        float lg = 0.0f;
        for (int w = 0; w < nw; ++w) {
            const f32x2 s = stat[w * 32 + l32];
            lg += s[1] * fast_exp2(s[0] - mbg);
        }
        inv = fast_exp2(mb - mbg) * __builtin_amdgcn_rcpf(lg);
    } else {
        __syncthreads();                          // every wave past its K
    }

    // ---- the strip as it lies in memory, o = its first element mod 8 ----
    const int rows = min(32, N - q0);
    const int64_t e0 = ((int64_t)h * N + q0) * N;
    const int o = (int)(e0 & 7);                  // (0 where N is a multiple of 8)
    const int pitch = strip_pitch(N);
    uint16_t* const blk = reinterpret_cast<uint16_t*>(lds);
    if (l32 < rows) {
        uint16_t* const rowp = blk + o + l32 * pitch;
        uint16_t* const dump = reinterpret_cast<uint16_t*>(lds + strip_area(N)) + wave * kStripDump;
        // bytes per staging write: 8 while N is a multiple of 4 (runs of 4 keys are whole or absent), 4 while it is even, pairs made up
        // across the half-waves where it is odd
        const int par = (o + l32 * N) & 1;        // (odd N) the row starts on an odd element of the staging area
        auto stage = [&](auto granc) __attribute__((always_inline)) {
            constexpr int GRAN = decltype(granc)::value;
            uint32_t end_val = 0u;
            bool end_here = false;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (t >= cnt) break;              // (wave-uniform)
                const bool last = t + 1 == cnt;   // (wave-uniform) the block after which this wave's keys end
                uint32_t W[8], next01 = 0u;       // the lane's 16 keys as 8 pairs, the first pair of the next block
#pragma unroll
                for (int i = 0; i < 8; ++i) W[i] = pack_bf16x2(X[t][2 * i] * inv, X[t][2 * i + 1] * inv);
                if constexpr (GRAN == 2 && NT > 1) next01 = pack_bf16x2(X[(t + 1) % NT][0] * inv, X[(t + 1) % NT][1] * inv);
                auto put = [&](auto lastc) __attribute__((always_inline)) {
                    constexpr bool LAST = decltype(lastc)::value != 0;
                    uint16_t* const dumpp = dump - (key0 + t * 32);
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const int key = key0 + t * 32 + 8 * r4 + 4 * half;
                        const uint32_t w01 = W[2 * r4], w23 = W[2 * r4 + 1];
                        if constexpr (GRAN == 8) {
                            *reinterpret_cast<u32x2*>((!LAST || key < N ? rowp : dumpp) + key) = u32x2{w01, w23};
                        } else if constexpr (GRAN == 4) {
                            *reinterpret_cast<uint32_t*>((!LAST || key < N ? rowp : dumpp) + key) = w01;
                            *reinterpret_cast<uint32_t*>((!LAST || key + 2 < N ? rowp : dumpp) + key + 2) = w23;
                        } else {
                            // Odd N: a row that starts odd pairs its keys as (1, 2), (3, 4) ...: the second word of a run takes its
                            // upper half from the run that follows in memory, which the other half-wave's lane of the same row
                            // holds (half 0: same r4 of half 1; half 1: the next r4, or the next block, of half 0).  Words with a
                            // key past this wave's last go to the dump area; the elements without a partner here follow below.
                            const uint32_t nxt = r4 < 3 ? W[(2 * r4 + 2) & 7] : next01;
                            uint32_t nw23 = w23;
#if defined(__HIP_DEVICE_COMPILE__)
                            const auto sw = __builtin_amdgcn_permlane32_swap(w01, nxt, false, false);
                            nw23 = half ? sw[0] : sw[1];
#endif
                            const uint32_t W1 = par ? __builtin_amdgcn_alignbit(w23, w01, 16) : w01;
                            const uint32_t W2 = par ? __builtin_amdgcn_alignbit(nw23, w23, 16) : w23;
                            const int k1 = key + par, k2 = key + 2 + par;
                            *reinterpret_cast<uint32_t*>(!LAST || k1 + 1 < key_end ? rowp + k1 : dumpp + key) = W1;
                            *reinterpret_cast<uint32_t*>(!LAST || k2 + 1 < key_end ? rowp + k2 : dumpp + key + 2) = W2;
                            if constexpr (LAST) {
                                const int e = key_end - 1 - key;
                                const uint32_t w = e < 2 ? w01 : w23;
                                if (e >= 0 && e < 4) {
                                    end_val = (e & 1) ? w >> 16 : w;
                                    end_here = true;
                                }
                            }
                        }
                    }
                };
                if (last) put(IC<1>{}); else put(IC<0>{});
            }
            if constexpr (GRAN == 2) {
                // the wave's first element in rows that start odd, its last where the pairs do not end with it
                if (cnt > 0 && par && half == 0) rowp[key0] = (uint16_t)(pack_bf16x2(X[0][0] * inv, 0.0f) & 0xffffu);
                if (end_here && ((key_end - par) & 1)) rowp[key_end - 1] = (uint16_t)(end_val & 0xffffu);
            }
        };
        if ((N & 3) == 0) stage(IC<8>{});
        else if ((N & 1) == 0) stage(IC<4>{});
        else stage(IC<2>{});
    }
    __syncthreads();                              // the strip is complete

    // ---- aligned chunks leave ----
    const int tid = threadIdx.x, nthreads = blockDim.x;
    const int staged = o + rows * N;
    const int n_whole = staged / 8;               // chunks that end inside the strip
    uint16_t* const gbase = out + (e0 - o);       // 16-byte aligned
    if (pitch != N) {                             // (o = 0, every chunk whole and inside one row)
        const uint32_t cpr = (uint32_t)N / 8;
        const uint32_t cpr_inv = ((1u << 20) + cpr - 1u) / cpr;   // ch / cpr = ch * cpr_inv >> 20 for ch < 32 cpr, cpr <= 160
#pragma unroll 4
        for (int ch = tid; ch < n_whole; ch += nthreads) {
            const int row = (int)(((uint32_t)ch * cpr_inv) >> 20);
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(blk + ch * 8 + row * 8), reinterpret_cast<u32x4*>(gbase + ch * 8));
        }
    } else {
        const int first = o != 0 ? 1 : 0;
#pragma unroll 4
        for (int ch = first + tid; ch < n_whole; ch += nthreads)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(blk + ch * 8), reinterpret_cast<u32x4*>(gbase + ch * 8));
        // the chunks shared with the neighbouring strips, element by element
        if (first && tid >= o && tid < 8) gbase[tid] = blk[tid];
        if (tid >= 8 && tid < 8 + (staged & 7)) gbase[n_whole * 8 + tid - 8] = blk[n_whole * 8 + tid - 8];
    }
}

template <int NT, int G>
hipError_t launch_strip_t(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int nw, float scale, hipStream_t stream)
{
    constexpr int NSLOT = G <= 4 ? 2 : 1;
    const int area = strip_area(N) + nw * 2 * kStripDump, rings = nw * NSLOT * 1024 * G;
    const size_t lds = (size_t)((area > rings ? area : rings) + nw * 32 * 8);
    const uint32_t strips = (uint32_t)((N + 31) / 32);
    const float c = scores_only ? scale : fabsf(scale) * kLog2e;
    const uint32_t flip = (!scores_only && scale < 0.0f) ? Mma<uint16_t>::kSignMask : 0u;
    return launch_by_heads(BH, strips, (uint32_t)(64 * nw), [&](int64_t first, int64_t heads) {
        const uint32_t total = (uint32_t)heads * strips;
        const uint32_t grid = (total + 7) / 8 * 8;
        const uint16_t* const q = static_cast<const uint16_t*>(Q) + first * N * 16 * G;
        const uint16_t* const k = static_cast<const uint16_t*>(K) + first * N * 16 * G;
        uint16_t* const p = static_cast<uint16_t*>(out) + first * N * N;
        if (scores_only)
            hipLaunchKernelGGL((qk_strip_kernel<NT, G, NSLOT, true>), dim3(grid), dim3(64 * nw), lds, stream, q, k, p, N, c, flip, strips, total);
        else
            hipLaunchKernelGGL((qk_strip_kernel<NT, G, NSLOT, false>), dim3(grid), dim3(64 * nw), lds, stream, q, k, p, N, c, flip, strips, total);
        return hipGetLastError();
    });
}

template <int NT>
hipError_t launch_strip(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d, int nw, float scale,
                        hipStream_t stream)
{
    switch (d / 16) {
    case 1: return launch_strip_t<NT, 1>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 2: return launch_strip_t<NT, 2>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 3: return launch_strip_t<NT, 3>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 4: return launch_strip_t<NT, 4>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 5: return launch_strip_t<NT, 5>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 6: return launch_strip_t<NT, 6>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 7: return launch_strip_t<NT, 7>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    case 8: return launch_strip_t<NT, 8>(scores_only, Q, K, out, BH, N, nw, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool qk_strip_supported(int64_t BH, int64_t N, int64_t d)
{
    return N > 128 && N <= 1280 && d >= 16 && d <= 128 && d % 16 == 0 && BH <= (int64_t)0x03ffffff;
}

hipError_t launch_qk_strip(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                           hipStream_t stream)
{
    const int blocks = (int)((N + 31) / 32);
    const int nw = blocks > 20 ? 8 : 4;
    switch ((blocks + nw - 1) / nw) {
    case 1:
    case 2: return launch_strip<2>(scores_only, Q, K, out, BH, (int)N, (int)d, nw, scale, stream);
    case 3: return launch_strip<3>(scores_only, Q, K, out, BH, (int)N, (int)d, nw, scale, stream);
    case 4: return launch_strip<4>(scores_only, Q, K, out, BH, (int)N, (int)d, nw, scale, stream);
    default: return launch_strip<5>(scores_only, Q, K, out, BH, (int)N, (int)d, nw, scale, stream);
    }
}

}  // namespace attnw
