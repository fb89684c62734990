// Fused attention weights  P = softmax(scale * Q K^T)  and scaled scores, bf16, N <= 384, d a multiple of 16 up to 256: a wave per
// (head, 32 queries) whose whole row of scores stays in its registers, the K of the head in LDS for the waves of a workgroup.
//
// (Paper: the fused kernel of the section "Fused Matrix Multiply + Scaling + Softmax" holds a block of scores in a core's SRAM from
// the multiply to the store; here a wave's registers hold 32 rows of scores: maximum and sum, Softmax section, Eq. 1, are register
// reductions and one lane exchange.)
//
// One LDS area serves twice: first the K of the head, brought by direct transfers with consecutive lanes on consecutive chunks, then,
// once every wave has its scores, the way out of each wave.  The 32 rows of a block are one contiguous piece of P; a wave stages
// them as they lie in memory (N a multiple of 16: row by row with 16 bytes between, free of bank conflicts) and stores aligned
// 16-byte chunks, consecutive lanes consecutive chunks; the first and last chunk, shared with the neighbouring blocks, element
// by element.  A workgroup is a few blocks of one head and ends with its stores, so nothing ever waits for a store.
//
// Measured, 1024 heads of N = 197, d = 64: 26.7 us (131 MB of Q, K and P: 4.9 TB/s).  The wave-per-head kernel whose waves each took K
// from memory as operands, every lane in a memory line of its own, 44.6 (half of that the vector-memory pipe); the kernel that spread the
// keys of a strip over eight waves, an exchange and a barrier per strip, 49.  Because the K area serves as staging too, three
// workgroups of four waves share a compute unit at that length, each at another phase.  What bounds it: the vector ALU, about 1000
// instructions per wave and 32 x 197 weights (exponentials, scaling and rounding, the pairs of an odd length), 16 of the 28 us,
// in the shadow of the stores.
#include "launchers.h"
#include "qk_common.h"

namespace attnw {
namespace {

constexpr int kHeadsWaves = 4;                    // waves per workgroup at most
constexpr int kDumpElems = 48;                    // where a wave's keys past N go (32 + a run of 4)

// elements of P between staged rows, bytes of a wave's staging area
inline __host__ __device__ int staged_pitch(int N) { return N % 16 == 0 ? N + 8 : N; }
inline __host__ __device__ int area_bytes(int N) { return ((32 * staged_pitch(N) + 8) * 2 + 15) / 16 * 16 + 2 * kDumpElems; }

// NKB: 32-key blocks of a head (32 (NKB - 1) < N <= 32 NKB); G: 16-element steps of the contraction (d = 16 G: a row padded to fewer
// instantiations would bring an infinity in K to zeros of Q, NaN for a key that weighs nothing)
// SCORES: write scale * Q K^T instead of the weights; c is then the scale itself
template <int NKB, int G, bool SCORES>
__global__ __launch_bounds__(64 * kHeadsWaves, (NKB <= 7 && G <= 8) ? 3 : 2)
void qk_heads_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, uint16_t* __restrict__ out, int N, float c,
                     uint32_t sign_flip, uint32_t groups, uint32_t total_groups)
{
    constexpr int DB = 32 * G, CPR = 2 * G;       // bytes and 16-byte chunks of a row
    // chunk XOR row / RPL stays inside the row and puts the 16 rows that a fragment read serves at a time on different banks
    constexpr int P2 = G % 8 == 0 ? 16 : G % 4 == 0 ? 8 : G % 2 == 0 ? 4 : 2;
    constexpr int RPL = 16 / P2, SWZ_MASK = P2 - 1;
    constexpr int LAST = NKB - 1;                 // the block of keys that N may cut
    extern __shared__ __align__(1024) char lds[];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;

    const uint32_t id = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
    if (id >= total_groups) return;
    const uint32_t h = id / groups;
    const int q0 = (int)((id - h * groups) * nw + wave) * 32;

    // ---- K of the head -> LDS (16-byte chunks XOR-swizzled by the row; rows past N are row N - 1 again), Q -> registers ----
    {
        const char* const Kh = reinterpret_cast<const char*>(K) + (int64_t)h * N * DB;
        for (int j = wave; j < NKB * G; j += nw) {
            const int s = j * 64 + lane;
            const int row = s / CPR;
            const int chunk = (s % CPR) ^ ((row / RPL) & SWZ_MASK);
            dma16(Kh + min(row, N - 1) * DB + chunk * 16, lds + j * 1024);
        }
    }
    u32x4 qf[G];
    {
        const char* const p = reinterpret_cast<const char*>(Q) + ((int64_t)h * N + min(q0 + l32, N - 1)) * DB + half * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *reinterpret_cast<const u32x4*>(p + g * 32) ^ sign_flip;
#if defined(__HIP_DEVICE_COMPILE__)
        // in registers before the barrier, under the transfers of K (the compiler sinks these loads behind it, one by one between the
        // matrix instructions: 2048 heads of N = 64, d = 192 23.0 -> 19.5 us, 800 of 129, d = 64 16.9 -> 14.6)
#pragma unroll
        for (int g = 0; g < G; ++g) asm volatile("" : "+v"(qf[g]));
#endif
    }
    wait_vmem();
    __syncthreads();                              // K is in place

    // ---- scores: X[kb][r] = q . k for key 32 kb + 8 (r / 4) + 4 half + r % 4 and query q0 + l32 ----
    f32x16 X[NKB];
    if (q0 < N) {                                 // (wave-uniform)
        int frag_off[G];
#pragma unroll
        for (int g = 0; g < G; ++g) frag_off[g] = l32 * DB + (((2 * g + half) ^ ((l32 / RPL) & SWZ_MASK)) * 16);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) X[kb][r] = 0.0f;
#pragma unroll
            for (int g = 0; g < G; ++g) Mma<uint16_t>::run(X[kb], *reinterpret_cast<const u32x4*>(lds + kb * 32 * DB + frag_off[g]), qf[g]);
        }
    }
    __syncthreads();                              // every wave has read K
    if (q0 >= N) return;

    // ---- row statistics and exponentials in place (Eq. 1) ----
    float inv = c;                                // SCORES: the scale
    if constexpr (!SCORES) {
        // (keys past N carry the score of key N - 1, whose K row they loaded: the maximum is not theirs alone)
        float mx[2] = {kNegBig, kNegBig};
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int r = 0; r < 16; r += 2) mx[(r / 2) & 1] = max3(mx[(r / 2) & 1], X[kb][r], X[kb][r + 1]);
        }
        float m = fmaxf(mx[0], mx[1]);
        m = fmaxf(m, __shfl_xor(m, 32, 64));      // lanes l and l + 32 hold the two halves of a query's keys
        const float mb = m * c;
        float ls[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // four chains of additions instead of one
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                X[kb][r] = fast_exp2(__builtin_fmaf(X[kb][r], c, -mb));
                if (kb == LAST) {                 // keys past N do not count
                    const int key = LAST * 32 + 8 * (r / 4) + 4 * half + (r % 4);
                    X[kb][r] = key < N ? X[kb][r] : 0.0f;
                }
                ls[r & 3] += X[kb][r];
            }
        }
        float l = (ls[0] + ls[1]) + (ls[2] + ls[3]);
        l += __shfl_xor(l, 32, 64);
        inv = __builtin_amdgcn_rcpf(l);
    }

    // ---- the block as it lies in memory, o = its first element mod 8 ----
    const int rows = min(32, N - q0);
    const int64_t e0 = ((int64_t)h * N + q0) * N;
    const int o = (int)(e0 & 7);                  // (0 where N is a multiple of 8)
    const int pitch = staged_pitch(N);
    uint16_t* const blk = reinterpret_cast<uint16_t*>(lds + wave * area_bytes(N));
    {
        uint32_t Wp[NKB][8];                      // the lane's 16 keys of a block as 8 pairs
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int i = 0; i < 8; ++i) Wp[kb][i] = pack_bf16x2(X[kb][2 * i] * inv, X[kb][2 * i + 1] * inv);
        if (l32 < rows) {
            uint16_t* const rowp = blk + o + l32 * pitch;
            // keys past N (last block only) go to a dump area instead: a select of the address, no branch
            uint16_t* const dumpp = blk + (area_bytes(N) / 2 - kDumpElems) - LAST * 32;
            // bytes per staging write: 8 while N is a multiple of 4 (runs of 4 keys are whole or absent), 4 while it is even,
            // pairs made up across the half-waves where it is odd
            const int par = (o + l32 * N) & 1;    // (odd N) the row starts on an odd element of the staging area
            auto stage = [&](auto granc) __attribute__((always_inline)) {
                constexpr int GRAN = decltype(granc)::value;
                uint32_t end_val = 0u;
                bool end_here = false;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const int key = kb * 32 + 8 * r4 + 4 * half;
                        const uint32_t w01 = Wp[kb][2 * r4], w23 = Wp[kb][2 * r4 + 1];
                        auto at = [&](int k) __attribute__((always_inline)) -> uint16_t* {
                            if (kb < LAST) return rowp + k;
                            return (k < N ? rowp : dumpp) + k;
                        };
                        if constexpr (GRAN == 8) {
                            *reinterpret_cast<u32x2*>(at(key)) = u32x2{w01, w23};
                        } else if constexpr (GRAN == 4) {
                            *reinterpret_cast<uint32_t*>(at(key)) = w01;
                            *reinterpret_cast<uint32_t*>(at(key + 2)) = w23;
                        } else {
                            // Odd N: a row that starts odd pairs its keys as (1, 2), (3, 4) ...: the second word of a run takes its
                            // upper half from the run that follows in memory, which the other half-wave's lane of the same row
                            // holds (half 0: same r4 of half 1; half 1: the next r4 of half 0).  Words with a key past N go to the
                            // dump area; the one element per row without a partner in its own row follows below.
                            uint32_t nxt = 0u;    // this lane's first pair of the run after this one
                            if (r4 < 3) nxt = Wp[kb][2 * r4 + 2];
                            else if (kb + 1 < NKB) nxt = Wp[kb + 1 < NKB ? kb + 1 : kb][0];
                            uint32_t nw23 = w23;
#if defined(__HIP_DEVICE_COMPILE__)
                            const auto sw = __builtin_amdgcn_permlane32_swap(w01, nxt, false, false);
                            nw23 = half ? sw[0] : sw[1];
#endif
                            const uint32_t W1 = par ? __builtin_amdgcn_alignbit(w23, w01, 16) : w01;
                            const uint32_t W2 = par ? __builtin_amdgcn_alignbit(nw23, w23, 16) : w23;
                            const int k1 = key + par, k2 = key + 2 + par;
                            uint16_t* const a1 = (kb < LAST || k1 + 1 < N) ? rowp + k1 : dumpp + key;
                            uint16_t* const a2 = (kb < LAST || k2 + 1 < N) ? rowp + k2 : dumpp + key + 2;
                            *reinterpret_cast<uint32_t*>(a1) = W1;
                            *reinterpret_cast<uint32_t*>(a2) = W2;
                            if (kb == LAST && !par) {     // the row's last element (N - 1 is even): the lower half of a word of its own
                                const bool c0 = key == N - 1, c2 = key + 2 == N - 1;
                                end_val = c0 ? w01 : (c2 ? w23 : end_val);
                                end_here = end_here || c0 || c2;
                            }
                        }
                    }
                }
                if constexpr (GRAN == 2) {
                    // the first element of a row that starts odd (key 0: half 0), the last of a row that starts even
                    uint16_t* ae = dumpp + LAST * 32;
                    uint32_t ve = Wp[0][0];
                    if (par) ae = half == 0 ? rowp : ae;
                    else {
                        ae = end_here ? rowp + (N - 1) : ae;
                        ve = end_val;
                    }
                    *ae = (uint16_t)(ve & 0xffffu);
                }
            };
            if ((N & 3) == 0) stage(IC<8>{});
            else if ((N & 1) == 0) stage(IC<4>{});
            else stage(IC<2>{});
        }
    }
    // (the lanes of a wave read what other lanes wrote: LDS serves a wave's operations in order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // ---- aligned chunks leave ----
    const int staged = o + rows * N;
    const int n_whole = staged / 8;               // chunks that end inside the block
    uint16_t* const gbase = out + (e0 - o);       // 16-byte aligned
    if (pitch != N) {                             // (o = 0, every chunk whole and inside one row)
        const uint32_t cpr = (uint32_t)N / 8;
        const uint32_t cpr_inv = (65536u + cpr - 1u) / cpr;   // ch / cpr = ch * cpr_inv >> 16 for ch < 1536
        for (int ch = lane; ch < n_whole; ch += 64) {
            const int row = (int)(((uint32_t)ch * cpr_inv) >> 16);
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(blk + ch * 8 + row * 8), reinterpret_cast<u32x4*>(gbase + ch * 8));
        }
    } else {
        const int first = o != 0 ? 1 : 0;
#pragma unroll 4
        for (int ch = first + lane; ch < n_whole; ch += 64)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(blk + ch * 8), reinterpret_cast<u32x4*>(gbase + ch * 8));
        // the chunks shared with the neighbouring blocks, element by element
        if (first && lane >= o && lane < min(8, staged)) gbase[lane] = blk[lane];
        if (lane >= 8 && lane < 8 + (staged & 7) && n_whole >= first) gbase[n_whole * 8 + lane - 8] = blk[n_whole * 8 + lane - 8];
    }
}

// Waves of a workgroup: as many waves per compute unit as LDS and registers hold, times the share of them that have queries.
inline int heads_waves(int blocks, int N, int k_bytes, int waves_per_simd, int& lds)
{
    int best = 1;
    float most = 0.0f;
    for (int nw = kHeadsWaves; nw >= 1; --nw) {
        const int stage = nw * area_bytes(N), need = stage > k_bytes ? stage : k_bytes;
        int resident = 160 * 1024 / need * nw;
        if (resident > 4 * waves_per_simd) resident = 4 * waves_per_simd / nw * nw;
        const int groups = (blocks + nw - 1) / nw;
        const float score = (float)resident * (float)blocks / (float)(groups * nw);
        if (score > most * 1.01f) {
            most = score;
            best = nw;
            lds = need;
        }
    }
    return best;
}

// K rows of G steps count as so many in the limit of 80 KiB of K
constexpr int counted_steps(int G) { return G <= 4 ? G : G <= 6 ? 6 : G <= 8 ? 8 : G <= 12 ? 12 : 16; }

template <int NKB, int G>
hipError_t launch_heads_t(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, float scale, hipStream_t stream)
{
    if constexpr (NKB * counted_steps(G) > 80) {
        return hipErrorInvalidValue;              // (not supported: see qk_heads_supported)
    } else {
        int lds = 0;
        const int nw = heads_waves(NKB, N, NKB * G * 1024, (NKB <= 7 && G <= 8) ? 3 : 2, lds);
        const uint32_t groups = (uint32_t)((NKB + nw - 1) / nw);
        const float c = scores_only ? scale : fabsf(scale) * kLog2e;
        const uint32_t flip = (!scores_only && scale < 0.0f) ? Mma<uint16_t>::kSignMask : 0u;
        return launch_by_heads(BH, groups, (uint32_t)(64 * nw), [&](int64_t first, int64_t heads) {
            const uint32_t total = (uint32_t)heads * groups;
            const uint32_t grid = (total + 7) / 8 * 8;
            const uint16_t* const q = static_cast<const uint16_t*>(Q) + first * N * 16 * G;
            const uint16_t* const k = static_cast<const uint16_t*>(K) + first * N * 16 * G;
            uint16_t* const p = static_cast<uint16_t*>(out) + first * N * N;
            if (scores_only)
                hipLaunchKernelGGL((qk_heads_kernel<NKB, G, true>), dim3(grid), dim3(64 * nw), (size_t)lds, stream, q, k, p, N, c, flip, groups, total);
            else
                hipLaunchKernelGGL((qk_heads_kernel<NKB, G, false>), dim3(grid), dim3(64 * nw), (size_t)lds, stream, q, k, p, N, c, flip, groups, total);
            return hipGetLastError();
        });
    }
}

template <int NKB>
hipError_t launch_heads(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int N, int d, float scale, hipStream_t stream)
{
    switch (d / 16) {
    case 1: return launch_heads_t<NKB, 1>(scores_only, Q, K, out, BH, N, scale, stream);
    case 2: return launch_heads_t<NKB, 2>(scores_only, Q, K, out, BH, N, scale, stream);
    case 3: return launch_heads_t<NKB, 3>(scores_only, Q, K, out, BH, N, scale, stream);
    case 4: return launch_heads_t<NKB, 4>(scores_only, Q, K, out, BH, N, scale, stream);
    case 5: return launch_heads_t<NKB, 5>(scores_only, Q, K, out, BH, N, scale, stream);
    case 6: return launch_heads_t<NKB, 6>(scores_only, Q, K, out, BH, N, scale, stream);
    case 7: return launch_heads_t<NKB, 7>(scores_only, Q, K, out, BH, N, scale, stream);
    case 8: return launch_heads_t<NKB, 8>(scores_only, Q, K, out, BH, N, scale, stream);
    case 9: return launch_heads_t<NKB, 9>(scores_only, Q, K, out, BH, N, scale, stream);
    case 10: return launch_heads_t<NKB, 10>(scores_only, Q, K, out, BH, N, scale, stream);
    case 11: return launch_heads_t<NKB, 11>(scores_only, Q, K, out, BH, N, scale, stream);
    case 12: return launch_heads_t<NKB, 12>(scores_only, Q, K, out, BH, N, scale, stream);
    case 13: return launch_heads_t<NKB, 13>(scores_only, Q, K, out, BH, N, scale, stream);
    case 14: return launch_heads_t<NKB, 14>(scores_only, Q, K, out, BH, N, scale, stream);
    case 15: return launch_heads_t<NKB, 15>(scores_only, Q, K, out, BH, N, scale, stream);
    case 16: return launch_heads_t<NKB, 16>(scores_only, Q, K, out, BH, N, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// (K of a head, rows counted as above, at most 80 KiB: two workgroups on a compute unit)
bool qk_heads_supported(int64_t BH, int64_t N, int64_t d)
{
    if (N < 1 || N > 384 || d < 16 || d > 256 || d % 16 != 0 || BH > (int64_t)0x0fffffff) return false;
    return (N + 31) / 32 * counted_steps((int)(d / 16)) <= 80;
}

hipError_t launch_qk_heads(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                           hipStream_t stream)
{
    switch ((N + 31) / 32) {
    case 1: return launch_heads<1>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 2: return launch_heads<2>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 3: return launch_heads<3>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 4: return launch_heads<4>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 5: return launch_heads<5>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 6: return launch_heads<6>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 7: return launch_heads<7>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 8: return launch_heads<8>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 9: return launch_heads<9>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 10: return launch_heads<10>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 11: return launch_heads<11>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    case 12: return launch_heads<12>(scores_only, Q, K, out, BH, (int)N, (int)d, scale, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace attnw
