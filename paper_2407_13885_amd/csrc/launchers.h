// Internal interface between the C-ABI layer and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace attnw {

enum class DType : int { F32 = 0, BF16 = 1 };

// Row softmax, arguments already validated.  Returns the launch status.
hipError_t launch_softmax(DType in, DType out, const void* S, void* P, int64_t rows, int64_t cols, hipStream_t stream);

// Fused attention weights (scores_only = false) or scaled scores (scores_only = true).
hipError_t launch_qk(DType dt, bool scores_only, const void* Q, const void* K, void* out,
                     int64_t BH, int64_t N, int64_t d, float scale, hipStream_t stream);

// Compute units of the current device (256 if the query fails).
int compute_units();

// A launch may hold less than 2^32 threads; a larger one starts what is left of its size modulo 2^32 and reports no error (seen
// with 2^24 + 64 heads of 256 threads: the first 64 heads had results).  Calls of so many heads go out as several launches:
// part(first head, heads) starts one, its grid at most seven workgroups more than the heads need.  (Heads by multiples of
// eight: an output of 2-byte elements and any N starts on a 16-byte boundary in each of them.)
template <typename Part>
hipError_t launch_by_heads(int64_t BH, uint32_t workgroups_per_head, uint32_t threads, Part&& part)
{
    int64_t most = ((((int64_t)1 << 32) - 1) / threads - 7) / workgroups_per_head;
    if (most >= 8) most &= ~(int64_t)7;
    if (most < 1) return hipErrorInvalidValue;
    for (int64_t first = 0; first < BH; first += most) {
        const hipError_t e = part(first, BH - first < most ? BH - first : most);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// bf16, by the round-based kernel: fused attention weights (statistics of one strip gathered while the
// weights of the previous one are written) or, with scores_only, the scaled scores (one sweep per
// strip through the same staging and store path; d = 64 only).  Only for the shapes
// qk_rounds_supported() accepts.
bool qk_rounds_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_rounds(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d,
                            float scale, hipStream_t stream);

// Fused attention weights, bf16, d = 64, N = 512 or 1024: the scores of a 32-query strip stay in registers
// between the contraction and the normalisation (one sweep over the keys).
bool qk_resident_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_resident(const void* Q, const void* K, void* out, int64_t BH, int64_t N, float scale,
                              hipStream_t stream);

// Fused attention weights or scaled scores, bf16, 8 <= N <= 64, d = 16, many heads: a wave per
// (head, 32 queries) with the K of the head as matrix operands in its registers, no LDS but the way out, no barriers.
bool qk_tiny_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_tiny(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d,
                          float scale, hipStream_t stream);

// Fused attention weights or scaled scores, bf16, N <= 384, d a multiple of 16 up to 256, K of a head at most 80 KiB: a
// wave per (head, 32 queries), the K of the head in LDS for the waves of a workgroup.
bool qk_heads_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_heads(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                           hipStream_t stream);

// Fused attention weights or scaled scores, bf16, 128 < N <= 1280, d a multiple of 16 up to 128: 32 queries per workgroup, the keys
// shared between its waves, scores in their registers.
bool qk_strip_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_strip(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                           hipStream_t stream);

// Fused attention weights or scaled scores, bf16, any N from 513 to 2^22, d a multiple of 16 up to 256: persistent workgroups, strips of 32
// queries whose keys are shared between the waves, the exponentials of up to 1792 keys (768 at d = 256 off the 16-byte boundaries, none up to d = 64) in
// their registers, the rest computed twice.
bool qk_stream_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_stream(bool scores_only, const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                            hipStream_t stream);

// Fused attention weights, bf16, d = 64 or 128, N a multiple of 512 from 1024 to 16384: the scores of a strip stay
// in the registers of the N / 512 workgroups that share its rows (one sweep over the keys; the workgroups exchange
// their row statistics through tables parked in P).  Two launches: table slots zeroed, then the kernel.
bool qk_gang_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_gang(const void* Q, const void* K, void* out, int64_t BH, int64_t N, int64_t d, float scale,
                          hipStream_t stream);

// Fused attention weights, fp32, d a multiple of 4 up to 128, N a multiple of 4: the contraction on the bf16 instruction,
// operands in three parts, K split once per 128 queries.
// (Scores of operands in parts carry a factor of 2^48 that leaves with the scale, which stays a normal number only from here on.)
inline bool split_takes_scale(float scale) { return scale == 0.0f || scale >= 0x1p-78f || scale <= -0x1p-78f; }
hipError_t launch_qk_f32_split(const void* Q, const void* K, void* P, int64_t BH, int64_t N, int64_t d, float scale, hipStream_t stream);

// Fused attention weights or scaled scores, fp32, any N with N d < 2^28, d a multiple of 4 up to 256: the same with 32-query strips whose
// scores stay in the registers of a workgroup (up to 2048 keys; the rest computed twice).
hipError_t launch_qk_f32_strip(bool scores_only, const void* Q, const void* K, void* P, int64_t BH, int64_t N, int64_t d, float scale,
                               hipStream_t stream);

// Fused attention weights, fp32, few heads of N up to 256 (d above 128: 192), d a multiple of 4 from 20 to 256: workgroups of 16 queries, K straight from memory.
bool prefers_f32_small(int64_t BH, int64_t N, int64_t d);
hipError_t launch_qk_f32_small(const void* Q, const void* K, void* P, int64_t BH, int64_t N, int64_t d, float scale, hipStream_t stream);

// Y = scale * X over count elements, rounded once to the storage type; X == Y allowed.
hipError_t launch_scale(DType dt, const void* X, void* Y, int64_t count, float scale, hipStream_t stream);

// Attention output O = softmax(scale Q K^T) V, bf16, d = 32 or 64, any N >= 1 (tiled through LDS).
bool attention_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                            float scale, hipStream_t stream);

// The same for fp32 (d a multiple of 4 up to 256): both contractions on the fp32 matrix instruction, tiled through LDS.
bool attention_f32_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_f32(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                float scale, hipStream_t stream);

// The same for many heads (d a multiple of 4, 36 to 128 and up to 32): both contractions on the bf16 instruction, operands in three parts.
hipError_t launch_attention_f32_turns(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                      float scale, hipStream_t stream);
hipError_t launch_attention_f32_split(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                      float scale, hipStream_t stream);

// The same for the other multiples of 16 up to 256: tiled through LDS, V turned by the transposing LDS read.
bool attention_wide_supported(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_wide(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                    float scale, hipStream_t stream);

// The same for d a multiple of 16 from 96 to 160 and N > 128, queries 0 .. q_end - 1 of every head, workgroups of four or eight waves: matrix and
// vector work of neighbouring tiles under way at once.  attention_pipe_waves: of how many where it is the faster one, else 0.
// attention_pipe_64, attention_pipe_32: whether four waves there are the faster ones at d = 64, 32 (workgroups of four only).
bool attention_pipe_supported(int64_t N, int64_t d);
bool attention_pipe_64(int64_t BH, int64_t N);
bool attention_pipe_32(int64_t BH, int64_t N);
int attention_pipe_waves(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_pipe(int waves, const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d, float scale,
                                 int q_end, hipStream_t stream);

// The same for d a multiple of 16 from 176 to 256, queries 0 .. q_end - 1 of every head: the two waves of a SIMD take turns at the matrix unit.
bool prefers_attention_turns(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_turns(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d, float scale,
                                  int q_end, hipStream_t stream);

// The same for a few heads (bf16, d a multiple of 16 up to 256), queries q_base .. N - 1 of every head: the keys of a query
// block shared between the waves of a workgroup.
bool prefers_attention_ranges(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_ranges(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                   float scale, int q_base, hipStream_t stream);

// The same for sequences of at most 32 tokens with 128 < d <= 256 (bf16: a multiple of 16, fp32: of 4): a wave per head, operands
// straight from global memory.
hipError_t launch_attention_short(DType dt, const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                  float scale, hipStream_t stream);

// The same for sequences whose K and V fit the LDS (bf16, d a multiple of 16 up to 128): a wave per (head, 32 queries), K and V of the head
// shared by the waves of a workgroup.
bool attention_heads_supported(int64_t BH, int64_t N, int64_t d);
bool prefers_attention_heads(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_heads(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d, float scale,
                                  hipStream_t stream);

// The same for many short sequences (bf16, d = 64 with N <= 128, d = 32 with N <= 224): a wave per (head, 32 queries), operands
// straight from global memory, the exponentials as they stand the operand of the second contraction.
bool attention_tiny_supported(int64_t BH, int64_t N, int64_t d);
bool prefers_attention_tiny(int64_t BH, int64_t N, int64_t d);
hipError_t launch_attention_tiny(const void* Q, const void* K, const void* V, void* O, int64_t BH, int64_t N, int64_t d,
                                 float scale, hipStream_t stream);

}  // namespace attnw
