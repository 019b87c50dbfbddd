// Device side of the sequence scorer: its view of the caller's memory and
// the kernel launchers (seqscorer.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "kernels.h"

namespace gambit {

constexpr float kSeqLnEps = 1e-5f;
// Row stride of a head's cached keys and values: max_steps rounded up to a
// multiple of 4 (16-byte loads of four consecutive steps).
__host__ __device__ constexpr int seq_kstride(int max_steps) { return (max_steps + 3) & ~3; }
// Floats of one (trace, layer, head) cache region: keys and values, plus 64
// floats of padding so that regions do not start at the same offset modulo
// a large power of two (every region's first lines would fall on the same
// memory channels).
__host__ __device__ constexpr size_t seq_region_floats(int max_steps) {
  return (size_t)2 * 64 * seq_kstride(max_steps) + 64;
}
enum : int { kEpiNone = 0, kEpiSwiGLU = 1, kEpiAdd = 2 };

struct SeqDev {
  const int32_t* ids;     // [n] listed trace slots, this boundary
  int32_t* lens;          // [max_traces] steps held per slot
  int32_t* err;           // device error word
  float* cache;           // [max_traces][n_layers][n_heads] regions of seq_region_floats: keys [ks / 4][64][4],
                          // values [ks][64], ks = seq_kstride
  const float* ln_out_g;
  const float* ln_out_b;
  const float* w_out;
  int32_t d_model, n_heads, n_layers, max_steps;
};

// fp32 products with W [N][K] row-major, K a multiple of 64:
//   seq_gemm_ln         C = LN(A; lg, lb) W^T, N a multiple of 192 (QKV)
//   seq_gemm_ln_swiglu  C[M][N / 2] = SiLU(a1) * a3 of a = LN(A) W^T, N a
//                       multiple of 128, W_1 and W_3 rows interleaved by 16
//   seq_gemm_add        C += A W^T, N a multiple of 64
// stats [M][columns / 16]: (mean, sum of squared deviations) of every 16
// columns of a row of x, written with x (seq_reduce_in, seq_gemm_add) and
// read by the products that normalise it.
hipError_t seq_gemm_ln(const float* A, const float* W, float* C, int M, int N, int K, const float* lg, const float* lb,
                       const float2* stats, hipStream_t s);
hipError_t seq_gemm_ln_swiglu(const float* A, const float* W, float* C, int M, int N, int K, const float* lg,
                              const float* lb, const float2* stats, hipStream_t s);
hipError_t seq_gemm_add(const float* A, const float* W, float* C, int M, int N, int K, float2* stats, hipStream_t s);
// The input projection's bf16 planes [3][dm][dim] of W_in scaled by the
// input LayerNorm's gain (hi + mid + lo equal it exactly), their row sums c
// and dv = W_in b (one launch, at creation).
hipError_t seq_prep_input(const float* w_in, const float* ln_g, const float* ln_b, int dim, int dm, uint16_t* planes,
                          float* c, float* dv, hipStream_t s);
// The input projection's K splits: enough 64 x 64 tiles for ~256 workgroups,
// at most one per 64 k.
inline int seq_in_splits(int n, int dim, int dm) {
  const long tiles = (long)((n + 63) / 64) * (dm / 64);
  const long s = 256 / tiles;
  return (int)(s < 1 ? 1 : (s < dim / 64 ? s : dim / 64));
}
// part[s][m][c] = split s's share of h W'^T (dim a multiple of 64, dm of 64).
hipError_t seq_proj_in(const uint16_t* h, const uint16_t* planes, int n, int dim, int dm, int splits, float* part,
                       hipStream_t s);
// x = GELU(LN_in(h) W_in^T) from those.
hipError_t seq_reduce_in(const uint16_t* h, int dim, const float* part, int splits, const float* c, const float* dv,
                         float* x, int d, float2* stats, int n, hipStream_t s);
// The output head's scores from x, and the step counts' advance.
hipError_t seq_head(const float* x, int d, const SeqDev& S, float* scores, int n, hipStream_t s);
hipError_t seq_attention(const SeqDev& S, int layer, const float* qkv, float* o, int n, hipStream_t s);
hipError_t seq_fork(const SeqDev& S, const int32_t* pairs, int n, hipStream_t s);
hipError_t seq_set_len(const SeqDev& S, const int32_t* ids, int n, int value, hipStream_t s);

}  // namespace gambit
