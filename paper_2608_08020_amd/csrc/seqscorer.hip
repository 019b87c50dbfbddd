// The history-aware sequence scorer (App. A.1, Eqs. 4-6), one new step per
// trace per thought boundary against cached keys and values of the trace's
// earlier steps.  fp32 weights, activations and caches; the step states
// arrive in bf16, and the input projection runs on the bf16 matrix cores
// with fp32 sums, its weights (scaled by the input LayerNorm's gain) split
// exactly into three bf16 planes when the scorer is created.
//
// Per boundary, for the n listed traces (rows):
//   x  = GELU(LN_in(h) W_in^T)             proj_in_kernel (h against the
//                                           planes, K split);
//                                           reduce_in_kernel (the splits
//                                           added, LN_in applied)
//   per layer: qkv = LN1(x) Wqkv^T; o = attention step (RoPE, append the step's
//   key and value, attend over the trace's steps 0..t); x += o Wo^T;
//   g = SiLU(LN2(x) W1^T) * (LN2(x) W3^T); x += g W2^T
//   y  = sigmoid(w_out . LN_out(x)), and the trace's step count advances.
// Each product takes the LayerNorm before it on its operand's way in and the
// residual or the gate on its result's way out: 13 launches per boundary with
// two layers.
#include <hip/hip_runtime.h>

#include "lds_dma.h"
#include "seq_kernels.h"

namespace gambit {
namespace {

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ inline float gelu_erf(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }

typedef float f32x4 __attribute__((ext_vector_type(4)));

// A 16-byte load with the non-temporal hint (the attention step's cached
// keys: each is read once per boundary, and the history of all traces is
// far larger than L2).  Measured at 512 traces, history 128: 23.5-23.9 vs
// 24.7-26.7 us per attention step; the same hint on the values as well
// made it slower (26.5-27.6 us).
__device__ inline float4 ld_stream4(const float* p) {
  const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}

// Sum over the four lanes (l / 16) that hold a row of an operand.
__device__ inline float row_sum(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// Sum over the 16 lanes of a lane group, in every lane, by data-parallel
// moves (quad xor 1 and 2, half-row mirror, row mirror).
template <int CTRL>
__device__ inline float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ inline float group_sum(float v) {
  v = dpp_add<0xB1>(v);
  v = dpp_add<0x4E>(v);
  v = dpp_add<0x141>(v);
  return dpp_add<0x140>(v);
}

// (mean, sum of squared deviations) over the 16 lanes of a lane group: 16
// consecutive columns of a row.
__device__ inline float2 row_stats(float x) {
  const float mean = group_sum(x) * 0.0625f, e = x - mean;
  return make_float2(mean, group_sum(e * e));
}

// C = f(A) W^T on the fp32 matrix cores (v_mfma_f32_16x16x4f32), f = LayerNorm
// of A's rows (LN) or nothing.  A workgroup takes a tile of 16 MB rows x 16 NB
// columns and splits K over its NW waves: wave w takes slabs (of 32 k) [w G /
// NW, (w + 1) G / NW) of the G = K / 32, and the waves' sums meet in LDS.
// These products are short (K = 256 or 768, 0.07-0.4 GFLOP at 512 rows): what
// bounds them is the round trip to the operands, the rate at which a CU takes
// them from L2, and the launch.  So a wave asks for two slabs of both operands
// at once, by direct loads into LDS that only it reads (no barrier), eight
// rows of 128 bytes per load (whole lines, where the matrix cores' own operand
// shape, 16 rows of 64 bytes, takes half of each).  Per boundary of 512 traces (d_model 256, d_ff 768, two
// layers) the eight products take 56 us; split over workgroups, the split sums
// through memory and a launch each to add them and take the LayerNorm, they
// and the four reduces took 70 us.
//
// LDS: a slab's rows are 128 bytes; row r's 16-byte chunk c sits at position
// c ^ ((r >> 1) & 7), so the 16 rows of an operand read fall on 16 different
// bank groups.  A lane reads 4 consecutive k of its row (16 bytes) and feeds
// them to 4 successive products: lane (q, i) contributes A[i][4q + kk] and
// W[i][4q + kk] to product kk, the same k for both operands; result element
// (4 (l / 16) + r, l % 16) sits in lane l, register r.
//
// LN: the rows' mean and mean squared deviation come from the kernel that
// wrote A, as (mean, sum of squared deviations) of every 16 columns
// (row_stats): equal counts, so the row's mean is the mean of the means and
// its squared deviations are the blocks' plus 16 times those of their means.
// (Measured and not kept: the row's sums taken from the operands, two barriers,
// 12.9 against 9.5 us for SwiGLU; the products on x as it is with W scaled by
// the gain, mean and bias added at the end, 11.6 us; eight waves of one slab
// instead of four of two, 10.8 us.)
//
// Epilogues: kEpiNone C = sum; kEpiAdd C += sum (the residual; C is not read
// by another workgroup) and the new row's statistics; kEpiSwiGLU: W holds W_1
// and W_3 rows interleaved in groups of 16, so column blocks 2 c and 2 c + 1
// are W_1 and W_3 of the same 16 outputs, and C[m][16 c + i] = SiLU(a1) * a3
// with row stride N / 2.
template <int MB, int NB, int NW, bool LN, int EPI>
__global__ __launch_bounds__(64 * NW) void gemm_kernel(const float* A, const float* W, float* C, int M, int N, int K,
                                                       const float* lg, const float* lb, float2* stats) {
  static_assert(EPI != kEpiSwiGLU || NB % 2 == 0, "W_1 and W_3 blocks in pairs");
  constexpr int SB = 2;                        // slabs asked for at once
  constexpr int kSlab = 16 * (MB + NB) * 128;  // bytes of one slab of both operands: A's rows, then W's
  constexpr int kLoads = 2 * (MB + NB);        // 1 KB loads per slab
  constexpr int T4 = MB * NB * 64;             // the tile in f32x4
  constexpr int kLds = NW * SB * kSlab > NW * T4 * 16 ? NW * SB * kSlab : NW * T4 * 16;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kLds];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * 16 * MB, n0 = blockIdx.x * 16 * NB;
  const int G = K / 32, g0 = wave * G / NW, g1 = (wave + 1) * G / NW;
  uint8_t* mine = lds + wave * SB * kSlab;
  // load d of a slab: rows 8 d .. 8 d + 7 (A's, then W's), lane l chunk
  // position l % 8 of row l / 8; rows past M re-read the last (never stored)
  auto fetch = [&](int g, int slot) {
    uint8_t* dst = mine + slot * kSlab;
#pragma unroll
    for (int d = 0; d < kLoads; ++d) {
      const int r = 8 * d + (lane >> 3);
      const int k = 32 * g + 4 * ((lane & 7) ^ ((r >> 1) & 7));
      const float* src = d < 2 * MB ? A + (size_t)min(m0 + r, M - 1) * K + k : W + (size_t)(n0 + r - 16 * MB) * K + k;
      dma16(src, dst + d * 1024);
    }
  };
  // the rows' statistics: lane (q, i) takes blocks q nb .. q nb + nb - 1 of
  // row i, the first four in registers
  const int nb = K / 64;
  const float2* sp[LN ? MB : 1];
  float2 st[LN ? MB : 1][4];
  if constexpr (LN) {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      sp[i] = stats + (size_t)min(m0 + 16 * i + li, M - 1) * (K / 16) + lq * nb;
#pragma unroll
      for (int k = 0; k < 4; ++k) st[i][k] = sp[i][min(k, nb - 1)];
    }
  }
  f32x4 gv[LN ? 2 : 1], bv[LN ? 2 : 1];  // gain and bias of the slab's two halves
  auto load_ln = [&](int g) {
    if constexpr (LN) {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        gv[x] = *reinterpret_cast<const f32x4*>(lg + 32 * g + 16 * x + 4 * lq);
        bv[x] = *reinterpret_cast<const f32x4*>(lb + 32 * g + 16 * x + 4 * lq);
      }
    }
  };
  if (g0 < g1) load_ln(g0);
#pragma unroll
  for (int k = 0; k < SB; ++k)
    if (g0 + k < g1) fetch(g0 + k, k);
  float rstd[MB], shift[MB];  // LN(x) = (x rstd + shift) gain + bias
  if constexpr (LN) {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      float s = 0.f, v = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) s += k < nb ? st[i][k].x : 0.f;
      for (int k = 4; k < nb; ++k) s += sp[i][k].x;
      const float mean = row_sum(s) / (4 * nb);
      auto dev = [&](const float2& x) {
        const float e = x.x - mean;
        return x.y + 16.f * e * e;
      };
#pragma unroll
      for (int k = 0; k < 4; ++k) v += k < nb ? dev(st[i][k]) : 0.f;
      for (int k = 4; k < nb; ++k) v += dev(sp[i][k]);
      rstd[i] = 1.f / sqrtf(row_sum(v) / K + kSeqLnEps);
      shift[i] = -mean * rstd[i];
    }
  }
  f32x4 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int at = li * 128, sw = (li >> 1) & 7;
  for (int g = g0, slot = 0; g < g1; ++g) {
    // slab g is in: at most the kLoads loads of the next one are on their way
    if (g + 1 < g1)
      wait_vmcnt<kLoads>();
    else
      wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const uint8_t* src = mine + slot * kSlab + at;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int pos = ((4 * x + lq) ^ sw) * 16;
      f32x4 a[MB], w[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        a[i] = *reinterpret_cast<const f32x4*>(src + i * 2048 + pos);
        if constexpr (LN) a[i] = (a[i] * rstd[i] + shift[i]) * gv[x] + bv[x];
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) w[j] = *reinterpret_cast<const f32x4*>(src + (MB + j) * 2048 + pos);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], w[j][e], acc[i][j], 0, 0, 0);
    }
    if (g + 1 < g1) load_ln(g + 1);
    if (g + SB < g1) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this slab's reads are done
      fetch(g + SB, slot);
    }
    slot = slot + 1 == SB ? 0 : slot + 1;
  }
  __syncthreads();  // every wave is done with its slabs
  f32x4* sums = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) sums[wave * T4 + (i * NB + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  auto total = [&](int p) {  // the waves' sums, in order
    f32x4 v = sums[p];
#pragma unroll
    for (int x = 1; x < NW; ++x) v += sums[x * T4 + p];
    return v;
  };
  if constexpr (EPI == kEpiSwiGLU) {
    for (int p = wave; p < MB * NB / 2; p += NW) {
      const int i = p / (NB / 2), c = p % (NB / 2);
      const f32x4 x = total((i * NB + 2 * c) * 64 + lane), y = total((i * NB + 2 * c + 1) * 64 + lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * i + 4 * lq + r;
        if (m < M) C[(size_t)m * (N / 2) + n0 / 2 + 16 * c + li] = x[r] / (1.f + expf(-x[r])) * y[r];
      }
    }
  } else {
    for (int p = wave; p < MB * NB; p += NW) {
      const int i = p / NB, j = p % NB;
      f32x4 v = total(p * 64 + lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * i + 4 * lq + r;
        float* o = C + (size_t)min(m, M - 1) * N + n0 + 16 * j + li;
        if constexpr (EPI == kEpiAdd) {
          v[r] += *o;
          const float2 rs = row_stats(v[r]);
          if (li == 0 && m < M) stats[(size_t)m * (N / 16) + n0 / 16 + j] = rs;
        }
        if (m < M) *o = v[r];
      }
    }
  }
}

// The same product with LayerNorm for large ones, whose time is the matrix
// cores' and not the round trip: TM x 64 tiles, the four waves share both
// operands, staged in LDS 128 k at a time (rows padded to 132 floats, so the 16
// rows of an operand read fall on 16 different bank groups), the next chunk's
// loads in flight in registers while this one is multiplied; each wave takes a
// (TM / 2) x 32 quarter.  A is normalised on its way into LDS; a chunk's sums
// are added to the tile's at its end, so the rounding stays that of 128
// products and K / 128 sums.
constexpr int kKC = 128;      // k per staged chunk
constexpr int kKP = kKC + 4;  // padded LDS row, floats
template <int TM, int EPI>
__global__ __launch_bounds__(256) void gemm_wide_kernel(const float* A, const float* W, float* C, int M, int N, int K,
                                                        const float* lg, const float* lb, const float2* stats) {
  constexpr int MB = TM / 32;  // 16-row blocks per wave
  constexpr int AV = TM / 8, WV = 8;  // float4 groups of A and of W per thread and chunk
  constexpr int kPer = 256 / TM;      // threads per row's statistics
  __shared__ __attribute__((aligned(16))) float As[TM * kKP];
  __shared__ __attribute__((aligned(16))) float Ws[64 * kKP];
  __shared__ float2 norm[TM];  // LN(x) = (x norm.x + norm.y) gain + bias
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * 64;
  const int li = lane & 15, lq = lane >> 4;
  const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * 32;
  // group v of a thread is row lr + 8 v, k offset lk
  const int lk = 4 * (tid & 31), lr = tid >> 5;
  f32x4 ar[AV], wr[WV], gv, bv;
  // chunk [kb, kb + kKC), groups past K are zero and read nothing; rows past M
  // re-read the last (never stored)
  auto fetch = [&](int kb) {
    const bool kin = kb + lk < K;
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    gv = kin ? *reinterpret_cast<const f32x4*>(lg + kb + lk) : zero;
    bv = kin ? *reinterpret_cast<const f32x4*>(lb + kb + lk) : zero;
#pragma unroll
    for (int v = 0; v < AV; ++v)
      ar[v] = kin ? *reinterpret_cast<const f32x4*>(A + (size_t)min(m0 + lr + 8 * v, M - 1) * K + kb + lk) : zero;
#pragma unroll
    for (int v = 0; v < WV; ++v)
      wr[v] = kin ? *reinterpret_cast<const f32x4*>(W + (size_t)(n0 + lr + 8 * v) * K + kb + lk) : zero;
  };
  fetch(0);
  {
    const int r = tid / kPer, nb = K / 16;
    const float2* sp = stats + (size_t)min(m0 + r, M - 1) * nb;
    auto row = [&](float v) {
#pragma unroll
      for (int o = 1; o < kPer; o <<= 1) v += __shfl_xor(v, o);
      return v;
    };
    float s = 0.f, v = 0.f;
    for (int b = tid % kPer; b < nb; b += kPer) s += sp[b].x;
    const float mean = row(s) / nb;
    for (int b = tid % kPer; b < nb; b += kPer) {
      const float2 x = sp[b];
      const float e = x.x - mean;
      v += x.y + 16.f * e * e;
    }
    const float rstd = 1.f / sqrtf(row(v) / K + kSeqLnEps);
    if (tid % kPer == 0) norm[r] = make_float2(rstd, -mean * rstd);
  }
  __syncthreads();
  float2 nr[AV];
#pragma unroll
  for (int v = 0; v < AV; ++v) nr[v] = norm[lr + 8 * v];
  f32x4 acc[MB][2], sum[MB][2];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = 0; kb < K; kb += kKC) {
    __syncthreads();  // the previous chunk's reads are done
#pragma unroll
    for (int v = 0; v < AV; ++v)
      *reinterpret_cast<f32x4*>(&As[(lr + 8 * v) * kKP + lk]) = (ar[v] * nr[v].x + nr[v].y) * gv + bv;
#pragma unroll
    for (int v = 0; v < WV; ++v) *reinterpret_cast<f32x4*>(&Ws[(lr + 8 * v) * kKP + lk]) = wr[v];
    __syncthreads();
    if (kb + kKC < K) fetch(kb + kKC);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kn = min(kKC, K - kb);  // a multiple of 64
    for (int kc = 0; kc < kn; kc += 16) {
      f32x4 a[MB], w[2];
#pragma unroll
      for (int i = 0; i < MB; ++i) a[i] = *reinterpret_cast<const f32x4*>(&As[(wm + 16 * i + li) * kKP + kc + 4 * lq]);
#pragma unroll
      for (int j = 0; j < 2; ++j) w[j] = *reinterpret_cast<const f32x4*>(&Ws[(wn + 16 * j + li) * kKP + kc + 4 * lq]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], w[j][e], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) sum[i][j] += acc[i][j];
  }
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm + 16 * i + 4 * lq + r;
      if (m >= M) continue;
      if constexpr (EPI == kEpiSwiGLU) {  // the wave's column blocks are W_1 and W_3 of the same 16 outputs
        const float x = sum[i][0][r], y = sum[i][1][r];
        C[(size_t)m * (N / 2) + (n0 + wn) / 2 + li] = x / (1.f + expf(-x)) * y;
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) C[(size_t)m * N + n0 + wn + 16 * j + li] = sum[i][j][r];
      }
    }
}

__device__ inline float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();  // red[] is free
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// The output head, one wave per row: LN_out of x (mean, then the mean squared
// deviation), scores[row] = sigmoid(w_out . LN_out(x)), and the trace's step
// count advances.
__global__ __launch_bounds__(256) void head_kernel(const float* x, int d, SeqDev S, float* scores, int n) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  const f32x4* xr = reinterpret_cast<const f32x4*>(x + (size_t)row * d);
  const f32x4 *g = reinterpret_cast<const f32x4*>(S.ln_out_g), *b = reinterpret_cast<const f32x4*>(S.ln_out_b),
              *w = reinterpret_cast<const f32x4*>(S.w_out);
  const int nd = d / 4;
  // the lane's first element group of everything (all of d_model 256) at once
  const int at = min(lane, nd - 1);
  const f32x4 x0 = xr[at], g0 = g[at], b0 = b[at], w0 = w[at];
  const bool in = lane < nd;
  auto sum4 = [](const f32x4& v) { return (v[0] + v[1]) + (v[2] + v[3]); };
  float s = in ? sum4(x0) : 0.f;
  for (int i = lane + 64; i < nd; i += 64) s += sum4(xr[i]);
  const float mean = wave_sum(s) / d;
  float v = in ? sum4((x0 - mean) * (x0 - mean)) : 0.f;
  for (int i = lane + 64; i < nd; i += 64) v += sum4((xr[i] - mean) * (xr[i] - mean));
  const float rstd = 1.f / sqrtf(wave_sum(v) / d + kSeqLnEps);
  float z = in ? sum4(((x0 - mean) * rstd * g0 + b0) * w0) : 0.f;
  for (int i = lane + 64; i < nd; i += 64) z += sum4(((xr[i] - mean) * rstd * g[i] + b[i]) * w[i]);
  z = wave_sum(z);
  if (lane == 0) {
    scores[row] = 1.f / (1.f + expf(-z));
    S.lens[S.ids[row]] += 1;
  }
}

// The input projection h W'^T, W' in its three bf16 planes, on the bf16 matrix
// cores: part[s][m][c] is split s's share.  A workgroup (eight waves) takes 64
// rows x 64 columns of one split, all three planes: they share the rows'
// operands, and one sum leaves instead of three - hi and mid + lo are summed
// apart (the small planes' sums round at their own size) and added at the end.
// Bound by the operands' way through LDS and by the partial sums' way to the
// reduce: with a product of N = 3 d_model in 128 x 128 tiles, 15.7 MB of them
// at 512 rows x 4096 -> 256, 10.4 us and 6.8 us for the reduce; 4.2 MB so, 8.7
// and 5.1 us.
//
// LDS: a ring of four slabs of 64 k, three in flight by direct loads; a slab
// holds 256 rows of 128 bytes, the 64 of h, then each plane's 64.  Row r's
// 16-byte chunk c sits at c ^ ((r >> 1) & 7), so the 16 rows of an operand
// read fall on 16 different bank groups.  Wave w fills rows 32 w .. 32 w + 31
// and computes rows 32 (w & 1) .. + 31, columns 16 (w >> 1) .. + 15.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kInTile = 64, kInRows = 4 * kInTile, kInSlab = kInRows * 128, kInStages = 4, kInWaves = 8;

__global__ __launch_bounds__(64 * kInWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void proj_in_kernel(
    const uint16_t* h, const uint16_t* planes, int n, int dim, int dm, int splits, float* part) {
  constexpr int kLoads = kInRows / 8 / kInWaves;  // 8-row loads per wave and slab
  __shared__ __attribute__((aligned(1024))) uint8_t ring[kInStages * kInSlab];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // items in (split, column tile, row tile) order; workgroup b runs on XCD b %
  // 8, and an XCD takes consecutive items (few splits' operands in its L2)
  const int G = gridDim.x;
  const int item = (G & 7) ? blockIdx.x : (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);
  const int tm = (n + kInTile - 1) / kInTile, tc = dm / kInTile;
  const int s = item / (tm * tc), tile = item - s * tm * tc;
  const int c0 = tile / tm * kInTile, m0 = tile % tm * kInTile;
  const int slabs = dim / 64;
  const int g0 = s * slabs / splits, ng = (s + 1) * slabs / splits - g0;
  const uint16_t* src[kLoads];
#pragma unroll
  for (int d = 0; d < kLoads; ++d) {
    const int r = 32 * wave + 8 * d + (lane >> 3);
    const uint16_t* row = r < kInTile ? h + (size_t)min(m0 + r, n - 1) * dim  // rows past n re-read the last (never stored)
                                      : planes + ((size_t)(r / kInTile - 1) * dm + c0 + r % kInTile) * dim;
    src[d] = row + 64 * g0 + 8 * ((lane & 7) ^ ((r >> 1) & 7));
  }
  auto issue = [&](int g) {
    uint8_t* st = ring + (g % kInStages) * kInSlab + wave * kLoads * 1024;
#pragma unroll
    for (int d = 0; d < kLoads; ++d) dma16(src[d] + 64 * g, st + d * 1024);
  };
  const int i = lane & 15, q = lane >> 4, sw = (i >> 1) & 7;
  const int mr = 32 * (wave & 1), cr = 16 * (wave >> 1);
  f32x4 hi[2], lo[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) hi[a] = lo[a] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int g = 0; g < kInStages - 1 && g < ng; ++g) issue(g);
  for (int g = 0; g < ng; ++g) {
    switch (min(kInStages - 2, ng - 1 - g)) {  // slabs asked for after this one
      case 2: wait_vmcnt<2 * kLoads>(); break;
      case 1: wait_vmcnt<kLoads>(); break;
      default: wait_vmcnt<0>(); break;
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of slab g - 1 are done
    barrier_no_fence();                  // slab g is in; every wave is done with slab g - 1
    if (g + kInStages - 1 < ng) issue(g + kInStages - 1);
    const uint8_t* st = ring + (g % kInStages) * kInSlab + i * 128;
    bf16x8 A[2][2], B[2][3];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int pos = ((4 * x + q) ^ sw) * 16;
#pragma unroll
      for (int a = 0; a < 2; ++a) A[x][a] = *reinterpret_cast<const bf16x8*>(st + (mr + 16 * a) * 128 + pos);
#pragma unroll
      for (int p = 0; p < 3; ++p) B[x][p] = *reinterpret_cast<const bf16x8*>(st + (kInTile * (p + 1) + cr) * 128 + pos);
    }
    __builtin_amdgcn_sched_barrier(0);  // all ten reads are issued before the first product
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        lo[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[x][a], B[x][2], lo[a], 0, 0, 0);
        hi[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[x][a], B[x][0], hi[a], 0, 0, 0);
        lo[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[x][a], B[x][1], lo[a], 0, 0, 0);
      }
  }
  // lane (q, i) holds rows mr + 16 a + 4 q + e of column cr + i: 64 consecutive
  // bytes of four rows per store
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + mr + 16 * a + 4 * q + e;
      if (m < n) part[((size_t)s * n + m) * dm + c0 + cr + i] = hi[a][e] + lo[a][e];
    }
}

// The input projection's reduce, one workgroup per row: the input
// LayerNorm's statistics of h[row] (mean, then the mean squared deviation),
// the split partial sums of h W'^T (part [splits][n][d]) added split by split
// in order, then x = GELU(rstd (y - mean c[i]) + dv[i]) (LN_in(h) W_in^T
// rearranged: c = the row sums of W', dv = W_in b).  The state's first 4096 values (four 8-byte loads per thread, kept in
// registers for both statistics passes) and the first column's partial sums
// of up to kInBatch splits are all requested before any of them is used.
constexpr int kInBatch = 16;

__global__ __launch_bounds__(256) void reduce_in_kernel(const uint16_t* h, int dim, const float* part, int splits,
                                                        const float* c, const float* dv, float* x, int d, float2* stats,
                                                        int n) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const uint2* h4 = reinterpret_cast<const uint2*>(h + (size_t)row * dim);  // four bf16 per load
  const int nh4 = dim / 4;
  const size_t MN = (size_t)n * d, base = (size_t)row * d;
  // split partials of column i, splits z0 .. z0 + kInBatch - 1 (indices
  // clamped: every load is in bounds; only splits < `splits` are added)
  float v[kInBatch];
  auto load_parts = [&](int i, int z0) {
#pragma unroll
    for (int e = 0; e < kInBatch; ++e) v[e] = part[(size_t)min(z0 + e, splits - 1) * MN + base + i];
  };
  uint2 hr[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) hr[j] = tid + 256 * j < nh4 ? h4[tid + 256 * j] : make_uint2(0u, 0u);
  if (tid < d) load_parts(tid, 0);
  auto f4 = [](uint2 w, float* o) {
    o[0] = __uint_as_float(w.x << 16), o[1] = __uint_as_float(w.x & 0xFFFF0000u);
    o[2] = __uint_as_float(w.y << 16), o[3] = __uint_as_float(w.y & 0xFFFF0000u);
  };
  float hs = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {  // zeros past the row add nothing
    float e[4];
    f4(hr[j], e);
    hs += (e[0] + e[1]) + (e[2] + e[3]);
  }
  for (int i = tid + 1024; i < nh4; i += 256) {
    float e[4];
    f4(h4[i], e);
    hs += (e[0] + e[1]) + (e[2] + e[3]);
  }
  const float hmean = block_sum(hs, red) / dim;
  float hv = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (tid + 256 * j < nh4) {
      float e[4];
      f4(hr[j], e);
#pragma unroll
      for (int k = 0; k < 4; ++k) hv += (e[k] - hmean) * (e[k] - hmean);
    }
  }
  for (int i = tid + 1024; i < nh4; i += 256) {
    float e[4];
    f4(h4[i], e);
#pragma unroll
    for (int k = 0; k < 4; ++k) hv += (e[k] - hmean) * (e[k] - hmean);
  }
  const float hrstd = 1.f / sqrtf(block_sum(hv, red) / dim + kSeqLnEps);
  for (int i = tid; i < d; i += 256) {
    float y = 0.f;
    for (int z0 = 0; z0 < splits; z0 += kInBatch) {
      if (i != tid || z0 != 0) load_parts(i, z0);
#pragma unroll
      for (int e = 0; e < kInBatch; ++e)
        if (z0 + e < splits) y += v[e];
    }
    y = gelu_erf(hrstd * (y - hmean * c[i]) + dv[i]);
    x[base + i] = y;
    const float2 st = row_stats(y);  // d is a multiple of 16: whole lane groups
    if ((tid & 15) == 0) stats[base / 16 + i / 16] = st;
  }
}

// The input projection's weights for the bf16 matrix cores, one workgroup
// per output row n: W'[n][k] = W_in[n][k] g[k] (an fp32 product) split into
// three bf16 planes, hi = bf16(W'), mid = bf16(W' - hi), lo = W' - hi - mid
// (each difference exact in fp32; lo has at most 8 significant bits, so
// hi + mid + lo = W' exactly), planes [3][dm][dim]; c[n] = sum_k W'[n][k]
// and dv[n] = sum_k W_in[n][k] b[k], added in fp64 and rounded once.
__device__ inline uint16_t bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__global__ __launch_bounds__(256) void prep_input_kernel(const float* w, const float* g, const float* b, int dim,
                                                         int dm, uint16_t* planes, float* c, float* dv) {
  __shared__ double red[2][4];
  const int n = blockIdx.x;
  double sc = 0.0, sd = 0.0;
  for (int k = threadIdx.x; k < dim; k += 256) {
    const float wv = w[(size_t)n * dim + k];
    const float x = wv * g[k];
    const uint16_t hi = bf16_rne(x);
    const float r1 = x - __uint_as_float((uint32_t)hi << 16);
    const uint16_t mid = bf16_rne(r1);
    const float r2 = r1 - __uint_as_float((uint32_t)mid << 16);
    planes[(size_t)n * dim + k] = hi;
    planes[((size_t)dm + n) * dim + k] = mid;
    planes[((size_t)2 * dm + n) * dim + k] = bf16_rne(r2);  // exact: r2 has at most 8 significant bits
    sc += (double)x;
    sd += (double)wv * (double)b[k];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sc += __shfl_xor(sc, o, 64);
    sd += __shfl_xor(sd, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = sc;
    red[1][threadIdx.x >> 6] = sd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c[n] = (float)(((red[0][0] + red[0][1]) + red[0][2]) + red[0][3]);
    dv[n] = (float)(((red[1][0] + red[1][1]) + red[1][2]) + red[1][3]);
  }
}

// One attention step of one (trace row, head), head_dim 64, four waves.
// The trace's step index t is its count of earlier steps.  Wave 0 (one
// element per lane) applies RoPE - (x_i, x_{i+32}) rotated by
// t * 10000^(-i/32) - and appends the rotated key and the value at t in the
// trace's cache: keys in groups of four steps, [ks / 4][64][4] (ks =
// max_steps rounded up to a multiple of 4), so one group's 64 dimensions
// are 1 KB of consecutive memory and four consecutive steps of a dimension
// one 16-byte load; values [ks][64].  Scores of the earlier steps: thread
// (j4, eq) takes steps 4 j4 .. 4 j4 + 3 over dimensions eq + 8 e, e < 8
// (the eight threads of a group read 128 consecutive bytes per load, so a
// wave's load touches eight whole lines; the first group's loads are issued
// before wave 0 has finished the append, which they do not depend on), and the eight
// parts are added by shuffles; steps past t - 1 in the last group are
// masked (their slots are read but never used).  The softmax is taken over
// steps 0..t; for the values, thread (g, c) takes dimensions 4 c .. 4 c + 3
// of steps j = g mod 16, and the sixteen groups' sums and step t's own term
// (its key and value in wave 0's registers) are added.
__device__ inline float block_max(float v, float* red) {
  v = wave_max(v);
  __syncthreads();  // red[] is free
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__global__ __launch_bounds__(256) void seq_attn_kernel(SeqDev S, int layer, const float* qkv, float* o, int n) {
  extern __shared__ __attribute__((aligned(16))) float lds[];  // p[ks], q[64], partial outputs [4][64], red[4]
  const int ks = seq_kstride(S.max_steps);
  float* p = lds;
  float* qs = p + ks;
  float* op = qs + 64;
  float* red = op + 4 * 64;
  const int row = blockIdx.x / S.n_heads, h = blockIdx.x % S.n_heads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (row >= n) return;  // uniform over the workgroup
  const int tr = S.ids[row];
  const int t = S.lens[tr];
  if (t >= S.max_steps) {  // the host bounds step counts; keep the cache in bounds regardless
    if (tid == 0) atomicOr(S.err, 1);
    return;
  }
  const int d = S.d_model;
  float* kq = S.cache + (((size_t)tr * S.n_layers + layer) * S.n_heads + h) * seq_region_floats(S.max_steps);
  float* vc = kq + (size_t)64 * ks;
  const int eq = tid & 7, jq = tid >> 3;
  // the first group of earlier steps' keys, before the append (disjoint slots)
  float4 kv[8];
  if (4 * jq < t) {
    const float* kr = kq + (size_t)jq * 256 + 4 * eq;
#pragma unroll
    for (int e = 0; e < 8; ++e) kv[e] = ld_stream4(kr + 32 * e);
  }
  float v = 0.f, st = 0.f;
  if (wave == 0) {
    const float* src = qkv + (size_t)row * 3 * d + h * 64;
    const float q = src[lane], k = src[d + lane];
    v = src[2 * d + lane];
    const int i = lane & 31;
    const float theta = exp2f(-(float)i * (13.287712379549449f / 32.f));  // 10000^(-i/32)
    float sn, cs;
    sincosf((float)t * theta, &sn, &cs);
    const float qp = __shfl_xor(q, 32, 64), kp = __shfl_xor(k, 32, 64);
    const float qr = lane < 32 ? q * cs - qp * sn : qp * sn + q * cs;
    const float kr = lane < 32 ? k * cs - kp * sn : kp * sn + k * cs;
    kq[(size_t)(t >> 2) * 256 + 4 * lane + (t & 3)] = kr;
    vc[(size_t)t * 64 + lane] = v;
    qs[lane] = qr;
    st = wave_sum(qr * kr) * 0.125f;  // scale 1 / sqrt(64)
  }
  __syncthreads();  // qs[] is visible
  float mx = -INFINITY;
  for (int j0 = 4 * jq; j0 < t; j0 += 128) {  // 32 groups of four steps per pass
    if (j0 != 4 * jq) {
      const float* kr = kq + (size_t)(j0 >> 2) * 256 + 4 * eq;
#pragma unroll
      for (int e = 0; e < 8; ++e) kv[e] = ld_stream4(kr + 32 * e);
    }
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float qe = qs[eq + 8 * e];
      a.x = fmaf(qe, kv[e].x, a.x);
      a.y = fmaf(qe, kv[e].y, a.y);
      a.z = fmaf(qe, kv[e].z, a.z);
      a.w = fmaf(qe, kv[e].w, a.w);
    }
#pragma unroll
    for (int m = 1; m <= 4; m <<= 1) {
      a.x += __shfl_xor(a.x, m, 64);
      a.y += __shfl_xor(a.y, m, 64);
      a.z += __shfl_xor(a.z, m, 64);
      a.w += __shfl_xor(a.w, m, 64);
    }
    a.x = j0 < t ? a.x * 0.125f : -INFINITY;
    a.y = j0 + 1 < t ? a.y * 0.125f : -INFINITY;
    a.z = j0 + 2 < t ? a.z * 0.125f : -INFINITY;
    a.w = j0 + 3 < t ? a.w * 0.125f : -INFINITY;
    if (eq == 0) *reinterpret_cast<float4*>(p + j0) = a;
    mx = fmaxf(mx, fmaxf(fmaxf(a.x, a.y), fmaxf(a.z, a.w)));
  }
  // the values of this thread's steps j0 + g + 16 i (i < 8) of a 128-step
  // chunk, all in flight at once; the first chunk's across the softmax
  const int c = tid & 15, g = tid >> 4;
  float4 vv[8];
  auto load_v = [&](int j0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = j0 + g + 16 * i;
      vv[i] = j < t ? *reinterpret_cast<const float4*>(vc + (size_t)j * 64 + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  load_v(0);
  if (wave == 0 && lane == 0) mx = fmaxf(mx, st);
  mx = block_max(mx, red);  // also publishes p[]
  float sum = 0.f;
  for (int j = tid; j < t; j += 256) {
    const float e = expf(p[j] - mx);
    p[j] = e;
    sum += e;
  }
  sum = block_sum(sum, red);  // also publishes the exponentials
  // steps g + 32 k into a0, g + 16 + 32 k into a1 (independent sums)
  float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = a0;
  for (int j0 = 0; j0 < t; j0 += 128) {
    if (j0) load_v(j0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = j0 + g + 16 * i;
      const float pj = j < t ? p[j] : 0.f;
      float4& a = (i & 1) ? a1 : a0;
      a.x = fmaf(pj, vv[i].x, a.x), a.y = fmaf(pj, vv[i].y, a.y), a.z = fmaf(pj, vv[i].z, a.z),
      a.w = fmaf(pj, vv[i].w, a.w);
    }
  }
  a0.x += a1.x, a0.y += a1.y, a0.z += a1.z, a0.w += a1.w;
#pragma unroll
  for (int m = 16; m <= 32; m <<= 1) {  // the wave's four step groups
    a0.x += __shfl_xor(a0.x, m, 64);
    a0.y += __shfl_xor(a0.y, m, 64);
    a0.z += __shfl_xor(a0.z, m, 64);
    a0.w += __shfl_xor(a0.w, m, 64);
  }
  if (lane < 16) *reinterpret_cast<float4*>(op + wave * 64 + 4 * lane) = a0;
  __syncthreads();
  if (wave == 0) {
    const float pt = expf(st - mx);
    const float total = sum + pt;
    o[(size_t)row * d + h * 64 + lane] =
        (((op[lane] + op[64 + lane]) + op[128 + lane]) + op[192 + lane] + pt * v) / total;
  }
}

// Branch: the child's history is the parent's (its whole cache region and
// its step count).  One workgroup per (pair, slice of the region).
__global__ __launch_bounds__(256) void seq_fork_kernel(SeqDev S, const int32_t* pairs, size_t region_f4) {
  const int child = pairs[2 * blockIdx.y], parent = pairs[2 * blockIdx.y + 1];
  const float4* src = reinterpret_cast<const float4*>(S.cache) + (size_t)parent * region_f4;
  float4* dst = reinterpret_cast<float4*>(S.cache) + (size_t)child * region_f4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < region_f4; i += (size_t)gridDim.x * 256)
    dst[i] = src[i];
  if (blockIdx.x == 0 && threadIdx.x == 0) S.lens[child] = S.lens[parent];
}

__global__ void seq_set_len_kernel(SeqDev S, const int32_t* ids, int n, int value) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) S.lens[ids[i]] = value;
}

}  // namespace

// The tile of a product, by its estimated time.  A tile's workgroups fill the
// chip per_cu to a compute unit (its LDS), in rounds; a round takes
// round + K (k_round + k_wg m) us with m workgroups to a unit, and the launch
// `once` more.  The four numbers of a tile are fitted to its times on MI355X
// over 16 to 1000 rows and d_model 128 to 1536 with d_ff 1 to 4 times that
// (mean error 2-4%); the tile picked from them takes 2% more than the best one
// on average, 13% at worst.  Picked by workgroup counts from fewer tiles, as
// before, a layer's four products took (us, before -> now; the kernels of one
// shared tile with split sums and reduces, which came before those, in
// brackets): 512 rows, d_model 256, d_ff 768 25.6 -> 25.5 (33.8); 400 rows, 384,
// 1152 54.2 -> 40.3 (44.2); 300 rows, 512, 2048 81.7 -> 60.5 (66.3); 1000 rows,
// 1024, 2048 438 -> 256 (250); 24 rows, 128, 256 16.1 -> 14.7 (21.3).
struct TileCost {
  int rows, cols, per_cu;
  float once, round, k_round, k_wg;
};
static float tile_us(const TileCost& t, int M, int N, int K) {
  constexpr int kCU = 256;
  const long n = (long)((M + t.rows - 1) / t.rows) * (N / t.cols);
  const long whole = n / (kCU * t.per_cu), rest = n % (kCU * t.per_cu);
  const float rounds = (float)(whole + (rest > 0)), wgs = (float)(whole * t.per_cu + (rest + kCU - 1) / kCU);
  return t.once + t.round * rounds + K * (t.k_round * rounds + t.k_wg * wgs);
}
template <int N_TILES>
static int pick_tile(const TileCost (&tiles)[N_TILES], int M, int N, int K) {
  int best = 0;
  float us = 0.f;
  for (int i = 0; i < N_TILES; ++i) {
    if (N % tiles[i].cols) continue;
    const float t = tile_us(tiles[i], M, N, K);
    if (us == 0.f || t < us) best = i, us = t;
  }
  return best;
}

template <int MB, int NB, int NW, bool LN, int EPI>
static hipError_t launch_gemm(const float* A, const float* W, float* C, int M, int N, int K, const float* lg,
                              const float* lb, float2* stats, hipStream_t s) {
  hipLaunchKernelGGL((gemm_kernel<MB, NB, NW, LN, EPI>), dim3(N / (16 * NB), (M + 16 * MB - 1) / (16 * MB)),
                     dim3(64 * NW), 0, s, A, W, C, M, N, K, lg, lb, stats);
  return hipGetLastError();
}
template <int TM, int EPI>
static hipError_t launch_wide(const float* A, const float* W, float* C, int M, int N, int K, const float* lg,
                              const float* lb, const float2* stats, hipStream_t s) {
  hipLaunchKernelGGL((gemm_wide_kernel<TM, EPI>), dim3(N / 64, (M + TM - 1) / TM), dim3(256), 0, s, A, W, C, M, N, K,
                     lg, lb, stats);
  return hipGetLastError();
}

// N a multiple of 64.
template <int EPI>
static hipError_t gemm_ln(const float* A, const float* W, float* C, int M, int N, int K, const float* lg,
                          const float* lb, const float2* stats, hipStream_t s) {
  static const TileCost tiles[] = {{16, 32, 3, 2.39f, 0.05f, 0.0022f, 0.0056f},
                                   {16, 64, 2, 2.07f, 0.41f, 0.0020f, 0.0085f},
                                   {32, 96, 1, 0.52f, 2.26f, 0.0231f, 0.f},
                                   {32, 64, 3, 3.10f, 0.f, 0.0063f, 0.0105f},
                                   {64, 64, 2, 3.53f, 0.f, 0.0087f, 0.0192f}};
  float2* st = const_cast<float2*>(stats);
  switch (pick_tile(tiles, M, N, K)) {
    case 0: return launch_gemm<1, 2, 4, true, EPI>(A, W, C, M, N, K, lg, lb, st, s);
    case 1: return launch_gemm<1, 4, 4, true, EPI>(A, W, C, M, N, K, lg, lb, st, s);
    case 2: return launch_gemm<2, 6, 4, true, EPI>(A, W, C, M, N, K, lg, lb, st, s);
    case 3: return launch_wide<32, EPI>(A, W, C, M, N, K, lg, lb, stats, s);
    default: return launch_wide<64, EPI>(A, W, C, M, N, K, lg, lb, stats, s);
  }
}

hipError_t seq_gemm_ln(const float* A, const float* W, float* C, int M, int N, int K, const float* lg, const float* lb,
                       const float2* stats, hipStream_t s) {
  return gemm_ln<kEpiNone>(A, W, C, M, N, K, lg, lb, stats, s);
}

hipError_t seq_gemm_ln_swiglu(const float* A, const float* W, float* C, int M, int N, int K, const float* lg,
                              const float* lb, const float2* stats, hipStream_t s) {
  return gemm_ln<kEpiSwiGLU>(A, W, C, M, N, K, lg, lb, stats, s);
}

hipError_t seq_gemm_add(const float* A, const float* W, float* C, int M, int N, int K, float2* stats, hipStream_t s) {
  static const TileCost tiles[] = {{16, 16, 2, 1.88f, 1.69f, 0.f, 0.0018f},
                                   {16, 32, 3, 1.72f, 1.16f, 0.f, 0.0035f},
                                   {32, 32, 2, 1.64f, 1.23f, 0.f, 0.0057f},
                                   {32, 48, 2, 3.21f, 1.80f, 0.0005f, 0.0071f},
                                   {32, 64, 1, 0.f, 3.95f, 0.0098f, 0.f}};
  switch (pick_tile(tiles, M, N, K)) {
    case 0: return launch_gemm<1, 1, 8, false, kEpiAdd>(A, W, C, M, N, K, nullptr, nullptr, stats, s);
    case 1: return launch_gemm<1, 2, 4, false, kEpiAdd>(A, W, C, M, N, K, nullptr, nullptr, stats, s);
    case 2: return launch_gemm<2, 2, 4, false, kEpiAdd>(A, W, C, M, N, K, nullptr, nullptr, stats, s);
    case 3: return launch_gemm<2, 3, 4, false, kEpiAdd>(A, W, C, M, N, K, nullptr, nullptr, stats, s);
    default: return launch_gemm<2, 4, 4, false, kEpiAdd>(A, W, C, M, N, K, nullptr, nullptr, stats, s);
  }
}

hipError_t seq_prep_input(const float* w_in, const float* ln_g, const float* ln_b, int dim, int dm, uint16_t* planes,
                          float* c, float* dv, hipStream_t s) {
  hipLaunchKernelGGL(prep_input_kernel, dim3(dm), dim3(256), 0, s, w_in, ln_g, ln_b, dim, dm, planes, c, dv);
  return hipGetLastError();
}

hipError_t seq_proj_in(const uint16_t* h, const uint16_t* planes, int n, int dim, int dm, int splits, float* part,
                       hipStream_t s) {
  const int tiles = (n + kInTile - 1) / kInTile * (dm / kInTile);
  hipLaunchKernelGGL(proj_in_kernel, dim3(tiles * splits), dim3(64 * kInWaves), 0, s, h, planes, n, dim, dm, splits, part);
  return hipGetLastError();
}

hipError_t seq_reduce_in(const uint16_t* h, int dim, const float* part, int splits, const float* c, const float* dv,
                         float* x, int d, float2* stats, int n, hipStream_t s) {
  hipLaunchKernelGGL(reduce_in_kernel, dim3(n), dim3(256), 0, s, h, dim, part, splits, c, dv, x, d, stats, n);
  return hipGetLastError();
}

hipError_t seq_head(const float* x, int d, const SeqDev& S, float* scores, int n, hipStream_t s) {
  hipLaunchKernelGGL(head_kernel, dim3((n + 3) / 4), dim3(256), 0, s, x, d, S, scores, n);
  return hipGetLastError();
}

hipError_t seq_attention(const SeqDev& S, int layer, const float* qkv, float* o, int n, hipStream_t s) {
  const size_t lds = sizeof(float) * ((size_t)seq_kstride(S.max_steps) + 64 + 4 * 64 + 4);
  hipLaunchKernelGGL(seq_attn_kernel, dim3(n * S.n_heads), dim3(256), lds, s, S, layer, qkv, o, n);
  return hipGetLastError();
}

hipError_t seq_fork(const SeqDev& S, const int32_t* pairs, int n, hipStream_t s) {
  const size_t region_f4 = (size_t)S.n_layers * S.n_heads * seq_region_floats(S.max_steps) / 4;
  const unsigned slices = (unsigned)std::max<size_t>(1, std::min<size_t>(64, (region_f4 + 255) / 256));
  hipLaunchKernelGGL(seq_fork_kernel, dim3(slices, n), dim3(256), 0, s, S, pairs, region_f4);
  return hipGetLastError();
}

hipError_t seq_set_len(const SeqDev& S, const int32_t* ids, int n, int value, hipStream_t s) {
  hipLaunchKernelGGL(seq_set_len_kernel, dim3((n + 255) / 256), dim3(256), 0, s, S, ids, n, value);
  return hipGetLastError();
}

}  // namespace gambit
