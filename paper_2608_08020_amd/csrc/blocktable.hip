// Block-table kernels: pool initialisation, lowest-free-first allocation,
// KV writes, prune (free) and branch (fork).
//
// Branch spawns a child from its parent's prefix by sharing the parent's KV
// blocks (Alg. 1 notation; Sec. 4.1 Case 2), so a fork copies block ids and
// bumps refcounts; only a partially filled last block is copied, because
// both traces keep appending into their own copy of it.  Prune frees the
// blocks nobody else references (Sec. 4.1 Case 2).
#include "kernels.h"

namespace gambit {
namespace {

constexpr int kAllocThreads = 1024;

__device__ inline int cdiv16(int x) { return (x + kBlock - 1) / kBlock; }

__global__ void pool_init_kernel(DevPool P) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t ntab = (size_t)P.max_traces * P.max_blocks;
  for (size_t i = i0; i < ntab; i += stride) P.table[i] = -1;
  for (size_t i = i0; i < (size_t)P.max_traces; i += stride) {
    P.seq_len[i] = 0;
    P.sbar[i] = 0.f;
    P.nscore[i] = 0;
    P.gen[i] = 0;
    P.ghost[i] = 0;
  }
  for (size_t i = i0; i < (size_t)P.num_blocks; i += stride) P.refcount[i] = 0;
  for (size_t w = i0; w < (size_t)P.nwords; w += stride) {
    const int lo = (int)w * 32;
    const int valid = min(32, P.num_blocks - lo);
    P.freebits[w] = valid >= 32 ? 0xFFFFFFFFu : ((1u << valid) - 1u);
  }
  if (i0 == 0) *P.err = 0;
}

// Exclusive scan of one int per thread across the workgroup (kAllocThreads
// = 16 waves): a shuffle scan inside each wave, then the wave totals.
__device__ int wg_exclusive_scan(int v, int* total) {
  __shared__ int wsum[kAllocThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int x = __shfl_up(incl, off);
    if (lane >= off) incl += x;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kAllocThreads / 64; ++k) {
    const int s = wsum[k];
    before += k < w ? s : 0;
    all += s;
  }
  __syncthreads();  // wsum may be reused
  *total = all;
  return before + incl - v;
}

// One workgroup.  Request i extends trace req_trace[i] by its token count;
// the blocks it needs are the next lowest free ids, in request order and
// ascending logical index.  Bound by its chain of round trips and by what one
// workgroup can issue, so:
//  * the free bitmap is read once, kScanAhead coalesced passes of one word per
//    thread in flight, only as far as the lowest `total` free blocks reach;
//    the ids go to alloc_list, and the pool is touched only when they suffice;
//  * what was taken is every free block up to the last one listed, so the
//    bitmap is cleared by word, without a second scan;
//  * the blocks are entered one per thread, by their place in the list (its
//    request found by bisection over the requests' first places in LDS), so a
//    long request costs no more than many short ones.
// One trace of 8191 tokens: 75 us with a thread per request, 7.4 us so; 512
// traces of 2560 tokens 342 -> 89 us; 32 branches' tails 28.6 -> 8.6 us.
constexpr int kScanAhead = 4;

__global__ __launch_bounds__(kAllocThreads) void alloc_kernel(DevPool P, const int32_t* req_trace,
                                                             const int32_t* req_ntok, int32_t uniform,
                                                             int32_t m, float new_scale, int32_t generated) {
  // per thread: its requests' first place in the list; its first request's
  // trace, first new block and count of them
  __shared__ int first_s[kAllocThreads], trace_s[kAllocThreads], j0_s[kAllocThreads], cnt_s[kAllocThreads];
  __shared__ int last_s;
  const int t = threadIdx.x;
  const int rpt = (m + kAllocThreads - 1) / kAllocThreads;
  const int r0 = min(m, t * rpt), r1 = min(m, r0 + rpt);
  // request i: its trace, the first block it adds and how many
  auto request = [&](int i, int& tr, int& j0) {
    tr = req_trace[i];
    const int L = P.seq_len[tr];
    const int nt = uniform >= 0 ? uniform : req_ntok[i];
    j0 = cdiv16(L);
    return cdiv16(L + nt) - j0;
  };
  int need = 0, tr0 = 0, j00 = 0, cnt0 = 0;
  for (int i = r0; i < r1; ++i) {
    int tr, j0;
    const int c = request(i, tr, j0);
    if (i == r0) tr0 = tr, j00 = j0, cnt0 = c;
    need += c;
  }
  int total = 0;
  first_s[t] = wg_exclusive_scan(need, &total);
  trace_s[t] = tr0, j0_s[t] = j00, cnt_s[t] = cnt0;
  if (total > 0) {  // uniform across the workgroup
    int found = 0;
    for (int w0 = 0; w0 < P.nwords && found < total; w0 += kScanAhead * kAllocThreads) {
      uint32_t words[kScanAhead];
#pragma unroll
      for (int x = 0; x < kScanAhead; ++x) {
        const int w = w0 + x * kAllocThreads + t;
        words[x] = w < P.nwords ? P.freebits[w] : 0u;
      }
#pragma unroll
      for (int x = 0; x < kScanAhead; ++x) {
        if (found >= total) break;
        uint32_t bits = words[x];
        int n = 0;
        int rank = found + wg_exclusive_scan(__popc(bits), &n);
        for (; bits && rank < total; ++rank) {
          const int b = (w0 + x * kAllocThreads + t) * 32 + __ffs(bits) - 1;
          bits &= bits - 1;
          P.alloc_list[rank] = b;
          if (rank == total - 1) last_s = b;
        }
        found += n;
      }
    }
    if (found < total) {  // the host mirror rules this out; leave the pool untouched
      if (t == 0) atomicOr(P.err, kErrAllocShort);
      return;
    }
    __syncthreads();  // alloc_list, last_s and the requests are complete
    const int last = last_s;
    for (int w = t; w <= last >> 5; w += kAllocThreads)
      P.freebits[w] = w < last >> 5 ? 0u : P.freebits[w] & ~((2u << (last & 31)) - 1u);
    for (int k = t; k < total; k += kAllocThreads) {
      const int b = P.alloc_list[k];
      int x = 0;  // the thread whose requests place k belongs to: the last one that starts at or before it
#pragma unroll
      for (int s = kAllocThreads / 2; s > 0; s >>= 1)
        if (first_s[x + s] <= k) x += s;
      int off = k - first_s[x], tr = trace_s[x], j0 = j0_s[x], c = cnt_s[x];
      for (int i = x * rpt; off >= c;) {
        off -= c;
        c = request(++i, tr, j0);
      }
      P.table[(size_t)tr * P.max_blocks + j0 + off] = b;
      P.refcount[b] = 1;
      if (P.kv_scale)
        for (int l = 0; l < P.num_layers; ++l) {
          float* sc = P.kv_scale + 2 * ((size_t)l * P.num_blocks + b);
          sc[0] = new_scale;
          sc[1] = new_scale;
        }
    }
    __syncthreads();  // the lengths are still the requests' old ones until here
  }
  for (int i = r0; i < r1; ++i) {
    const int tr = req_trace[i];
    const int nt = uniform >= 0 ? uniform : req_ntok[i];
    P.seq_len[tr] += nt;
    if (generated) P.gen[tr] += nt;
  }
}

// 16 bytes of the caller's K or V (no alignment beyond the element's is asked
// of those buffers).
struct __attribute__((packed, aligned(1))) Raw16 {
  uint32_t w[4];
};
__device__ inline uint4 ld_raw16(const uint8_t* p) {
  const Raw16 r = *reinterpret_cast<const Raw16*>(p);
  return make_uint4(r.w[0], r.w[1], r.w[2], r.w[3]);
}

// A run of tokens into one layer's caches: one workgroup per (block, KV head,
// layer), one thread per 16-byte chunk of a tile (ES = bytes per element, 128
// ES threads).  Bound by HBM.  Both tiles are read in whole token rows (256
// or 128 bytes) and turned in LDS, so that every store is 16 bytes of a tile
// written in order: K into its d-chunks at token row k_phys(row), V into
// [d][token].  V's rows are padded by 8 bytes in LDS: the two token halves
// that a wave gathers fall in different banks; K's chunks by 16.  A block that
// the run covers in part keeps its other tokens: K's chunks are whole tokens,
// a V chunk that is not whole is stored by element.
//   k, v: [layers][n][Hkv][128]; started scales: [layers][started][2]
template <int ES>
__global__ __launch_bounds__(128 * ES) void write_kernel(DevPool P0, int32_t trace, int32_t pos0, int32_t n,
                                                         const uint8_t* k, const uint8_t* v,
                                                         const float* started_scales, int32_t started) {
  constexpr int kRow = kHeadDim * ES, kChunks = kRow / 16, kPer = 16 / ES;  // bytes and chunks a token, elements a chunk
  constexpr int kVRow = kRow + 8, kKCol = kBlock * 16 + 16;
  __shared__ __attribute__((aligned(16))) uint8_t klds[kChunks * kKCol], vlds[kBlock * kVRow];
  const int head = blockIdx.x % P0.Hkv, l = blockIdx.y, t = threadIdx.x;
  const int j = pos0 / kBlock + (int)(blockIdx.x / P0.Hkv);  // logical block
  const DevPool P = P0.layer(l);
  const int r0 = max(pos0 - j * kBlock, 0), r1 = min(pos0 + n - j * kBlock, kBlock);  // its rows in the run
  const int blk = P.table[(size_t)trace * P.max_blocks + j];
  {
    const int row = t / kChunks, c = t % kChunks;
    // rows outside the run re-read one inside it (never stored)
    const int tok = j * kBlock + min(max(row, r0), r1 - 1) - pos0;
    const size_t src = (((size_t)l * n + tok) * P.Hkv + head) * kRow + c * 16;
    const uint4 kk = ld_raw16(k + src), vv = ld_raw16(v + src);
    *reinterpret_cast<uint4*>(klds + c * kKCol + k_phys(row) * 16) = kk;
    uint2* vd = reinterpret_cast<uint2*>(vlds + row * kVRow + c * 16);
    vd[0] = make_uint2(vv.x, vv.y);
    vd[1] = make_uint2(vv.z, vv.w);
  }
  if ((unsigned)blk >= (unsigned)P.num_blocks) {  // uniform over the workgroup
    if (t == 0) atomicOr(P.err, kErrBadBlock);
    return;
  }
  __syncthreads();
  const size_t tile = ((size_t)blk * P.Hkv + head) * kBlock * kRow;
  const int krow = k_phys(t % kBlock);  // k_phys is its own inverse
  if (krow >= r0 && krow < r1)
    *reinterpret_cast<uint4*>(P.k_cache + tile + t * 16) =
        *reinterpret_cast<const uint4*>(klds + (t / kBlock) * kKCol + (t % kBlock) * 16);
  const int d = t / ES, f = (t % ES) * kPer;  // the chunk's tokens: f .. f + kPer - 1 of element d
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const uint8_t* src = vlds + (f + e) * kVRow + d * ES;
    const uint32_t x = ES == 2 ? *reinterpret_cast<const uint16_t*>(src) : *src;
    w[e * ES / 4] |= x << (8 * (e * ES % 4));
  }
  uint8_t* dst = P.v_cache + tile + t * 16;
  if (f >= r0 && f + kPer <= r1) {
    *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
  } else {
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (f + e < r0 || f + e >= r1) continue;
      const uint32_t x = w[e * ES / 4] >> (8 * (e * ES % 4));
      if (ES == 2)
        reinterpret_cast<uint16_t*>(dst)[e] = (uint16_t)x;
      else
        dst[e] = (uint8_t)x;
    }
  }
  if (started_scales && t == 0 && head == 0 && r0 == 0) {
    const int k2 = l * started + j - (pos0 + kBlock - 1) / kBlock;
    P.kv_scale[2 * blk] = started_scales[2 * k2];
    P.kv_scale[2 * blk + 1] = started_scales[2 * k2 + 1];
  }
}

// Blocks of a row that a thread of the prune and branch kernels has in flight:
// a row's entry, its refcount and its free bit are a chain of round trips, so
// 256 threads take 1024 blocks (16384 tokens) through one such chain.
constexpr int kRowAhead = 4;

// Prune (or evict): one workgroup per trace.  A row may be empty (a ghost
// leaving the tree view).
__global__ __launch_bounds__(256) void free_kernel(DevPool P, const int32_t* ids, int32_t mode) {
  const int tr = ids[blockIdx.x];
  const int nb = cdiv16(P.seq_len[tr]);
  int32_t* row = P.table + (size_t)tr * P.max_blocks;
  for (int j0 = threadIdx.x; j0 < nb; j0 += kRowAhead * blockDim.x) {
    int b[kRowAhead], old[kRowAhead];
#pragma unroll
    for (int x = 0; x < kRowAhead; ++x) {
      const int j = j0 + x * blockDim.x;
      b[x] = j < nb ? row[j] : -1;
    }
#pragma unroll
    for (int x = 0; x < kRowAhead; ++x) {
      const bool in = (unsigned)b[x] < (unsigned)P.num_blocks;
      old[x] = in ? atomicSub(&P.refcount[b[x]], 1) : 0;
      if (j0 + x * (int)blockDim.x < nb) {
        row[j0 + x * blockDim.x] = -1;
        if (!in) atomicOr(P.err, kErrBadBlock);
      }
    }
#pragma unroll
    for (int x = 0; x < kRowAhead; ++x) {
      if ((unsigned)b[x] >= (unsigned)P.num_blocks) continue;
      if (old[x] == 1) atomicOr(&P.freebits[b[x] >> 5], 1u << (b[x] & 31));
      if (old[x] < 1) atomicOr(P.err, kErrRefUnderflow);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    P.seq_len[tr] = 0;
    P.gen[tr] = 0;
    if (mode == kFreeEvict) {
      P.ghost[tr] = 1;  // keeps its score and its place in the tree view
    } else {
      P.ghost[tr] = 0;
      P.sbar[tr] = 0.f;
      P.nscore[tr] = 0;
    }
  }
}

// Branch, part 1: the child row takes the parent's full blocks (refcount + 1)
// and the child length is set to the full-block prefix; the partial tail is
// requested from the allocator (req_ntok = parent length mod 16).
__global__ __launch_bounds__(256) void fork_share_kernel(DevPool P, const int32_t* pairs, int32_t* req_trace,
                                  int32_t* req_ntok) {
  const int child = pairs[2 * blockIdx.x], parent = pairs[2 * blockIdx.x + 1];
  const int L = P.seq_len[parent];
  const int full = L / kBlock;
  const int32_t* prow = P.table + (size_t)parent * P.max_blocks;
  int32_t* crow = P.table + (size_t)child * P.max_blocks;
  for (int j0 = threadIdx.x; j0 < full; j0 += kRowAhead * blockDim.x) {
    int b[kRowAhead];
#pragma unroll
    for (int x = 0; x < kRowAhead; ++x) b[x] = prow[min(j0 + x * (int)blockDim.x, full - 1)];
#pragma unroll
    for (int x = 0; x < kRowAhead; ++x) {
      const int j = j0 + x * blockDim.x;
      if (j >= full) break;
      crow[j] = b[x];
      if ((unsigned)b[x] < (unsigned)P.num_blocks)
        atomicAdd(&P.refcount[b[x]], 1);
      else
        atomicOr(P.err, kErrBadBlock);
    }
  }
  if (threadIdx.x == 0) {
    P.seq_len[child] = full * kBlock;
    req_trace[blockIdx.x] = child;
    req_ntok[blockIdx.x] = L % kBlock;
    // the child's trace is the parent's prefix: it inherits the parent's
    // thought scores, and has generated nothing of its own yet
    P.sbar[child] = P.sbar[parent];
    P.nscore[child] = P.nscore[parent];
    P.gen[child] = 0;
    P.ghost[child] = 0;
  }
}

// Branch, part 2: copy the partial tail block (whole tiles, the slots past the
// tail are never read unmasked) and its fp8 scales into the child's new block;
// one workgroup per (pair, layer, KV head), one 16-byte chunk of K and of V per
// thread, so a small branch is one round trip.
__global__ __launch_bounds__(256) void fork_tail_kernel(DevPool P0, const int32_t* pairs) {
  const DevPool P = P0.layer(blockIdx.y);
  const int child = pairs[2 * blockIdx.x], parent = pairs[2 * blockIdx.x + 1];
  const int L = P.seq_len[parent];
  if (L % kBlock == 0) return;
  const int j = L / kBlock;
  const int src = P.table[(size_t)parent * P.max_blocks + j];
  const int dst = P.table[(size_t)child * P.max_blocks + j];
  if ((unsigned)src >= (unsigned)P.num_blocks || (unsigned)dst >= (unsigned)P.num_blocks) {
    if (threadIdx.x == 0) atomicOr(P.err, kErrBadBlock);
    return;
  }
  const size_t chunks = (size_t)kBlock * kHeadDim * P.esize / 16;  // of a tile: the workgroup's size
  const size_t s = ((size_t)src * P.Hkv + blockIdx.z) * chunks + threadIdx.x;
  const size_t d = ((size_t)dst * P.Hkv + blockIdx.z) * chunks + threadIdx.x;
  uint4 *kc = reinterpret_cast<uint4*>(P.k_cache), *vc = reinterpret_cast<uint4*>(P.v_cache);
  const uint4 kk = kc[s], vv = vc[s];
  kc[d] = kk;
  vc[d] = vv;
  if (P.kv_scale && threadIdx.x == 0 && blockIdx.z == 0) {
    P.kv_scale[2 * dst] = P.kv_scale[2 * src];
    P.kv_scale[2 * dst + 1] = P.kv_scale[2 * src + 1];
  }
}

}  // namespace

hipError_t launch_pool_init(const DevPool& P, hipStream_t s) {
  hipLaunchKernelGGL(pool_init_kernel, dim3(1024), dim3(256), 0, s, P);
  return hipGetLastError();
}

hipError_t launch_alloc(const DevPool& P, const int32_t* req_trace, const int32_t* req_ntok,
                        int32_t uniform_ntok, int32_t m, float new_scale, bool generated, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(alloc_kernel, dim3(1), dim3(kAllocThreads), 0, s, P, req_trace, req_ntok,
                     uniform_ntok, m, new_scale, (int32_t)generated);
  return hipGetLastError();
}

hipError_t launch_write(const DevPool& P, int32_t trace, int32_t pos0, int32_t n, const void* k,
                        const void* v, const float* started_scales, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int first = (pos0 + kBlock - 1) / kBlock, last = (pos0 + n - 1) / kBlock;
  const int started = last >= first ? last - first + 1 : 0;
  const dim3 grid((unsigned)(last - pos0 / kBlock + 1) * P.Hkv, P.num_layers);
  const auto *ks = static_cast<const uint8_t*>(k), *vs = static_cast<const uint8_t*>(v);
  if (P.esize == 2)
    hipLaunchKernelGGL(write_kernel<2>, grid, dim3(256), 0, s, P, trace, pos0, n, ks, vs, started_scales, started);
  else
    hipLaunchKernelGGL(write_kernel<1>, grid, dim3(128), 0, s, P, trace, pos0, n, ks, vs, started_scales, started);
  return hipGetLastError();
}

hipError_t launch_free(const DevPool& P, const int32_t* ids, int32_t n, int32_t mode, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(free_kernel, dim3(n), dim3(256), 0, s, P, ids, mode);
  return hipGetLastError();
}

hipError_t launch_fork(const DevPool& P, const int32_t* pairs, int32_t n, int32_t* req_trace,
                       int32_t* req_ntok, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fork_share_kernel, dim3(n), dim3(256), 0, s, P, pairs, req_trace, req_ntok);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_alloc(P, req_trace, req_ntok, -1, n, 1.0f, false, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fork_tail_kernel, dim3(n, P.num_layers, P.Hkv), dim3(128 * P.esize), 0, s, P, pairs);
  return hipGetLastError();
}

}  // namespace gambit
