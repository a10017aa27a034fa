// HIP kernels (gfx950) of the cluster-adaptive IVF-PQ search.
//
// Stage map (paper Sec. 2.1 and Sec. 4.1):
//   k_sqnorm / k_coarse  CL distances on FP32 MFMA (16x16x4) with norm epilogue
//   k_topn*              CL selection: nprobe smallest by (distance, list id)
//   k_pairs              RC on the operand grid, PPM features and the fixed-point
//                        RBF regressor -> LUT width per (query, probed list)
//   k_qhist/qscan/qscatter  work queue: pairs grouped by (lane class, list)
//   k_scan<...>          persistent: LC on BF16 MFMA (exact on the grid),
//                        per-pair quantisation, packed-lane DC scan, pruning
//                        against the query's running threshold (TSM forwarding)
//   k_merge              TS: per-query top-k by (distance, id)
#include "build_kernels.h"
#include "scan_kernels.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

namespace amp {

// ------------------------------------------------------------------ front
// The first launch of a search: the per-search resets of the workspace (fills
// by kernel, not memsets: a captured search graph holds no memset node), the
// per-query sizes handed over in device memory, and one pass over the query
// rows that widens BF16 rows, takes their squared norms and puts them on the
// operand grid, as far as the search needs each.  (Separate launches took 5 us
// each, 30 us of a 4096 x 768 BF16 batch in all: 12 us now.)
struct FrontArgs {
  uint32_t* cnt;     // bucket counters -> 0
  size_t ncnt;
  uint32_t* counters;  // unit counters -> 0
  size_t ncounters;
  uint32_t* flags;   // [4] -> 0
  uint64_t* work;    // [4] -> 0
  uint64_t* tau;     // [nq] -> no bound
  uint32_t* ccount;  // [nq] -> 0
  int32_t* ipmask;   // [nq] -> 0, or null (with the table reductions below)
  int32_t* ipspan;   // [nq] -> 0
  int64_t* iplsum;   // [nq] -> 0
  const int32_t* kin;   // device sizes, or null: each k into [1, kmax] and
  const int32_t* npin;  // nprobe into [1, npmax] (flag 32 if one was outside)
  int32_t* kout;
  int32_t* npout;
  int kmax, npmax;
  const float* q;        // FP32 rows, or
  const uint16_t* qb;    // BF16 rows, widened (exact) into qw
  float* qw;
  float* qn;             // [nq] squared norms, or null
  int16_t* qi;           // [nq][d] rows on the grid, or null
  int rows;              // 1: any of qw, qn, qi is wanted
  int nq, d, grid_e, grid_kind;
};
__device__ __forceinline__ void clamp_sizes(const FrontArgs& a, int i) {
  const int kv = a.kin[i], nv = a.npin[i];
  const int kc = kv < 1 ? 1 : (kv > a.kmax ? a.kmax : kv);
  const int nc = nv < 1 ? 1 : (nv > a.npmax ? a.npmax : nv);
  if (kc != kv || nc != nv) atomicOr(&a.flags[0], 32u);
  a.kout[i] = kc;
  a.npout[i] = nc;
}
// queries whose sizes workgroup 0 clamps itself (it has reset the flags they
// may raise); more of them take a launch of their own
constexpr int kFrontSizes = 8192;
__global__ __launch_bounds__(256) void k_front(FrontArgs a) {
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, st = (size_t)gridDim.x * blockDim.x;
  if (i0 < 4) {
    a.flags[i0] = 0;
    a.work[i0] = 0;
  }
  if (blockIdx.x == 0 && a.kin && a.nq <= kFrontSizes) {
    __threadfence();  // the flags are zero before any thread raises one
    __syncthreads();
#pragma unroll 4
    for (int i = threadIdx.x; i < a.nq; i += 256) clamp_sizes(a, i);
  }
  for (size_t i = i0; i < a.ncnt; i += st) a.cnt[i] = 0;
  for (size_t i = i0; i < a.ncounters; i += st) a.counters[i] = 0;
  for (size_t i = i0; i < (size_t)a.nq; i += st) {
    a.tau[i] = ~0ull;
    a.ccount[i] = 0;
    if (a.ipmask) {
      a.ipmask[i] = 0;
      a.ipspan[i] = 0;
      a.iplsum[i] = 0;
    }
  }
  if (!a.rows) return;
  const int lane = threadIdx.x & 63;
  for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < a.nq; r += (int64_t)gridDim.x * 4) {
    const size_t o = (size_t)r * a.d;
    float s = 0.f;  // lane-strided partial sums, then a butterfly: k_sqnorm's order
    for (int t = lane; t < a.d; t += 64) {
      const float x = a.qb ? __uint_as_float((uint32_t)a.qb[o + t] << 16) : a.q[o + t];
      if (a.qb) a.qw[o + t] = x;
      if (a.qi) a.qi[o + t] = (int16_t)grid_val(x, a.grid_e, a.grid_kind);
      s = fmaf(x, x, s);
    }
    if (a.qn) {
      for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
      if (lane == 0) a.qn[r] = s;
    }
  }
}
__global__ void k_sizes(FrontArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.nq) clamp_sizes(a, i);
}

// status word of a search from its error flags (the host-mode mapping):
// 16 / 8 internal errors, 32 a clamped size, 4 unit table and 2 candidate
// overflow
__global__ void k_status(const int32_t* __restrict__ flags, int32_t* __restrict__ out) {
  if (threadIdx.x != 0) return;
  const int32_t f = flags[0];
  int32_t s = AMP_OK;
  if (f & (16 | 8)) s = AMP_EDEVICE;
  else if (f & 32) s = AMP_EINVAL;
  else if (f) s = AMP_EOVERFLOW;
  *out = s;
}

// ------------------------------------------------------------------ CL
// squared norm of each row, FP32: one wave per row, lane-strided partial sums
// combined by a butterfly (a fixed order for a given d)
__global__ void k_sqnorm(const float* __restrict__ X, int rows, int d, float* __restrict__ out) {
  const int r = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= rows) return;
  const float* x = X + (size_t)r * d;
  float s = 0.f;
  for (int t = lane; t < d; t += 64) s = fmaf(x[t], x[t], s);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) out[r] = s;
}

// D[q][c] = (|q|^2 + |c|^2) - 2 q.c (L2) or -q.c (IP).  64x64 tile per
// workgroup, each wave a 32x32 quarter of 2x2 MFMA 16x16x4 FP32 tiles; K in
// chunks of KC staged through LDS, the next chunk's loads issued before the
// current chunk's products (16-byte loads when d is a multiple of 4 and the
// rows 16-byte aligned).  The products run in k order whatever the chunk, so
// the sums do not depend on it.
constexpr int CL_T = 64, CL_K = 32;
template <int KC, bool VEC>
__global__ __launch_bounds__(256) void k_coarse(const float* __restrict__ Q, const float* __restrict__ C,
                                                const float* __restrict__ qn, const float* __restrict__ cn,
                                                float* __restrict__ D, int nq, int nlist, int d, int metric) {
  __shared__ float Qs[CL_T][KC + 1];
  __shared__ float Cs[CL_T][KC + 1];
  const int q0 = blockIdx.y * CL_T, c0 = blockIdx.x * CL_T;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  constexpr int NV = CL_T * KC / 4 / 256;  // 16-byte loads per thread and tile
  float4 qa[NV], ca[NV];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int f = tid + 256 * u, r = f / (KC / 4), gk = k0 + 4 * (f % (KC / 4));
      if (VEC) {
        qa[u] = (q0 + r < nq && gk < d) ? *reinterpret_cast<const float4*>(Q + (size_t)(q0 + r) * d + gk)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
        ca[u] = (c0 + r < nlist && gk < d) ? *reinterpret_cast<const float4*>(C + (size_t)(c0 + r) * d + gk)
                                           : make_float4(0.f, 0.f, 0.f, 0.f);
      } else {
        float* qv = &qa[u].x;
        float* cv = &ca[u].x;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          qv[e] = (q0 + r < nq && gk + e < d) ? Q[(size_t)(q0 + r) * d + gk + e] : 0.f;
          cv[e] = (c0 + r < nlist && gk + e < d) ? C[(size_t)(c0 + r) * d + gk + e] : 0.f;
        }
      }
    }
  };
  f4 acc[2][2];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  load(0);
  for (int k0 = 0; k0 < d; k0 += KC) {
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int f = tid + 256 * u, r = f / (KC / 4), kk = 4 * (f % (KC / 4));
      Qs[r][kk] = qa[u].x; Qs[r][kk + 1] = qa[u].y; Qs[r][kk + 2] = qa[u].z; Qs[r][kk + 3] = qa[u].w;
      Cs[r][kk] = ca[u].x; Cs[r][kk + 1] = ca[u].y; Cs[r][kk + 2] = ca[u].z; Cs[r][kk + 3] = ca[u].w;
    }
    __syncthreads();
    if (k0 + KC < d) load(k0 + KC);
#pragma unroll
    for (int kk = 0; kk < KC; kk += 4) {
      float a0 = Qs[wr + (lane & 15)][kk + (lane >> 4)];
      float a1 = Qs[wr + 16 + (lane & 15)][kk + (lane >> 4)];
      float b0 = Cs[wc + (lane & 15)][kk + (lane >> 4)];
      float b1 = Cs[wc + 16 + (lane & 15)][kk + (lane >> 4)];
      acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
    }
    __syncthreads();
  }
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j)
      for (int r = 0; r < 4; ++r) {
        int qi = q0 + wr + 16 * i + 4 * (lane >> 4) + r;
        int ci = c0 + wc + 16 * j + (lane & 15);
        if (qi < nq && ci < nlist) {
          float dot = acc[i][j][r];
          D[(size_t)qi * nlist + ci] = metric == AMP_L2 ? (qn[qi] + cn[ci]) - 2.f * dot : -dot;
        }
      }
}

// CL under L1: D = sum_t |q_t - c_t| (no dense product to put on MFMA):
// 64 x 64 (query, centroid) tile per workgroup staged through LDS, each
// thread 16 sums
__global__ __launch_bounds__(256) void k_coarse_l1(const float* __restrict__ Q, const float* __restrict__ C,
                                                   float* __restrict__ D, int nq, int nlist, int d) {
  __shared__ float Qs[CL_T][CL_K + 1];
  __shared__ float Cs[CL_T][CL_K + 1];
  const int q0 = blockIdx.y * CL_T, c0 = blockIdx.x * CL_T;
  const int tid = threadIdx.x, tq = tid >> 4, tc = tid & 15;
  float acc[4][4];
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < d; k0 += CL_K) {
    for (int i = tid; i < CL_T * CL_K; i += 256) {
      const int r = i / CL_K, kk = i % CL_K, gk = k0 + kk;
      Qs[r][kk] = (q0 + r < nq && gk < d) ? Q[(size_t)(q0 + r) * d + gk] : 0.f;
      Cs[r][kk] = (c0 + r < nlist && gk < d) ? C[(size_t)(c0 + r) * d + gk] : 0.f;
    }
    __syncthreads();
    for (int kk = 0; kk < CL_K; ++kk)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += fabsf(Qs[tq + 16 * i][kk] - Cs[tc + 16 * j][kk]);
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      const int qi = q0 + tq + 16 * i, ci = c0 + tc + 16 * j;
      if (qi < nq && ci < nlist) D[(size_t)qi * nlist + ci] = acc[i][j];
    }
}

// grid codebook as int16 [M][256][8] (zero-padded), for the L1 LUT build
__global__ void k_prep_cbi(const float* __restrict__ cb, int M, int dsub, int grid_e, int grid_kind,
                           int16_t* __restrict__ cbi) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M * kKsub * 8) return;
  const int t = i & 7, e = i >> 3;
  cbi[i] = t < dsub ? (int16_t)grid_val(cb[(size_t)e * dsub + t], grid_e, grid_kind) : (int16_t)0;
}

// ------------------------------------------------------------------ index build
// squared norms of n rows of dd floats with leading dimension ld (a wave per row)
__global__ void k_sqnorm_ld(const float* __restrict__ X, int64_t n, int dd, int ld, float* __restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= n) return;
  float s = 0.f;
  for (int t = lane; t < dd; t += 64) {
    const float v = X[r * ld + t];
    s = fmaf(v, v, s);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) out[r] = s;
}

// nearest of k centroids (squared L2 in FP32, ties to the lower index) for n
// rows of dd floats (leading dimension ld) and its distance.  64 rows per
// workgroup; centroids in tiles of 64 on FP32 MFMA 16x16x4 (the coarse
// distance kernel's tiling); each tile's distances go through LDS and the
// row's thread keeps the running minimum.
__global__ __launch_bounds__(256) void k_assign(const float* __restrict__ X, const float* __restrict__ xn,
                                                int64_t n, int dd, int ld, const float* __restrict__ C,
                                                const float* __restrict__ cn, int k, int32_t* __restrict__ out_a,
                                                float* __restrict__ out_d) {
  __shared__ float Xs[CL_T][CL_K + 1];
  __shared__ float Cs[CL_T][CL_K + 1];
  __shared__ float Ds[CL_T][CL_T + 1];
  const int64_t r0 = (int64_t)blockIdx.x * CL_T;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  float best = 3.4e38f;
  int besti = 0;
  for (int c0 = 0; c0 < k; c0 += CL_T) {
    f4 acc[2][2];
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < dd; k0 += CL_K) {
      for (int i = tid; i < CL_T * CL_K; i += 256) {
        const int r = i / CL_K, kk = i % CL_K, gk = k0 + kk;
        Xs[r][kk] = (r0 + r < n && gk < dd) ? X[(r0 + r) * ld + gk] : 0.f;
        Cs[r][kk] = (c0 + r < k && gk < dd) ? C[(size_t)(c0 + r) * dd + gk] : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < CL_K; kk += 4) {
        const float a0 = Xs[wr + (lane & 15)][kk + (lane >> 4)];
        const float a1 = Xs[wr + 16 + (lane & 15)][kk + (lane >> 4)];
        const float b0 = Cs[wc + (lane & 15)][kk + (lane >> 4)];
        const float b1 = Cs[wc + 16 + (lane & 15)][kk + (lane >> 4)];
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
      }
      __syncthreads();
    }
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j)
        for (int q = 0; q < 4; ++q) {
          const int rr = wr + 16 * i + 4 * (lane >> 4) + q, cc = wc + 16 * j + (lane & 15);
          Ds[rr][cc] = c0 + cc < k ? cn[c0 + cc] - 2.f * acc[i][j][q] : 3.4e38f;
        }
    __syncthreads();
    if (tid < CL_T)
      for (int c = 0; c < CL_T && c0 + c < k; ++c) {
        const float v = Ds[tid][c];
        if (v < best) {
          best = v;
          besti = c0 + c;
        }
      }
    __syncthreads();
  }
  if (tid < CL_T && r0 + tid < n) {
    out_a[r0 + tid] = besti;
    if (out_d) out_d[r0 + tid] = best + xn[r0 + tid];
  }
}

// residual rows x - c_a of a chunk
__global__ void k_residual(const float* __restrict__ X, const int32_t* __restrict__ a, const float* __restrict__ C,
                           int64_t n, int d, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * d) return;
  const int64_t r = i / d;
  const int t = (int)(i - r * d);
  out[i] = X[i] - C[(size_t)a[r] * d + t];
}

// ------------------------------------------------------------------ sorting
// ascending bitonic sort of n (power of two) 64-bit keys in LDS by the block
__device__ void block_bitonic_u64(uint64_t* keys, int n) {
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < (n >> 1); i += blockDim.x) {
        int pos = 2 * i - (i & (stride - 1));
        int oth = pos + stride;
        bool asc = (pos & size) == 0;
        uint64_t a = keys[pos], b = keys[oth];
        if ((a > b) == asc) {
          keys[pos] = b;
          keys[oth] = a;
        }
      }
      __syncthreads();
    }
  }
}

// the kk-th smallest (1-based, kk <= n) of n 64-bit keys in LDS, by radix
// select: passes over 8-bit digits, most significant first, each
// counting the digits of the keys that share the digits chosen so far and
// choosing the digit whose count range holds the remaining rank.  hist: 256
// counters in LDS; sel: two words in LDS.  Every thread of the block returns
// the key.
__device__ uint64_t block_select_u64(const uint64_t* keys, int n, int kk, uint32_t* hist, uint32_t* sel) {
  const int tid = threadIdx.x, lane = tid & 63;
  // the digits above the highest bit where the smallest and largest keys
  // differ are common to every key: the passes start below them
  uint64_t lo = ~0ull, hi = 0;
  for (int i = tid; i < n; i += blockDim.x) {
    const uint64_t k = keys[i];
    lo = k < lo ? k : lo;
    hi = k > hi ? k : hi;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  uint64_t* mm = reinterpret_cast<uint64_t*>(hist);  // two words a wave (at most 16 waves)
  if (lane == 0) {
    mm[2 * (tid >> 6)] = lo;
    mm[2 * (tid >> 6) + 1] = hi;
  }
  __syncthreads();
  lo = mm[0];
  hi = mm[1];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
    lo = mm[2 * w] < lo ? mm[2 * w] : lo;
    hi = mm[2 * w + 1] > hi ? mm[2 * w + 1] : hi;
  }
  __syncthreads();  // hist is cleared by the first pass
  if (lo == hi) return lo;
  const int top = (63 - __builtin_clzll(lo ^ hi)) & ~7;
  uint64_t mask = top >= 56 ? 0ull : ~((1ull << (top + 8)) - 1);
  uint64_t prefix = lo & mask;
  uint32_t rank = (uint32_t)kk;
  for (int shift = top; shift >= 0; shift -= 8) {
    for (int i = tid; i < 256; i += blockDim.x) hist[i] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += blockDim.x) {
      const uint64_t k = keys[i];
      if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255], 1u);
    }
    __syncthreads();
    if (tid < 64) {
      // four bins a lane, inclusive scan over the wave
      const uint32_t h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
      const uint32_t own = h0 + h1 + h2 + h3;
      uint32_t inc = own;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(inc, o);
        if (lane >= o) inc += v;
      }
      const uint32_t below = inc - own;
      if (below < rank && rank <= inc) {
        uint32_t c = below, dg = 4 * lane;
        if (c + h0 < rank) {
          c += h0;
          ++dg;
          if (c + h1 < rank) {
            c += h1;
            ++dg;
            if (c + h2 < rank) {
              c += h2;
              ++dg;
            }
          }
        }
        sel[0] = dg;
        sel[1] = c;
      }
    }
    __syncthreads();
    prefix |= (uint64_t)sel[0] << shift;
    mask |= 255ull << shift;
    rank -= sel[1];
    __syncthreads();  // sel and hist are rewritten by the next pass
  }
  return prefix;
}

// same with a secondary signed 64-bit tie-breaker
__device__ void block_bitonic_u64_i64(uint64_t* keys, int64_t* vals, int n) {
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < (n >> 1); i += blockDim.x) {
        int pos = 2 * i - (i & (stride - 1));
        int oth = pos + stride;
        bool asc = (pos & size) == 0;
        uint64_t a = keys[pos], b = keys[oth];
        int64_t va = vals[pos], vb = vals[oth];
        bool gt = (a > b) || (a == b && va > vb);
        if (gt == asc) {
          keys[pos] = b;
          keys[oth] = a;
          vals[pos] = vb;
          vals[oth] = va;
        }
      }
      __syncthreads();
    }
  }
}

// OR of the wave's 64 values, on every lane
__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
  auto step = [&](auto ctrl) {
    x |= (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, decltype(ctrl)::value, 0xF, 0xF, false);
  };
  step(std::integral_constant<int, 0x111>{});  // within rows of sixteen: 1, 2, 4, 8 to the right
  step(std::integral_constant<int, 0x112>{});
  step(std::integral_constant<int, 0x114>{});
  step(std::integral_constant<int, 0x118>{});
  step(std::integral_constant<int, 0x142>{});  // a row's last lane to the next row
  step(std::integral_constant<int, 0x143>{});  // lane 31 to the upper half
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// CL selection: the nprobe smallest (distance, list) of each query.
// General case: a workgroup per query, bitonic sort of all nlist keys in LDS.
__global__ __launch_bounds__(256) void k_topn(const float* __restrict__ D, int nlist, int np2,
                                              const int32_t* __restrict__ npq, int npconst, int npmax,
                                              int32_t* __restrict__ probes) {
  extern __shared__ uint64_t keys[];
  const int q = blockIdx.x;
  const float* row = D + (size_t)q * nlist;
  for (int i = threadIdx.x; i < np2; i += blockDim.x)
    keys[i] = i < nlist ? (((uint64_t)fkey(row[i]) << 32) | (uint32_t)i) : ~0ull;
  __syncthreads();
  block_bitonic_u64(keys, np2);
  const int np = npq ? npq[q] : npconst;
  for (int r = threadIdx.x; r < npmax; r += blockDim.x)
    probes[(size_t)q * npmax + r] = r < np ? (int32_t)(keys[r] & 0xFFFFFFFFu) : -1;
}

// nlist <= 256 * PER (larger rows or nprobe > 64): a workgroup per query
// holds the row in registers (key j * 256 + thread).  The nprobe-th smallest
// order key x is found bit by bit, from the highest bit in which the row's keys
// differ to the first candidate with exactly nprobe keys below it (distances of
// like size share their exponents, and the candidates separate long before the
// last bit; always 32 steps before: 1 query over 1024 lists 7.6 -> 5.4 us, 4096
// over 4096 79 -> 60, 4096 over 2048 42 -> 39; a wave per query, 10000 over 1024,
// 37 -> 30): the count of keys below a candidate is
// the sum over the four waves of ballot bit counts, exchanged through LDS
// (two alternating slots: one barrier per bit).  The keys up to x, with
// their list ids, are gathered in LDS (any order); up to 512 of them each
// take the output row of their rank by (key, list id) among them, more are
// padded to a power of two and sorted.  The first nprobe are the probes,
// the same as a sort of the whole row.
template <int PER>
__global__ __launch_bounds__(256) void k_topn_wg(const float* __restrict__ D, int nlist,
                                                 const int32_t* __restrict__ npq, int npconst, int npmax,
                                                 int32_t* __restrict__ probes) {
  extern __shared__ uint64_t sel[];  // room for the next power of two >= nlist
  __shared__ int s_cnt[2][4];
  __shared__ uint32_t s_diff[4];
  __shared__ int s_n;
  const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float* row = D + (size_t)q * nlist;
  uint32_t key[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = j * 256 + tid;
    key[j] = i < nlist ? fkey(row[i]) : 0xFFFFFFFFu;
  }
  const int k = npq ? npq[q] : npconst;
  if (tid == 0) s_n = 0;
  const uint32_t ref = fkey(row[0]);
  uint32_t diff = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) diff |= j * 256 + tid < nlist ? key[j] ^ ref : 0u;
  diff = wave_or(diff);
  if (lane == 0) s_diff[wv] = diff;
  __syncthreads();
  diff = s_diff[0] | s_diff[1] | s_diff[2] | s_diff[3];
  // largest value with fewer than k keys below it: the k-th smallest; or, once
  // exactly k keys are below a candidate, the value before it
  uint32_t x = diff ? ref & ~((2u << (31 - __clz((int)diff))) - 1u) : ref;
  for (int bit = 31 - __clz((int)diff); bit >= 0; --bit) {
    const uint32_t t = x | (1u << bit);
    int c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) c += __popcll(__ballot(key[j] < t));
    if (lane == 0) s_cnt[bit & 1][wv] = c;
    __syncthreads();
    const int n = s_cnt[bit & 1][0] + s_cnt[bit & 1][1] + s_cnt[bit & 1][2] + s_cnt[bit & 1][3];
    if (n < k) x = t;
    else if (n == k) {  // (uniform over the workgroup)
      x = t - 1;
      break;
    }
  }
  // gather the keys <= x (at least k of them; ties at x all come along)
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = j * 256 + tid;
    const bool take = i < nlist && key[j] <= x;
    const uint64_t bal = __ballot(take);
    int base = 0;
    if (lane == 0 && bal) base = atomicAdd(&s_n, __popcll(bal));
    base = __shfl(base, 0);
    if (take) sel[base + __popcll(bal & ((1ull << lane) - 1))] = ((uint64_t)key[j] << 32) | (uint32_t)i;
  }
  __syncthreads();
  const int n = s_n;
  if (n <= 512) {  // uniform over the workgroup
    // (key, list id) are distinct: each selected key's output row is the
    // count of selected keys below it (no sort, no barrier)
    for (int t = tid; t < n; t += 256) {
      const uint64_t v = sel[t];
      int rank = 0;
      for (int j = 0; j < n; ++j) rank += sel[j] < v;
      if (rank < npmax) probes[(size_t)q * npmax + rank] = rank < k ? (int32_t)(v & 0xFFFFFFFFu) : -1;
    }
    for (int r = n + tid; r < npmax; r += 256) probes[(size_t)q * npmax + r] = -1;
    return;
  }
  int n2 = 1;
  while (n2 < n) n2 <<= 1;
  for (int i = n + tid; i < n2; i += 256) sel[i] = ~0ull;
  __syncthreads();
  for (int size = 2; size <= n2; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < (n2 >> 1); i += 256) {
        const int pos = 2 * i - (i & (stride - 1));
        const bool asc = (pos & size) == 0;
        const uint64_t u = sel[pos], v = sel[pos + stride];
        if ((u > v) == asc) {
          sel[pos] = v;
          sel[pos + stride] = u;
        }
      }
      __syncthreads();
    }
  for (int r = tid; r < npmax; r += 256)
    probes[(size_t)q * npmax + r] = r < k ? (int32_t)(sel[r] & 0xFFFFFFFFu) : -1;
}

// nlist <= 64 * PER and nprobe <= 64: one wave per query, no sort of the
// whole row.  Lane l holds keys l, l + 64, ...  The nprobe-th smallest
// order key is found bit by bit (count of keys below a candidate, summed
// over the wave); the keys below it, and the equal ones with the lowest list
// ids, are compacted and sorted by (key, list) across the lanes.
template <int PER>
__global__ __launch_bounds__(256) void k_topn_wave(const float* __restrict__ D, int nlist, int nq,
                                                   const int32_t* __restrict__ npq, int npconst, int npmax,
                                                   int32_t* __restrict__ probes) {
  __shared__ uint64_t s_sel[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int q = blockIdx.x * 4 + wv;
  const bool on = q < nq;  // no early return: the workgroup synchronises below
  uint32_t key[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = j * 64 + lane;
    key[j] = on && i < nlist ? fkey(D[(size_t)q * nlist + i]) : 0xFFFFFFFFu;
  }
  const int k = on ? (npq ? npq[q] : npconst) : 0;
  // wave-wide count of keys below t: one ballot per key slot and a bit
  // count of the mask (no cross-lane shuffles)
  auto count_below = [&](uint32_t t) {
    int c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) c += __popcll(__ballot(key[j] < t));
    return c;
  };
  const uint32_t ref = (uint32_t)__builtin_amdgcn_readfirstlane((int)key[0]);
  uint32_t diff = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) diff |= j * 64 + lane < nlist ? key[j] ^ ref : 0u;
  diff = wave_or(diff);
  // largest value with fewer than k keys below it: the k-th smallest; or, once
  // exactly k keys are below a candidate, the value before it
  uint32_t x = diff ? ref & ~((2u << (31 - __clz((int)diff))) - 1u) : ref;
  for (int bit = 31 - __clz((int)diff); bit >= 0; --bit) {
    const uint32_t t = x | (1u << bit);
    const int c = count_below(t);
    if (c < k) x = t;
    else if (c == k) {
      x = t - 1;
      break;
    }
  }
  int need_eq = k - count_below(x);  // keys equal to x to take, lowest list id first
  s_sel[wv][lane] = ~0ull;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {  // list ids ascend with (j, lane)
    const bool eq = key[j] == x;
    const uint64_t meq = __ballot(eq);
    const int eq_rank = __popcll(meq & ((1ull << lane) - 1));
    const bool sel = on && (key[j] < x || (eq && eq_rank < need_eq));
    need_eq -= __popcll(meq) < need_eq ? __popcll(meq) : need_eq;
    const uint64_t msel = __ballot(sel);
    if (sel) {
      const int pos = base + __popcll(msel & ((1ull << lane) - 1));
      s_sel[wv][pos] = ((uint64_t)key[j] << 32) | (uint32_t)(j * 64 + lane);
    }
    base += __popcll(msel);
  }
  __syncthreads();
  uint64_t v = s_sel[wv][lane];
  for (int kb = 2; kb <= 64; kb <<= 1)
    for (int jb = kb >> 1; jb > 0; jb >>= 1) {
      const uint64_t o = __shfl_xor(v, jb);
      const bool keep_min = ((lane & kb) == 0) == ((lane & jb) == 0);
      v = keep_min ? (o < v ? o : v) : (o > v ? o : v);
    }
  if (on && lane < npmax) probes[(size_t)q * npmax + lane] = lane < k ? (int32_t)(v & 0xFFFFFFFFu) : -1;
}

// ------------------------------------------------------------------ PPM
struct PairArgs {
  const float* Q;
  const float* C;
  const int16_t* qi16;    // inner product: queries and centroids on the grid (d' = |qi - ci|^2)
  const int16_t* ci16;
  const int64_t* dq2_in;  // d' of every pair where the base kernel has computed it (L2), or null
  int64_t* dot_out;       // adaptive inner product: qi.ci of every pair (read in the same pass), or null
  int32_t* ipmask;        // with dot_out: the widths each query's pairs use
  const int32_t* probes;
  const int32_t* radq;
  const int64_t* offsets;
  const uint8_t* xbits;
  uint8_t* pbits;
  int nq, d, npmax, grid_e, grid_kind, metric, policy, fixed_bits, lane_sel_M;
  int lg_npp;  // log2 of the pair slots per query (power of two >= npmax)
  int lg_T;    // log2 of the threads per pair (small batches: several share the work)
  uint32_t allowed;
  int64_t margin;
};

__device__ __forceinline__ int64_t mitchell_q8(int64_t x) {
  uint64_t y = (uint64_t)x + 1;
  int k = 63 - __clzll((long long)y);
  return 256 * (int64_t)k + (int64_t)((y << 8) >> k) - 256;
}

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int pick_bits(int64_t y, const int64_t* theta, uint32_t allowed, int64_t margin) {
  int last = 16;
  for (int b = 4; b <= 16; b += 4) {
    if (!(allowed & (1u << b))) continue;
    last = b;
    if (b == 16 || y + margin <= theta[b / 4 - 1]) return b;
  }
  return last;
}

// 256 threads per workgroup: 256 / (npp T) queries, npp (power of two >=
// npmax) pair slots per query, T threads per pair (T > 1 only for batches too
// small to fill the chip: the T threads split the residual norm and the
// support-vector sum, then combine them across their lanes)
__global__ __launch_bounds__(256) void k_pairs(PairArgs a, ModelArgs ma) {
  __shared__ unsigned long long s_best[256];
  __shared__ int64_t s_dq2[256];
  __shared__ int32_t s_dot[256];
  __shared__ int32_t s_wmask[256];  // widths of each query slot's pairs (with dot_out)
  __shared__ int32_t s_table[kTableN];
  const int lg = a.lg_npp, lt = a.lg_T, T = 1 << lt;
  const int t = threadIdx.x & (T - 1);
  const int slot = threadIdx.x >> (lg + lt), r = (threadIdx.x >> lt) & ((1 << lg) - 1);
  const int q = blockIdx.x * (256 >> (lg + lt)) + slot;
  const bool adaptive = a.policy == AMP_POLICY_ADAPTIVE;
  if (adaptive)
    for (int i = threadIdx.x; i < kTableN; i += blockDim.x) s_table[i] = ma.table[i];
  if ((threadIdx.x & ((1 << (lg + lt)) - 1)) == 0) {
    s_best[slot] = ~0ull;
    s_wmask[slot] = 0;
  }
  __syncthreads();
  const bool valid = q < a.nq && r < a.npmax;
  const int p = valid ? a.probes[(size_t)q * a.npmax + r] : -1;
  // d' = |grid residual|^2 of pair (qq, pp): the part of lane t of tn
  // (four coordinates per step, d % 4 == 0)
  // (inner product: also the part of qi.ci, into dot)
  auto dq2_part = [&](int qq, int pp, int t0, int tn, int& dot) -> int64_t {
    int64_t s2 = 0;
    const bool l2 = a.metric != AMP_IP;  // L2 and L1: d' of the grid residual
    if (!l2 && a.qi16) {
      // inner product: both sides already on the grid
      auto acc2 = [&](uint32_t x, uint32_t c) {
        const int x0 = (int)(int16_t)(x & 0xFFFFu), x1 = (int)(int16_t)(x >> 16);
        const int c0 = (int)(int16_t)(c & 0xFFFFu), c1 = (int)(int16_t)(c >> 16);
        const int v0 = x0 - c0, v1 = x1 - c1;
        s2 += (int64_t)(v0 * v0 + v1 * v1);
        dot += x0 * c0 + x1 * c1;
      };
      if ((a.d & 7) == 0) {
        // eight coordinates per 16-byte read (rows 16-byte aligned)
        const u32x4* xq = reinterpret_cast<const u32x4*>(a.qi16 + (size_t)qq * a.d);
        const u32x4* xc = reinterpret_cast<const u32x4*>(a.ci16 + (size_t)pp * a.d);
        for (int i = t0; i < (a.d >> 3); i += tn) {
          const u32x4 x = xq[i], c = xc[i];
          acc2(x[0], c[0]);
          acc2(x[1], c[1]);
          acc2(x[2], c[2]);
          acc2(x[3], c[3]);
        }
        return s2;
      }
      const u32x2* xq = reinterpret_cast<const u32x2*>(a.qi16 + (size_t)qq * a.d);
      const u32x2* xc = reinterpret_cast<const u32x2*>(a.ci16 + (size_t)pp * a.d);
      for (int i = t0; i < (a.d >> 2); i += tn) {
        const u32x2 x = xq[i], c = xc[i];
        const int x0 = (int)(int16_t)(x[0] & 0xFFFFu), x1 = (int)(int16_t)(x[0] >> 16);
        const int x2 = (int)(int16_t)(x[1] & 0xFFFFu), x3 = (int)(int16_t)(x[1] >> 16);
        const int c0 = (int)(int16_t)(c[0] & 0xFFFFu), c1 = (int)(int16_t)(c[0] >> 16);
        const int c2 = (int)(int16_t)(c[1] & 0xFFFFu), c3 = (int)(int16_t)(c[1] >> 16);
        const int v0 = x0 - c0, v1 = x1 - c1, v2 = x2 - c2, v3 = x3 - c3;
        s2 += (int64_t)(v0 * v0 + v1 * v1) + (int64_t)(v2 * v2 + v3 * v3);
        dot += x0 * c0 + x1 * c1 + x2 * c2 + x3 * c3;
      }
      return s2;
    }
    const float4* qv = reinterpret_cast<const float4*>(a.Q + (size_t)qq * a.d);
    const float4* cv = reinterpret_cast<const float4*>(a.C + (size_t)pp * a.d);
    for (int i = t0; i < (a.d >> 2); i += tn) {
      const float4 x = qv[i], c = cv[i];
      int v0, v1, v2, v3;
      if (l2) {
        v0 = grid_val(x.x - c.x, a.grid_e, a.grid_kind);
        v1 = grid_val(x.y - c.y, a.grid_e, a.grid_kind);
        v2 = grid_val(x.z - c.z, a.grid_e, a.grid_kind);
        v3 = grid_val(x.w - c.w, a.grid_e, a.grid_kind);
      } else {
        v0 = grid_val(x.x, a.grid_e, a.grid_kind) - grid_val(c.x, a.grid_e, a.grid_kind);
        v1 = grid_val(x.y, a.grid_e, a.grid_kind) - grid_val(c.y, a.grid_e, a.grid_kind);
        v2 = grid_val(x.z, a.grid_e, a.grid_kind) - grid_val(c.z, a.grid_e, a.grid_kind);
        v3 = grid_val(x.w, a.grid_e, a.grid_kind) - grid_val(c.w, a.grid_e, a.grid_kind);
      }
      s2 += (int64_t)(v0 * v0 + v1 * v1) + (int64_t)(v2 * v2 + v3 * v3);
    }
    return s2;
  };
  int64_t dq2 = 0;
  int dot = 0;  // (inner product with dot_out)
  if (adaptive && a.dq2_in) {
    if (p >= 0) dq2 = a.dq2_in[(size_t)q * a.npmax + r];  // the same on the T threads of the pair
  } else if (adaptive && T == 1) {
    // a thread per pair: the rows are read by sixteen lanes per pair, sixteen
    // pairs of the workgroup at a time (coalesced 128-byte segments), and the
    // norms handed over through LDS; the thread of a pair slot is its index
    const int l16 = threadIdx.x & 15, grp = threadIdx.x >> 4;
    for (int e0 = 0; e0 < 256; e0 += 16) {
      const int e = e0 + grp;
      const int qs = blockIdx.x * (256 >> lg) + (e >> lg), rs = e & ((1 << lg) - 1);
      const int pp = qs < a.nq && rs < a.npmax ? a.probes[(size_t)qs * a.npmax + rs] : -1;
      int dp = 0;
      int64_t s2 = pp >= 0 ? dq2_part(qs, pp, l16, 16, dp) : 0;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        s2 += __shfl_xor(s2, o, 16);
        dp += __shfl_xor(dp, o, 16);
      }
      if (l16 == 0) {
        s_dq2[e] = s2;
        s_dot[e] = dp;
      }
    }
    __syncthreads();
    dq2 = s_dq2[threadIdx.x];
    dot = s_dot[threadIdx.x];
  } else if (adaptive && p >= 0) {
    dq2 = dq2_part(q, p, t, T, dot);
  }
  // the T threads of a pair are adjacent lanes of one wave (T <= 64)
  if (T > 1 && !a.dq2_in)
    for (int o = 1; o < T; o <<= 1) {
      dq2 += __shfl_xor(dq2, o);
      dot += __shfl_xor(dot, o);
    }
  if (adaptive && p >= 0 && t == 0)
    atomicMin(&s_best[slot], (unsigned long long)((uint64_t)dq2 << 13 | (uint64_t)p));
  __syncthreads();
  if (valid) {
    uint8_t bits = 0;
    if (p >= 0) {
      if (a.policy == AMP_POLICY_FP32) {
        bits = 32;
      } else if (a.policy == AMP_POLICY_FIXED) {
        bits = (uint8_t)a.fixed_bits;
      } else if (a.policy == AMP_POLICY_EXPLICIT) {
        bits = a.xbits[(size_t)q * a.npmax + r];
      } else {
        const int c1 = (int)(s_best[slot] & 8191ull);
        int64_t x[5];
        x[0] = dq2;
        x[1] = a.radq[c1];
        x[2] = a.radq[p];
        x[3] = a.offsets[c1 + 1] - a.offsets[c1];
        x[4] = a.offsets[p + 1] - a.offsets[p];
        int32_t u[5];
        for (int f = 0; f < 5; ++f) {
          int64_t v = ((mitchell_q8(x[f]) - ma.feat_lo[f]) * ma.feat_mul[f]) >> 16;
          u[f] = (int32_t)(v < 0 ? 0 : (v > 1023 ? 1023 : v));
        }
        // integer sum: the split over threads and the order do not change the
        // result.  |u - sv|^2 = |u|^2 + |sv|^2 - 2 u.sv on 16-bit pair products
        // (u and sv lie in [0, 1023], sv checked when the model is set: exact,
        // below 2^23), four operations instead of ten; the table index is the
        // high word of one product with g_mul < 2^32, a full-rate 24-bit one
        // where g_mul < 2^24 (gamma up to 63).  (Bound by the VALU with a thread
        // per pair: 278k pairs x 1280 support vectors 169 -> 112 us; with several
        // threads per pair by the latency of a support vector's loads, six words
        // a vector one at a time before: 1726 pairs 52 -> 28 us.)
        const uint32_t gm = (uint32_t)ma.g_mul;
        const int un = u[0] * u[0] + u[1] * u[1] + u[2] * u[2] + u[3] * u[3] + u[4] * u[4];
        const s16x2 u01 = {(short)(-2 * u[0]), (short)(-2 * u[1])}, u23 = {(short)(-2 * u[2]), (short)(-2 * u[3])};
        const s16x2 u4 = {(short)(-2 * u[4]), 0};
        auto sum = [&](auto small_g) {
          auto term = [&](int w0, int w1, int w2, int w3, int beta) -> int64_t {
            int d2 = un + w3;
            d2 = __builtin_amdgcn_sdot2(u01, __builtin_bit_cast(s16x2, w0), d2, false);
            d2 = __builtin_amdgcn_sdot2(u23, __builtin_bit_cast(s16x2, w1), d2, false);
            d2 = __builtin_amdgcn_sdot2(u4, __builtin_bit_cast(s16x2, w2), d2, false);
            const uint32_t idx = decltype(small_g)::value ? __umulhi((uint32_t)d2 & 0xFFFFFFu, gm & 0xFFFFFFu)
                                                          : __umulhi((uint32_t)d2, gm);
            return (int64_t)beta * s_table[idx < (uint32_t)(kTableN - 1) ? idx : (uint32_t)(kTableN - 1)];
          };
          int64_t y = 0;
          int i = t;
          if (T == 1) {
            // a thread per pair: the support-vector index is the same across
            // the wave, so records come through scalar loads, two per load
            // (one word at a time, each load was waited for alone)
            const i32x16* rec = reinterpret_cast<const i32x16*>(ma.sv);
            for (; i + 3 < ma.n_sv; i += 4) {
              const i32x16 r0 = rec[i / 2], r1 = rec[i / 2 + 1];
              y += term(r0[0], r0[1], r0[2], r0[3], r0[4]);
              y += term(r0[8], r0[9], r0[10], r0[11], r0[12]);
              y += term(r1[0], r1[1], r1[2], r1[3], r1[4]);
              y += term(r1[8], r1[9], r1[10], r1[11], r1[12]);
            }
          } else {
            const int4* rec = reinterpret_cast<const int4*>(ma.sv);
            // eight records on the way per thread; past the end the last one
            // again, with weight zero
            constexpr int UN = 8;
            for (; i < ma.n_sv; i += UN * T) {
              int4 r[UN];
              int bt[UN];
#pragma unroll
              for (int k = 0; k < UN; ++k) {
                const int e = i + k * T < ma.n_sv ? i + k * T : ma.n_sv - 1;
                r[k] = rec[2 * e];
                bt[k] = ma.sv[kSvWords * e + 4];
              }
#pragma unroll
              for (int k = 0; k < UN; ++k)
                y += term(r[k].x, r[k].y, r[k].z, r[k].w, i + k * T < ma.n_sv ? bt[k] : 0);
            }
          }
          for (; i < ma.n_sv; i += T) {
            const int32_t* w = ma.sv + kSvWords * i;
            y += term(w[0], w[1], w[2], w[3], w[4]);
          }
          return y;
        };
        int64_t y = gm < (1u << 24) ? sum(std::true_type{}) : sum(std::false_type{});
        for (int o = 1; o < T; o <<= 1) y += __shfl_xor(y, o);
        bits = (uint8_t)pick_bits(ma.beta0 + y, ma.theta, a.allowed, a.margin);
      }
    }
    if (t == 0) a.pbits[(size_t)q * a.npmax + r] = bits;
    if (a.dot_out && p >= 0 && t == 0) {
      // the pair's list term for its base (k_ipq subtracts it from the sum
      // of the query's row minima) and its width in the query slot's mask
      a.dot_out[(size_t)q * a.npmax + r] = dot;
      atomicOr(&s_wmask[slot], 1 << ((bits >> 2) - 1));
    }
  }
  if (a.dot_out) {
    // one atomic per query for the widths its tables are needed at
    __syncthreads();
    if ((threadIdx.x & ((1 << (lg + lt)) - 1)) == 0 && q < a.nq && s_wmask[slot])
      atomicOr(&a.ipmask[q], s_wmask[slot]);
  }
}

// ------------------------------------------------------------------ queue
// Buckets are class-major.  Phase 1 holds the rank-0 pair of every query,
// phase 2 every active pair.  One atomic per pair on its (class, list)
// counter gives its rank inside the bucket; the scatter and the work-unit
// table are then written without atomics.  Counters are indexed by list id
// (the most-probed lists stay spread over memory channels), offsets and
// units by the list's position in the launch order lorder (largest first).
struct QueueArgs {
  const int32_t* probes;
  const uint8_t* pbits;
  const int32_t* kq;      // per-query k, or null (kconst)
  int kconst;
  const int64_t* offsets;
  const int32_t* lorder;  // bucket position -> list (largest list first)
  const int32_t* lpos;    // list -> bucket position
  int32_t* cnt;       // [2][kQSub][NB] by (sub-counter, class, list id)
  int32_t* rank;      // [2][nq*npmax]
  int64_t* pairoff;   // [2][NB+1] by (class, launch position)
  int64_t* unitoff;   // [2][NB+1] by (class, launch position)
  int32_t* sorted;    // [2][nq*npmax]
  int4* units;        // [2][max_units]: {list, first pair, pair count, chunk}
  int32_t* flags;
  int nq, npmax, nlist, M, ncls, wpr;
  int gran;               // quantiser granularity (lane classes of 4-bit pairs)
  int64_t chunk[2], max_units;  // list chunk of a work unit in phase 1, phase 2
  int ph0, ph1;           // queue phases built by this launch: [ph0, ph1) of {0 bound, 1 full scan}
  const int64_t* pbase;   // lower bound of every pair's estimates (integer: exact base; FP32 policy,
                          // inner product: the key of its in-order FP32 bound), or null: every pair
                          // joins phase 2
  int fkeys;              // pbase holds FP32 keys (FP32 policy)
  const uint64_t* tau;    // the queries' phase-1 bounds (with pbase)
  int all_offsets;        // k_queue_small: every bucket's offsets are wanted (statistics)
  uint64_t* work;         // phase-2 work counters (pairs dropped here count as skipped), or null
};

// a pair joins the full scan unless its lower bound already exceeds its
// query's phase-1 bound (then no vector of its list can reach the top-k)
__device__ __forceinline__ bool pair_live(const QueueArgs& a, size_t i) {
  if (!a.pbase) return true;
  const uint64_t key = a.fkeys ? (uint64_t)a.pbase[i] : ikey(a.pbase[i]);
  return key <= a.tau[i / a.npmax];
}

// pairs of a work unit: the LUT words of its class's rows times their fields
__device__ __forceinline__ int class_pairs(int cls, int wpr, bool fp32, int gran, int M) {
  return fp32 ? wpr : unit_pairs(lane_bits(cls, gran, M), wpr);
}

// sub-counter of a pair: the pairs of a much-probed list spread over kQSub
// counters (in different cache lines), so their atomics do not queue on one
__device__ __forceinline__ int pair_sub(size_t i) {
  return (int)(((uint32_t)i * 0x9E3779B1u) >> 28) & (kQSub - 1);
}

// the phase-1 bound of a query comes from its nearest probes: rank 0, and
// each further rank while the lists of the ranks before it hold fewer than k
// vectors (so that the bound covers k distinct vectors whenever the probed
// lists hold that many)
__device__ __forceinline__ bool in_phase1(const QueueArgs& a, size_t i) {
  const size_t q = i / a.npmax;
  const int r = (int)(i - q * a.npmax);
  if (r == 0) return true;
  const int kk = a.kq ? a.kq[q] : a.kconst;
  int64_t cum = 0;
  for (int j = 0; j < r; ++j) {
    const int p = a.probes[q * a.npmax + j];
    cum += a.offsets[p + 1] - a.offsets[p];
    if (cum >= kk) return false;
  }
  return true;
}

__global__ void k_qhist(QueueArgs a) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t n = (size_t)a.nq * a.npmax;
  if (i >= n) return;
  const int p = a.probes[i];
  if (p < 0) return;
  const int cls = pair_class(a.pbits[i], a.M, a.gran);
  const int NB = a.ncls * a.nlist;
  const size_t b = (size_t)pair_sub(i) * NB + cls * a.nlist + p;
  if (a.ph1 > 1) {
    if (pair_live(a, i)) a.rank[n + i] = atomicAdd(&a.cnt[(size_t)kQSub * NB + b], 1);
    else if (a.work) atomicAdd((unsigned long long*)&a.work[2], 1ull);
  }
  if (a.ph0 == 0 && in_phase1(a, i)) a.rank[i] = atomicAdd(&a.cnt[b], 1);
}

// per (phase, class, list) bucket: its pair total from the sub-counters
// (which become offsets inside the bucket) and its unit count, stored at the
// bucket's launch position (pairoff / unitoff hold counts until k_qscan)
__global__ void k_qtot(QueueArgs a, int fp32) {
  const int NB = a.ncls * a.nlist;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (a.ph1 - a.ph0) * NB) return;
  const int ph = a.ph0 + i / NB, b = i % NB, cls = b / a.nlist, p = b % a.nlist;
  int32_t* cnt = a.cnt + (size_t)ph * kQSub * NB;
  int x[kQSub];
#pragma unroll
  for (int u = 0; u < kQSub; ++u) x[u] = cnt[(size_t)u * NB + b];
  int c = 0;
#pragma unroll
  for (int u = 0; u < kQSub; ++u) {
    const int xu = x[u];
    x[u] = c;
    c += xu;
  }
#pragma unroll
  for (int u = 0; u < kQSub; ++u) cnt[(size_t)u * NB + b] = x[u];
  const int64_t n = a.offsets[p + 1] - a.offsets[p];
  const int64_t ck0 = a.chunk[0], ck = ph ? a.chunk[1] : ck0;
  const int64_t nch = (n + ck - 1) / ck;
  const int G = class_pairs(cls, a.wpr, fp32, a.gran, a.M);
  const int pos = cls * a.nlist + a.lpos[p];
  a.pairoff[(size_t)ph * (NB + 1) + pos] = c;
  a.unitoff[(size_t)ph * (NB + 1) + pos] = ((c + G - 1) / G) * nch;
}

// inclusive sum over the wave's lanes (row shifts, then row broadcasts: no LDS
// permutes, whose latency is most of a scan in a one-workgroup kernel)
__device__ __forceinline__ uint32_t wave_sum_scan(uint32_t v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
  return v;
}
// exclusive sums of two counts over a workgroup of up to 1024 threads; s_w:
// 16 pairs of words of LDS, free again on return
__device__ __forceinline__ uint2 block_exclusive2(uint32_t a, uint32_t b, uint2* s_w, uint2* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t ia = wave_sum_scan(a), ib = wave_sum_scan(b);
  if (threadIdx.x < 16) s_w[threadIdx.x] = make_uint2(0, 0);
  __syncthreads();
  if (lane == 63) s_w[wv] = make_uint2(ia, ib);
  __syncthreads();
  uint2 below = make_uint2(0, 0), all = make_uint2(0, 0);
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const uint2 t = s_w[w];
    if (w < wv) below = make_uint2(below.x + t.x, below.y + t.y);
    all = make_uint2(all.x + t.x, all.y + t.y);
  }
  __syncthreads();
  *total = all;
  return make_uint2(below.x + ia - a, below.y + ib - b);
}
// buckets of a thread's run (odd: the runs start in distinct LDS banks)
__host__ __device__ __forceinline__ int bucket_run(int NB, int threads) { return ((NB + threads - 1) / threads) | 1; }

// exclusive sum of a 64-bit count over a workgroup of 1024 threads; s_w: 16
// words of LDS of its own
__device__ __forceinline__ int64_t block_exclusive64(int64_t v, int64_t* s_w, int64_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int64_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t x = __shfl_up(inc, o);
    if (lane >= o) inc += x;
  }
  if (lane == 63) s_w[wv] = inc;
  __syncthreads();
  // (every wave scans the totals: sixteen lanes, no second barrier and, the
  // kernel's sixteen waves being one workgroup, few registers)
  int64_t t = s_w[lane & 15];
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    const int64_t x = __shfl_up(t, o, 16);
    if ((lane & 15) >= o) t += x;
  }
  *total = __shfl(t, 15);
  const int64_t below = __shfl(t, wv ? wv - 1 : 0);
  return (wv ? below : 0) + inc - v;
}

// k_qscan for up to kFewBuckets buckets, where a thread's run is at most 32
// bytes: its counts straight into registers, one barrier per scan (900, 1536,
// 3072 and 4095 buckets 5.4, 6.0, 7.5 and 9.1 us through LDS, 4.5, 4.6, 5.1 and
// 6.0 this way).  33 registers: beside another stream's persistent scan a CU has
// little room for a workgroup of sixteen waves (with 92 the kernel was as fast
// alone, but searches on three streams became 2 to 3 % slower).
constexpr int kFewPer = 4, kFewBuckets = kFewPer * 1024;
__global__ __launch_bounds__(1024) void k_qscan_few(QueueArgs a) {
  __shared__ int64_t s_w[2][16];
  const int NB = a.ncls * a.nlist, per = (NB + 1023) / 1024, b0 = threadIdx.x * per;
#pragma unroll 1
  for (int i = 2 * a.ph0; i < 2 * a.ph1; ++i) {  // pair and unit counts of each phase
    int64_t* arr = (i & 1 ? a.unitoff : a.pairoff) + (size_t)(i >> 1) * (NB + 1) + b0;
    int64_t c[kFewPer], sum = 0, total;
#pragma unroll
    for (int u = 0; u < kFewPer; ++u) c[u] = u < per && b0 + u < NB ? arr[u] : 0;
#pragma unroll
    for (int u = 0; u < kFewPer; ++u) sum += c[u];
    int64_t x = block_exclusive64(sum, s_w[i & 1], &total);
#pragma unroll
    for (int u = 0; u < kFewPer; ++u) {
      if (u < per && b0 + u < NB) arr[u] = x;
      x += c[u];
    }
    if (threadIdx.x == 0) arr[NB] = total;
  }
}

// exclusive scans of the pair and unit counts in launch order, one workgroup
// of 1024 threads: the counts come in coalesced and are scanned in LDS, each
// thread a contiguous run.  (Runs read straight from memory took a cache line
// per lane: 35 us for 12288 buckets, 13 this way.)  A bucket's units are held
// in 32 bits, saturated: beyond any unit table.
__global__ __launch_bounds__(1024) void k_qscan(QueueArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  uint32_t* v = reinterpret_cast<uint32_t*>(lds);  // [NB]
  __shared__ int64_t s_base[1024], s_w[16];
  const int NB = a.ncls * a.nlist, tid = threadIdx.x;
  const int per = bucket_run(NB, 1024), b0 = tid * per, b1 = b0 + per < NB ? b0 + per : NB;
  for (int ph = a.ph0; ph < a.ph1; ++ph)
    for (int t = 0; t < 2; ++t) {
      int64_t* arr = (t ? a.unitoff : a.pairoff) + (size_t)ph * (NB + 1);
#pragma unroll 4
      for (int b = tid; b < NB; b += 1024) {
        const int64_t c = arr[b];
        v[b] = c < 0xFFFFFFFFll ? (uint32_t)c : 0xFFFFFFFFu;
      }
      __syncthreads();
      int64_t sum = 0;
      for (int b = b0; b < b1; ++b) {
        const uint32_t c = v[b];
        v[b] = (uint32_t)sum;  // offset inside the run (a run that overflows it has overflowed any table)
        sum += c;
      }
      // 64-bit sums of the runs: wave scans, then the sixteen wave totals
      const int lane = tid & 63, wv = tid >> 6;
      int64_t inc = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int64_t x = __shfl_up(inc, o);
        if (lane >= o) inc += x;
      }
      if (lane == 63) s_w[wv] = inc;
      __syncthreads();
      int64_t below = 0, total = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        if (w < wv) below += s_w[w];
        total += s_w[w];
      }
      s_base[tid] = below + inc - sum;
      __syncthreads();
      for (int b = tid; b < NB; b += 1024) arr[b] = s_base[b / per] + v[b];
      if (tid == 0) arr[NB] = total;
      __syncthreads();  // the LDS is filled again
    }
}

__global__ void k_qscatter(QueueArgs a) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t n = (size_t)a.nq * a.npmax;
  if (i >= n) return;
  const int p = a.probes[i];
  if (p < 0) return;
  const int cls = pair_class(a.pbits[i], a.M, a.gran);
  const int b = cls * a.nlist + a.lpos[p];
  const int NB = a.ncls * a.nlist;
  const size_t bs = (size_t)pair_sub(i) * NB + cls * a.nlist + p;  // sub-counter offset
  if (a.ph1 > 1 && pair_live(a, i))
    a.sorted[n + a.pairoff[(NB + 1) + b] + a.cnt[(size_t)kQSub * NB + bs] + a.rank[n + i]] = (int32_t)i;
  if (a.ph0 == 0 && in_phase1(a, i)) a.sorted[a.pairoff[b] + a.cnt[bs] + a.rank[i]] = (int32_t)i;
}

// grid-stride over (phase, unit): find the unit's bucket by binary search of
// the unit offsets and write its descriptor
__global__ void k_qunits(QueueArgs a, int fp32) {
  const int NB = a.ncls * a.nlist;
  for (int ph = a.ph0; ph < a.ph1; ++ph) {
    const int64_t* po = a.pairoff + (size_t)ph * (NB + 1);
    const int64_t* uo = a.unitoff + (size_t)ph * (NB + 1);
    const int64_t total = uo[NB];
    if (total > a.max_units) {
      if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&a.flags[0], 4);
      continue;
    }
    int4* units = a.units + (size_t)ph * a.max_units;
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total;
         u += (int64_t)gridDim.x * blockDim.x) {
      int lo = 0, hi = NB;  // uo[lo] <= u < uo[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (uo[mid] <= u) lo = mid; else hi = mid;
      }
      const int b = lo, cls = b / a.nlist, p = a.lorder[b % a.nlist];
      const int64_t n = a.offsets[p + 1] - a.offsets[p];
      const int64_t ck0 = a.chunk[0], ck = ph ? a.chunk[1] : ck0;
      const int64_t nch = (n + ck - 1) / ck;
      const int G = class_pairs(cls, a.wpr, fp32, a.gran, a.M);
      const int64_t local = u - uo[b], grp = local / nch, ch = local % nch;
      const int64_t left = (po[b + 1] - po[b]) - grp * G;
      units[u] = make_int4(p, (int)(po[b] + grp * G), (int)(left < G ? left : G), (int)ch);
    }
  }
}

// The whole queue build of a small batch (at most kSmallQueue pairs) in one
// workgroup: U pairs per thread in registers, list lengths, bucket counts and
// offsets in LDS; the first pair of a unit writes it.  The five launches above
// are latency and launch gaps there (each 2 to 5 us for one query, 42 us per
// search for the two builds; 11 us this way).  What remains is two dependent
// reads of fresh data (the pairs, then their lists): all of a thread's pairs
// are read before any is used.  Whole searches with five launches / with one:
// 132 / 106 us for 512 pairs over 1024 lists, 140 / 116 for 2048, 166 / 148 for
// 4096, 172 / 175 for 8192; over 4096 lists 222 / 179 us for 512 pairs, 379 /
// 389 for 8192.
constexpr int kSmallQueue = 4096;
constexpr int kSmallBuckets = 15360;  // eight bytes of LDS each, beside four per pair
template <int U>
__global__ __launch_bounds__(1024) void k_queue_small(QueueArgs a, int fp32) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, nt = blockDim.x, NB = a.ncls * a.nlist, n = a.nq * a.npmax;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(lds);  // [NB] pairs, then with their offset << 14
  uint32_t* off = cnt + NB;                          // [NB] list chunks, then the unit offset
  uint32_t* len = off + NB;                          // [n] list lengths
  __shared__ uint2 s_w[16];
  const int per = bucket_run(NB, nt), b0 = tid * per, b1 = b0 + per < NB ? b0 + per : NB;
  // pairs of a unit by class: powers of two
  const int g0 = __builtin_ctz(class_pairs(0, a.wpr, fp32, a.gran, a.M));
  const int g1 = __builtin_ctz(class_pairs(1, a.wpr, fp32, a.gran, a.M));
  const int g2 = __builtin_ctz(class_pairs(2, a.wpr, fp32, a.gran, a.M));
  const int nl = a.nlist, lgs = g0 | g1 << 8 | g2 << 16;
  auto lg_pairs = [nl, lgs](int b) { return lgs >> (8 * ((b >= nl) + (b >= 2 * nl))) & 255; };
  // (lists are shorter than 2^31, so a longer chunk is one)
  const uint32_t ck0 = a.chunk[0] < (1ll << 31) ? (uint32_t)a.chunk[0] : 1u << 31;
  const uint32_t ck1 = a.chunk[1] < (1ll << 31) ? (uint32_t)a.chunk[1] : 1u << 31;
  int p[U], cls[U], kk[U];
  int64_t key[U];
  uint64_t tau[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * nt, j = i < n ? i : 0;
    p[u] = i < n ? a.probes[j] : -1;
    cls[u] = a.pbits[j];
    key[u] = a.pbase ? a.pbase[j] : 0;
    tau[u] = a.pbase ? a.tau[j / a.npmax] : 0;
    kk[u] = a.ph0 == 0 ? (a.kq ? a.kq[j / a.npmax] : a.kconst) : 0;
  }
  uint32_t ln[U];
  int lp[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int l = p[u] < 0 ? 0 : p[u];
    ln[u] = (uint32_t)(a.offsets[l + 1] - a.offsets[l]);
    lp[u] = a.lpos[l];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * nt;
    if (i < n) len[i] = ln[u];
    cls[u] = p[u] < 0 ? 0 : pair_class(cls[u], a.M, a.gran);
  }
  for (int ph = a.ph0; ph < a.ph1; ++ph) {
    const uint32_t ch = ph ? ck1 : ck0;
    for (int b = tid; b < NB; b += nt) cnt[b] = 0;
    int rank[U];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = tid + u * nt;
      rank[u] = -1;
      if (p[u] < 0) continue;
      bool in;
      if (ph == 0) {  // in_phase1: the lists of the ranks before hold fewer than k vectors
        const int r = i % a.npmax;
        int64_t cum = 0;
        in = true;
        for (int j = i - r; j < i && in; ++j) {
          cum += len[j];
          in = cum < kk[u];
        }
      } else {
        in = !a.pbase || (a.fkeys ? (uint64_t)key[u] : ikey(key[u])) <= tau[u];
        if (!in && a.work) atomicAdd((unsigned long long*)&a.work[2], 1ull);
      }
      if (!in) continue;
      const int b = cls[u] * a.nlist + lp[u];
      rank[u] = (int)atomicAdd(&cnt[b], 1u);
      off[b] = (ln[u] + ch - 1) / ch;  // (the same for every pair of the bucket)
    }
    __syncthreads();
    // exclusive scans of pairs and units in launch order, a run per thread
    uint32_t sp = 0, su = 0;
    for (int b = b0; b < b1; ++b) {
      const uint32_t c = cnt[b], nc = off[b];  // (nc: garbage in an empty bucket)
      const int lg = lg_pairs(b);
      sp += c;
      su += c ? ((c + (1u << lg) - 1) >> lg) * nc : 0;
    }
    uint2 tot;
    const uint2 ex = block_exclusive2(sp, su, s_w, &tot);
    uint32_t xp = ex.x, xu = ex.y;
    int64_t* po = a.pairoff + (size_t)ph * (NB + 1);
    int64_t* uo = a.unitoff + (size_t)ph * (NB + 1);
    for (int b = b0; b < b1; ++b) {
      const uint32_t c = cnt[b], nc = off[b];
      const int lg = lg_pairs(b);
      // (the scan kernels read the class boundaries only; all of them on request)
      if (a.all_offsets || b == 0 || b == a.nlist || b == 2 * a.nlist) {
        po[b] = xp;
        uo[b] = xu;
      }
      cnt[b] = c | xp << 14;
      off[b] = xu;
      xp += c;
      xu += c ? ((c + (1u << lg) - 1) >> lg) * nc : 0;
    }
    const bool fits = (int64_t)tot.y <= a.max_units;
    if (tid == 0) {
      po[NB] = tot.x;
      uo[NB] = tot.y;
      if (!fits) atomicOr(&a.flags[0], 4);
    }
    __syncthreads();
    int4* units = a.units + (size_t)ph * a.max_units;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = rank[u];
      if (r < 0) continue;
      const int b = cls[u] * a.nlist + lp[u];
      const int c = (int)(cnt[b] & 16383u), first = (int)(cnt[b] >> 14), lg = lg_pairs(b);
      a.sorted[(size_t)ph * n + first + r] = tid + u * nt;
      if (fits && (r & ((1 << lg) - 1)) == 0) {
        const int nc = (int)((ln[u] + ch - 1) / ch), left = c - r < 1 << lg ? c - r : 1 << lg;
        int4* w = units + off[b] + (size_t)(r >> lg) * nc;
        for (int k = 0; k < nc; ++k) w[k] = make_int4(p[u], first + r, left, k);
      }
    }
    __syncthreads();  // the counts are cleared for the next phase
  }
}

// ------------------------------------------------------------------ bound
// tau[q] = the k-th smallest key of the query's phase-1 bound buffer (every
// entry is the estimate of a distinct vector, so it bounds the query's k-th
// smallest estimate from above), or no bound with fewer than k entries; the
// buffer is emptied for phase 2.  Queries with at most 64 entries: one wave
// each (register bitonic sort); the rest: k_tau, a workgroup each (radix
// select).
__device__ __forceinline__ void tau_wave(uint32_t* ccount, const uint64_t* ckey, uint64_t* tau, int q, int n, int kk,
                                         size_t capq) {
  const int lane = threadIdx.x & 63;
  uint64_t key = lane < n ? ckey[(size_t)q * capq + lane] : ~0ull;
  for (int kb = 2; kb <= 64; kb <<= 1)
    for (int jb = kb >> 1; jb > 0; jb >>= 1) {
      const uint64_t o = __shfl_xor(key, jb);
      const bool keep_min = ((lane & kb) == 0) == ((lane & jb) == 0);
      key = keep_min ? (o < key ? o : key) : (o > key ? o : key);
    }
  const uint64_t kth = __shfl(key, kk <= 64 ? kk - 1 : 63);
  if (lane == 0) {
    tau[q] = n >= kk ? kth : ~0ull;
    ccount[q] = 0;
  }
}
__global__ __launch_bounds__(256) void k_tau_wave(uint32_t* ccount, const uint64_t* ckey, uint64_t* tau,
                                                  const int32_t* kq, int kconst, int nq, size_t capq,
                                                  int32_t* nrerun) {
  const int lane = threadIdx.x & 63;
  const int q = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q == 0 && lane < 2) nrerun[lane] = 0;  // no work units of a phase-2 re-run yet (two rounds)
  if (q >= nq) return;
  const uint32_t cnt = ccount[q];
  const int n = (int)(cnt < capq ? cnt : capq);
  if (n > 64) return;
  tau_wave(ccount, ckey, tau, q, n, kq ? kq[q] : kconst, capq);
}
__global__ __launch_bounds__(256) void k_tau(uint32_t* ccount, const uint64_t* ckey, uint64_t* tau,
                                             const int32_t* kq, int kconst, int nq, size_t capq) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
  uint32_t* hist = reinterpret_cast<uint32_t*>(lds + capq * 8);  // [256]
  uint32_t* sel = hist + 256;                                     // [2]
  int* s_n = reinterpret_cast<int*>(sel + 2);
  int* s_q = s_n + 1;  // [blockDim.x]
  // the workgroup's queries q = blockIdx.x + i * gridDim.x, a thread each:
  // the entry counts are read side by side, and only the queries with more
  // than 64 entries are sorted
  for (int64_t base = blockIdx.x; base < nq; base += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = base + (int64_t)threadIdx.x * gridDim.x;
    bool big = false;
    if (q < nq) {
      const uint32_t c = ccount[q];
      big = (c < capq ? c : capq) > 64;  // (the others: k_tau_wave)
    }
    if (threadIdx.x == 0) *s_n = 0;
    __syncthreads();
    if (big) s_q[atomicAdd(s_n, 1)] = (int)q;
    __syncthreads();
    const int nb = *s_n;
    for (int t = 0; t < nb; ++t) {
      const int qq = s_q[t];
      const uint32_t cnt = ccount[qq];
      const int n = (int)(cnt < capq ? cnt : capq);
      const int kk = kq ? kq[qq] : kconst;
      if (n < kk) {  // uniform over the workgroup
        if (threadIdx.x == 0) {
          tau[qq] = ~0ull;
          ccount[qq] = 0;
        }
        continue;
      }
      for (int i = threadIdx.x; i < n; i += blockDim.x) keys[i] = ckey[(size_t)qq * capq + i];
      __syncthreads();
      const uint64_t kth = block_select_u64(keys, n, kk, hist, sel);
      if (threadIdx.x == 0) {
        tau[qq] = kth;
        ccount[qq] = 0;
      }
      // (the select ends on a barrier: the LDS is free for the next query)
    }
    __syncthreads();  // every thread has read the list before it is reset
  }
}

// both of them for a small batch (at most kSmallBatch queries), a workgroup
// per query (with the merge kernels fused the same way, whole searches 122.5 ->
// 114.7 us for 64 queries, 564 -> 550 for 512 of k 100; even at 1024, slower
// beyond)
constexpr int kSmallBatch = 512;
__global__ __launch_bounds__(256) void k_tau_small(uint32_t* ccount, const uint64_t* ckey, uint64_t* tau,
                                                   const int32_t* kq, int kconst, size_t capq, int32_t* nrerun) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
  uint32_t* hist = reinterpret_cast<uint32_t*>(lds + capq * 8);  // [256]
  uint32_t* sel = hist + 256;                                     // [2]
  const int q = blockIdx.x;
  if (q == 0 && threadIdx.x < 2) nrerun[threadIdx.x] = 0;
  const uint32_t cnt = ccount[q];
  const int n = (int)(cnt < capq ? cnt : capq), kk = kq ? kq[q] : kconst;
  __syncthreads();  // every thread has read the count before it is reset
  if (n <= 64) {
    if (threadIdx.x < 64) tau_wave(ccount, ckey, tau, q, n, kk, capq);
    return;
  }
  uint64_t kth = ~0ull;
  if (n >= kk) {  // uniform over the workgroup
    for (int i = threadIdx.x; i < n; i += blockDim.x) keys[i] = ckey[(size_t)q * capq + i];
    __syncthreads();
    kth = block_select_u64(keys, n, kk, hist, sel);
  }
  if (threadIdx.x == 0) {
    tau[q] = kth;
    ccount[q] = 0;
  }
}

// after phase 2: a query whose candidates overflowed the buffer takes the
// k-th smallest (distance, id) of the candidates kept (distinct vectors, each
// within its old bound) as a tighter bound, and its pairs still within it
// become the work units of a re-run of phase 2, one pair and list chunk each
// (in the phase-1 unit and pair arrays, which are free by then).  Block 0
// also rewinds the phase-2 unit counters.
// (Re-running the phase-2 queue itself with the other queries masked out made
// the re-run pay for claiming and skipping every unit, and for scanning the
// other pairs' lanes: 640 us and 210 us for the bounds by full sorts, for a
// few queries of a 4096-query batch at 5M x 768; 154 and 49 us this way.)
struct RetryArgs {
  uint32_t* ccount;
  const uint64_t* ckey;
  const int64_t* cid;
  uint64_t* tau;
  int64_t* tau_id;
  const int32_t* kq;
  int kconst, nq, ncounters;
  size_t capq;
  int32_t* nrerun;       // this round's unit count
  uint32_t* counters;
  int4* units;           // this round's units
  int32_t* sorted;       // [pair] = pair
};

__global__ __launch_bounds__(256) void k_retry(RetryArgs r, QueueArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
  uint64_t* vals = reinterpret_cast<uint64_t*>(lds + r.capq * 8);   // ids of the keys equal to the k-th smallest
  uint32_t* hist = reinterpret_cast<uint32_t*>(lds + r.capq * 16);  // [256]
  uint32_t* sel = hist + 256;                                        // [2]
  int* s_n = reinterpret_cast<int*>(sel + 2);
  int* s_q = s_n + 1;  // [blockDim.x]
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < r.ncounters; i += blockDim.x) r.counters[i] = 0;
  // the workgroup's queries q = blockIdx.x + i * gridDim.x, a thread each:
  // the candidate counts are read side by side (no chain of dependent
  // loads), and only the overflowed queries go on to the selection
  for (int64_t base = blockIdx.x; base < r.nq; base += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = base + (int64_t)threadIdx.x * gridDim.x;
    const bool over = q < r.nq && r.ccount[q] > r.capq;
    if (threadIdx.x == 0) *s_n = 0;
    __syncthreads();
    if (over) s_q[atomicAdd(s_n, 1)] = (int)q;
    __syncthreads();
    const int n = *s_n;
    __syncthreads();  // s_n counts again below
    for (int t = 0; t < n; ++t) {
      const int qq = s_q[t], nc = (int)r.capq;
      const int kk = r.kq ? r.kq[qq] : r.kconst;
      for (int i = threadIdx.x; i < nc; i += blockDim.x) keys[i] = r.ckey[(size_t)qq * r.capq + i];
      if (threadIdx.x == 0) sel[0] = *s_n = 0;
      __syncthreads();
      const uint64_t key = block_select_u64(keys, nc, kk, hist, sel);
      if (threadIdx.x == 0) sel[0] = 0;
      __syncthreads();
      // its id: the ids of the equal keys, of which (k - smaller keys) are taken
      for (int i = threadIdx.x; i < nc; i += blockDim.x) {
        if (keys[i] < key) atomicAdd(&sel[0], 1u);
        else if (keys[i] == key) vals[atomicAdd(s_n, 1)] = ikey(r.cid[(size_t)qq * r.capq + i]);
      }
      __syncthreads();
      const int below = (int)sel[0], neq = *s_n;
      __syncthreads();
      const int64_t id = ikey_val(block_select_u64(vals, neq, kk - below, hist, sel));
      if (threadIdx.x == 0) {
        r.tau[qq] = key;
        r.tau_id[qq] = id;
        r.ccount[qq] = 0;
      }
      // the pairs that may still hold a candidate
      for (int j = threadIdx.x; j < a.npmax; j += blockDim.x) {
        const size_t i = (size_t)qq * a.npmax + j;
        const int p = a.probes[i];
        if (p < 0) continue;
        if (a.pbase && (a.fkeys ? (uint64_t)a.pbase[i] : ikey(a.pbase[i])) > key) continue;
        const int nch = (int)((a.offsets[p + 1] - a.offsets[p] + a.chunk[1] - 1) / a.chunk[1]);
        if (!nch) continue;
        const int u = atomicAdd(r.nrerun, nch);
        r.sorted[i] = (int32_t)i;
        for (int c = 0; c < nch; ++c) r.units[u + c] = make_int4(p, (int)i, 1, c);
      }
      __syncthreads();  // the LDS is reused by the next query
    }
    __syncthreads();  // every thread has read the list before it is reset
  }
}

// ------------------------------------------------------------------ TS
struct MergeArgs {
  const uint32_t* ccount;
  const uint64_t* ckey;
  const int64_t* cid;
  const int32_t* kq;
  int32_t* flags;
  int64_t* out_ids;
  float* out_dist;
  int64_t* out_qdist;
  int kconst, kmax, fp32;
  float h2;
  size_t capq;
};

// output row r of query q from its sorted candidate r (n candidates)
__device__ __forceinline__ void merge_emit(const MergeArgs& a, int q, int r, int n, int kk, uint64_t key,
                                           int64_t id) {
  const size_t o = (size_t)q * a.kmax + r;
  if (r < kk && r < n) {
    a.out_ids[o] = id;
    if (a.fp32) {
      a.out_dist[o] = fkey_val((uint32_t)key);
      if (a.out_qdist) a.out_qdist[o] = -1;
    } else {
      const int64_t D = ikey_val(key);
      a.out_dist[o] = __ll2float_rn(D) * a.h2;
      if (a.out_qdist) a.out_qdist[o] = D;
    }
  } else {
    a.out_ids[o] = -1;
    a.out_dist[o] = __builtin_inff();
    if (a.out_qdist) a.out_qdist[o] = INT64_MAX;
  }
}

// queries with at most 64 candidates: one wave per query, a register bitonic
// sort of (key, id) across the lanes
__device__ __forceinline__ void merge_wave(const MergeArgs& a, int q, int n, int kk) {
  const int lane = threadIdx.x & 63;
  uint64_t key = lane < n ? a.ckey[(size_t)q * a.capq + lane] : ~0ull;
  int64_t id = lane < n ? a.cid[(size_t)q * a.capq + lane] : INT64_MAX;
  for (int kb = 2; kb <= 64; kb <<= 1)
    for (int jb = kb >> 1; jb > 0; jb >>= 1) {
      const uint64_t ok = __shfl_xor(key, jb);
      const int64_t oid = __shfl_xor(id, jb);
      const bool other_less = ok < key || (ok == key && oid < id);
      const bool other_more = ok > key || (ok == key && oid > id);
      const bool keep_min = ((lane & kb) == 0) == ((lane & jb) == 0);
      if (keep_min ? other_less : other_more) {
        key = ok;
        id = oid;
      }
    }
  for (int r = lane; r < a.kmax; r += 64) merge_emit(a, q, r, n, kk, key, id);
}
__global__ __launch_bounds__(256) void k_merge_wave(MergeArgs a, int nq) {
  const int q = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= nq) return;
  const uint32_t cnt = a.ccount[q];
  if (cnt > a.capq && (threadIdx.x & 63) == 0) atomicOr(&a.flags[0], 2);
  const int n = (int)(cnt < a.capq ? cnt : a.capq);
  if (n > 64) return;  // the workgroup kernel takes it
  merge_wave(a, q, n, a.kq ? a.kq[q] : a.kconst);
}

// queries with more than 64 candidates and more than k: a workgroup per
// query (strided over the queries).  A radix select finds the k-th smallest
// key; the candidates up to it, when at most kMergeSel, take their output
// rows from their rank (key, id, position) among themselves.  The other
// queries (at most k candidates, or more than kMergeSel up to the k-th key)
// are left to k_merge_full, marked by id -2 in their first output row.
constexpr int kMergeSel = 256;
inline size_t merge_select_lds(size_t capq) { return capq * 8 + kMergeSel * 20 + 4 * (256 + 3); }

// by selection; false (nothing written) with more than kMergeSel candidates
// up to the k-th key.  Ends with the LDS free.
__device__ __forceinline__ bool merge_select(const MergeArgs& a, int q, int n, int kk, char* lds) {
  uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
  uint64_t* skey = reinterpret_cast<uint64_t*>(lds + a.capq * 8);  // [kMergeSel]
  int64_t* sval = reinterpret_cast<int64_t*>(skey + kMergeSel);    // [kMergeSel]
  int32_t* sidx = reinterpret_cast<int32_t*>(sval + kMergeSel);    // [kMergeSel]
  uint32_t* hist = reinterpret_cast<uint32_t*>(sidx + kMergeSel);  // [256]
  uint32_t* sel = hist + 256;                                       // [2]
  uint32_t* s_cnt = sel + 2;
  for (int i = threadIdx.x; i < n; i += blockDim.x) keys[i] = a.ckey[(size_t)q * a.capq + i];
  if (threadIdx.x == 0) *s_cnt = 0;
  __syncthreads();
  const uint64_t v = block_select_u64(keys, n, kk, hist, sel);
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    if (keys[i] <= v) {
      const uint32_t j = atomicAdd(s_cnt, 1u);
      if (j < (uint32_t)kMergeSel) {
        skey[j] = keys[i];
        sval[j] = a.cid[(size_t)q * a.capq + i];
        sidx[j] = i;
      }
    }
  __syncthreads();
  const int ns = (int)*s_cnt;
  if (ns <= kMergeSel) {
    for (int t = threadIdx.x; t < ns; t += blockDim.x) {
      const uint64_t kt = skey[t];
      const int64_t it = sval[t];
      const int xt = sidx[t];
      int rank = 0;
      for (int j = 0; j < ns; ++j) {
        const uint64_t kj = skey[j];
        const int64_t ij = sval[j];
        rank += kj < kt || (kj == kt && (ij < it || (ij == it && sidx[j] < xt)));
      }
      if (rank < kk) merge_emit(a, q, rank, n, kk, kt, it);
    }
    for (int r = kk + threadIdx.x; r < a.kmax; r += blockDim.x) merge_emit(a, q, r, n, kk, ~0ull, INT64_MAX);
  }
  __syncthreads();
  return ns <= kMergeSel;
}

// by a sort of every candidate by (key, id) in LDS (bitonic over the next
// power of two).  Ends with the LDS free.
__device__ __forceinline__ void merge_sort(const MergeArgs& a, int q, int n, int kk, char* lds) {
  uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
  int64_t* vals = reinterpret_cast<int64_t*>(lds + a.capq * 8);
  int np2 = 1;
  while (np2 < n) np2 <<= 1;
  for (int i = threadIdx.x; i < np2; i += blockDim.x) {
    keys[i] = i < n ? a.ckey[(size_t)q * a.capq + i] : ~0ull;
    vals[i] = i < n ? a.cid[(size_t)q * a.capq + i] : INT64_MAX;
  }
  __syncthreads();
  block_bitonic_u64_i64(keys, vals, np2);
  for (int r = threadIdx.x; r < a.kmax; r += blockDim.x)
    merge_emit(a, q, r, n, kk, r < n ? keys[r] : ~0ull, r < n ? vals[r] : INT64_MAX);
  __syncthreads();
}

__global__ __launch_bounds__(256) void k_merge(MergeArgs a, int nq) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  for (int q = blockIdx.x; q < nq; q += gridDim.x) {
    const uint32_t cnt = a.ccount[q];
    if (cnt > a.capq && threadIdx.x == 0) atomicOr(&a.flags[0], 2);
    const int n = (int)(cnt < a.capq ? cnt : a.capq);
    if (n <= 64) continue;  // uniform over the workgroup
    const int kk = a.kq ? a.kq[q] : a.kconst;
    if (kk >= n || !merge_select(a, q, n, kk, lds)) {
      if (threadIdx.x == 0) a.out_ids[(size_t)q * a.kmax] = -2;
    }
  }
}

// the queries k_merge left (id -2 in the first output row): a workgroup per
// query (strided over the queries)
__global__ __launch_bounds__(256) void k_merge_full(MergeArgs a, int nq) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  for (int q = blockIdx.x; q < nq; q += gridDim.x) {
    const uint32_t cnt = a.ccount[q];
    const int n = (int)(cnt < a.capq ? cnt : a.capq);
    if (n <= 64 || a.out_ids[(size_t)q * a.kmax] != -2) continue;  // uniform over the workgroup
    __syncthreads();  // every thread has read the mark before it is overwritten
    merge_sort(a, q, n, a.kq ? a.kq[q] : a.kconst, lds);
  }
}

// all three for a small batch (at most kSmallBatch queries), a workgroup per
// query
__global__ __launch_bounds__(256) void k_merge_small(MergeArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int q = blockIdx.x, kk = a.kq ? a.kq[q] : a.kconst;
  const uint32_t cnt = a.ccount[q];
  if (cnt > a.capq && threadIdx.x == 0) atomicOr(&a.flags[0], 2);
  const int n = (int)(cnt < a.capq ? cnt : a.capq);
  if (n <= 64) {
    if (threadIdx.x < 64) merge_wave(a, q, n, kk);
  } else if (kk >= n || !merge_select(a, q, n, kk, lds)) {
    merge_sort(a, q, n, kk, lds);
  }
}

// ------------------------------------------------------------------ index prep
// MFMA B fragments of the grid codebook: for m-pair mp, codeword tile jt and
// lane l (group kg = l/16, codeword j = 16 jt + l%16):
//   kg even: cbi[m][j][0..dsub) zero-padded to 8;  kg odd: digits of
//   cc = |cbi[m][j]|^2 (base 256, most significant first) then 65536, 256, 1
// bsw: BF16 (all groups); bsw16: FP16 dims (odd groups zero).
__global__ void k_prep_bsw(const float* __restrict__ cb, int M, int dsub, int grid_e, int grid_kind,
                           u32x4* __restrict__ bsw, u32x4* __restrict__ bsw16, u32x2* __restrict__ bsw8) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int total = (M / 2) * 16 * 64;
  if (idx >= total) return;
  const int lane = idx & 63, jt = (idx >> 6) & 15, mp = idx >> 10;
  const int kg = lane >> 4, j = jt * 16 + (lane & 15);
  const int m = 2 * mp + (kg >> 1);
  const float* c = cb + ((size_t)m * kKsub + j) * dsub;
  float v[8];
  int ci[kMaxDsub];
  int cc = 0;
  for (int t = 0; t < kMaxDsub; ++t) {
    ci[t] = t < dsub ? grid_val(c[t], grid_e, grid_kind) : 0;
    cc += ci[t] * ci[t];
  }
  uint32_t h[4] = {0, 0, 0, 0}, f8[2] = {0, 0};
  if ((kg & 1) == 0) {
    for (int t = 0; t < 8; ++t) v[t] = (float)ci[t];
    for (int t = 0; t < 4; ++t) h[t] = f16_bits(v[2 * t]) | (f16_bits(v[2 * t + 1]) << 16);
    // e4m3 bytes (exact on the e4m3 grid; the FP8 build is only offered there)
    f8[0] = f8_bits4(v[0], v[1], v[2], v[3]);
    f8[1] = f8_bits4(v[4], v[5], v[6], v[7]);
  } else {
    v[0] = (float)(cc >> 16);
    v[1] = (float)((cc >> 8) & 255);
    v[2] = (float)(cc & 255);
    v[3] = 65536.f;
    v[4] = 256.f;
    v[5] = 1.f;
    v[6] = 0.f;
    v[7] = 0.f;
  }
  u32x4 o;
  for (int t = 0; t < 4; ++t) o[t] = bf16_bits(v[2 * t]) | (bf16_bits(v[2 * t + 1]) << 16);
  bsw[idx] = o;
  bsw16[idx] = (u32x4){h[0], h[1], h[2], h[3]};
  bsw8[idx] = (u32x2){f8[0], f8[1]};
}

// L2, FP32 policy: fragments of the FP32 codebook for the pair bounds
// (k_base_l2f).  For subspace m, tile t of 32 codewords and lane l (codeword
// j = 32 t + l % 32): fragment 0 holds the BF16 high parts of the codeword's
// dims (lanes 0-31) and the BF16 low parts (the rest rounded, lanes 32-63);
// fragment 1 the high parts again, |c|^2 in three BF16 pieces and three ones
// (for the pieces of |r|^2).  The word
// after the last fragment is the sum over the subspaces of the largest |c|^2.
__device__ __forceinline__ uint32_t bf16_rn(float v, float& rest) {
  const __bf16 h = (__bf16)v;
  rest = v - (float)h;
  return (uint32_t)__builtin_bit_cast(uint16_t, h);
}
__global__ void k_prep_bswf(const float* __restrict__ cb, int M, int dsub, u32x4* __restrict__ bswf) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= M * 8 * 64) return;
  const int lane = idx & 63, t = (idx >> 6) & 7, m = idx >> 9;
  const float* c = cb + ((size_t)m * kKsub + t * 32 + (lane & 31)) * dsub;
  uint32_t hi[8], lo[8];
  float cc = 0.f;
  for (int i = 0; i < 8; ++i) {
    const float v = i < dsub ? c[i] : 0.f;
    float r;
    hi[i] = bf16_rn(v, r);
    lo[i] = bf16_rn(r, r);
    cc = fmaf(v, v, cc);
  }
  const u32x4 h = {hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16), hi[4] | (hi[5] << 16), hi[6] | (hi[7] << 16)};
  const u32x4 l = {lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16), lo[4] | (lo[5] << 16), lo[6] | (lo[7] << 16)};
  float r;
  const uint32_t c0 = bf16_rn(cc, r), c1 = bf16_rn(r, r), c2 = bf16_rn(r, r);
  u32x4* o = bswf + ((size_t)(m * 8 + t) * 2) * 64 + lane;
  o[0] = lane < 32 ? h : l;
  o[64] = lane < 32 ? h : (u32x4){c0 | (c1 << 16), c2 | 0x3F800000u, 0x3F803F80u, 0u};
}
__global__ __launch_bounds__(256) void k_prep_cbsum(const float* __restrict__ cb, int M, int dsub, float* out) {
  __shared__ float s_w[4];
  float sum = 0.f;
  for (int m = 0; m < M; ++m) {
    const float* c = cb + ((size_t)m * kKsub + threadIdx.x) * dsub;
    float cc = 0.f;
    for (int i = 0; i < dsub; ++i) cc = fmaf(c[i], c[i], cc);
    // (a NaN must survive the maximum: it disables the bounds)
    for (int o = 32; o > 0; o >>= 1) {
      const float v = __shfl_xor(cc, o);
      cc = v > cc || v != v ? v : cc;
    }
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = cc;
    __syncthreads();
    float mx = s_w[0];
    for (int w = 1; w < 4; ++w) mx = s_w[w] > mx || s_w[w] != s_w[w] ? s_w[w] : mx;
    sum += mx;
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sum;
}

// ------------------------------------------------------------------ inner-product tables
// queries on the operand grid (inner product)
__global__ void k_qgrid(const float* __restrict__ Q, int16_t* __restrict__ qi, size_t n, int grid_e, int grid_kind) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    qi[i] = (int16_t)grid_val(Q[i], grid_e, grid_kind);
}

constexpr int kTabQ = 8;  // queries per workgroup of the table build (one 8-row MFMA tile)

// inner product, integer policies: each query's exact table T[m][j] =
// -qi_m . cbi_mj (LUT pass 1 on MFMA, the entries kept) and its row minima;
// the largest row span and the sum of the minima are gathered per query with
// one atomic each (k_ipq completes the pair bases from them).  mps m-pairs of
// the table per workgroup: all of them where the queries alone fill the chip
// (the codebook fragments, M * 8 KB, are read once per eight queries), fewer
// for small batches, whose workgroups were each a chain of M / 8 steps on an
// otherwise idle chip (M 96: 300 queries 69 us with 38 workgroups, 14 with 456;
// 4096 queries 98 us with one workgroup per eight queries, 88 with the
// pair bases formed by k_ipq)
template <int DT>
__global__ __launch_bounds__(kThreads) void k_iptab(BaseArgs b, int mps) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const ScanLds L = base_lds_layout(kTabQ, b.M, b.d);
  ScanArgs a{};
  a.d = b.d;
  a.dsub = b.dsub;
  a.M = b.M;
  a.tab_out = b.iptab;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int M = b.M;
  const int q0 = blockIdx.x * kTabQ;
  const int nqb = b.nq - q0 < kTabQ ? b.nq - q0 : kTabQ;
  const int mp0 = blockIdx.y * mps, mp1 = mp0 + mps < M / 2 ? mp0 + mps : M / 2;
  int32_t* pq = reinterpret_cast<int32_t*>(lds + L.pq);
  if (tid < kTabQ) pq[tid] = q0 + tid;
  const int d4 = b.d >> 2, rs4 = ri_stride(b.d) >> 2;
  for (int e = tid; e < kTabQ * d4; e += kThreads) {
    const int g = e / d4, t4 = e - g * d4;
    u32x2 v = {0u, 0u};
    if (g < nqb) v = reinterpret_cast<const u32x2*>(b.qi16 + (size_t)(q0 + g) * b.d)[t4];
    reinterpret_cast<u32x2*>(lds + L.ri)[g * rs4 + t4] = v;
  }
  __syncthreads();
  for (int mp = mp0 + wave; mp < mp1; mp += kThreads / 64) {
    u32x4 Bt[16], Bd[16];
    base_frags<DT>(b, mp, lane, Bt, Bd);
    lut_mpair<32, kTabQ, DT, 4, true>(a, lds, L, M, nqb, mp, Bt, Bd);
  }
  __syncthreads();
  const int32_t* lo = reinterpret_cast<const int32_t*>(lds + L.lo);
  const int32_t* hi = reinterpret_cast<const int32_t*>(lds + L.hi);
  // per query (a wave each): span and sum of minima (per-subspace
  // granularity: the sum of the row spans instead of the largest)
  for (int g = wave; g < nqb; g += kThreads / 64) {
    int32_t span = 0;
    int64_t sum = 0, rsum = 0;
    for (int m = 2 * mp0 + lane; m < 2 * mp1; m += 64) {
      const int32_t l = lo[g * M + m], h = hi[g * M + m];
      b.iplo[(size_t)(q0 + g) * M + m] = l;
      span = h - l > span ? h - l : span;
      rsum += h - l;
      sum += l;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const int32_t o = __shfl_xor(span, off);
      span = o > span ? o : span;
      sum += __shfl_xor(sum, off);
      rsum += __shfl_xor(rsum, off);
    }
    if (lane == 0) {
      if (b.gran) atomicAdd(&b.ipspan[q0 + g], (int32_t)rsum);
      else atomicMax(&b.ipspan[q0 + g], span);
      atomicAdd(reinterpret_cast<unsigned long long*>(&b.iplsum[q0 + g]), (unsigned long long)sum);
    }
  }
}

// inner product, FP32 policy: each query's dot products q_m . c_mj in FP32
// (the FMA chain of the scan's FP32 entries, in the same order) and the
// largest of each row
// A thread holds one codeword of subspace m in registers and walks over the
// workgroup's queries, whose coordinates are uniform (scalar loads): bound by
// the table writes (1024 queries x 96 x 256: 100 MB, 21 us at the copy rate;
// a thread per entry with both operands read from memory, and the rows read again
// for their maxima, took 359 us; 36 now).
constexpr int kTabF = 32;  // queries per workgroup (a multiple of four)

// largest of the wave's 64 values on lane 63 (a lane without a source in a step
// keeps its own; NaN is passed over)
__device__ __forceinline__ float wave_max63(float x) {
  auto step = [&](auto ctrl) {
    const int xi = __float_as_int(x);
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(xi, xi, decltype(ctrl)::value, 0xF, 0xF, false)));
  };
  step(std::integral_constant<int, 0x111>{});  // within rows of sixteen: 1, 2, 4, 8 to the right
  step(std::integral_constant<int, 0x112>{});
  step(std::integral_constant<int, 0x114>{});
  step(std::integral_constant<int, 0x118>{});
  step(std::integral_constant<int, 0x142>{});  // a row's last lane to the next row
  step(std::integral_constant<int, 0x143>{});  // lane 31 to the upper half
  return x;
}

template <int DS>  // dsub
__global__ __launch_bounds__(256) void k_iptab_f32(BaseArgs b) {
  __shared__ float s_mx[kTabF][4];
  const int m = blockIdx.x, j = threadIdx.x, lane = j & 63;
  const int q0 = (blockIdx.z * gridDim.y + blockIdx.y) * kTabF;
  if (q0 >= b.nq) return;
  const int nqb = b.nq - q0 < kTabF ? b.nq - q0 : kTabF;
  float c[DS];
#pragma unroll
  for (int t = 0; t < DS; ++t) c[t] = b.codebook[((size_t)m * kKsub + j) * DS + t];
  float* out = reinterpret_cast<float*>(b.iptab);
  for (int g0 = 0; g0 < nqb; g0 += 4) {
    float dot[4] = {0.f, 0.f, 0.f, 0.f};
    // (past the last query: its row again, not stored)
    const float* r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = b.Q + (size_t)(q0 + (g0 + u < nqb ? g0 + u : nqb - 1)) * b.d + m * DS;
#pragma unroll
    for (int t = 0; t < DS; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) dot[u] = fmaf(r[u][t], c[t], dot[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (g0 + u < nqb) out[((size_t)(q0 + g0 + u) * b.M + m) * kKsub + j] = dot[u];
      const float mx = wave_max63(dot[u]);
      if (lane == 63) s_mx[g0 + u][j >> 6] = mx;
    }
  }
  __syncthreads();
  if (j < nqb)
    reinterpret_cast<float*>(b.iplo)[(size_t)(q0 + j) * b.M + m] =
        fmaxf(fmaxf(s_mx[j][0], s_mx[j][1]), fmaxf(s_mx[j][2], s_mx[j][3]));
}

// inner product: qi.ci of each pair (exact integers; k_ipq subtracts it
// from the sum of the query's row minima: the pair's base), for the
// policies whose predictor pass does not compute it.  A workgroup per query,
// sixteen lanes per probed list (sixteen lists per step); the widths the
// query's pairs use (the tables k_ipq builds) are gathered in the workgroup
// and set with one atomic.
__global__ __launch_bounds__(256) void k_ipbase(BaseArgs b) {
  __shared__ int s_mask;
  const size_t q = blockIdx.x;
  const int tid = threadIdx.x, r = tid & 15, grp = tid >> 4;
  if (tid == 0) s_mask = 0;
  __syncthreads();
  const u32x2* qv = reinterpret_cast<const u32x2*>(b.qi16 + q * b.d);
  const int d4 = b.d >> 2;
  int mask = 0;
  for (int j0 = 0; j0 < b.npmax; j0 += 16) {
    const int j = j0 + grp;
    const size_t i = q * b.npmax + j;
    const int p = j < b.npmax ? b.probes[i] : -1;
    int acc = 0;
    if (p >= 0) {
      const u32x2* cv = reinterpret_cast<const u32x2*>(b.ci16 + (size_t)p * b.d);
      for (int t4 = r; t4 < d4; t4 += 16) {
        const u32x2 x = qv[t4], c = cv[t4];
        acc += (int)(int16_t)(x[0] & 0xFFFFu) * (int)(int16_t)(c[0] & 0xFFFFu) +
               (int)(int16_t)(x[0] >> 16) * (int)(int16_t)(c[0] >> 16) +
               (int)(int16_t)(x[1] & 0xFFFFu) * (int)(int16_t)(c[1] & 0xFFFFu) +
               (int)(int16_t)(x[1] >> 16) * (int)(int16_t)(c[1] >> 16);
      }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 16);
    if (p >= 0 && r == 0) {
      b.pbase[i] = acc;  // qi.ci: k_ipq turns it into the base once the query's minima are known
      mask |= 1 << ((b.pbits[i] >> 2) - 1);
    }
  }
  if (mask) atomicOr(&s_mask, mask);
  __syncthreads();
  if (tid == 0 && s_mask) atomicOr(&b.ipmask[q], s_mask);
}

// inner product, FP32 policy: the key of a lower bound of each pair's in-order
// FP32 sums, from the pair's coarse distance D = -q.c: D - sum_m max_j dot_mj
// less a slack for every rounding on the way (a workgroup per query).  Rounding
// is monotone, so the scan's in-order sum of a vector's entries is at least that
// of the rows' smallest ones.  With mag = |q| |c| + sum_m |max_j dot_mj| the
// coarse sum differs from the exact one by at most d roundings of 2^-24 mag, the
// scan's list term by dsub + M, its sum of M entries by M, the sum here by
// M / 256 + 8; twice their count is taken, and norms below which squares
// underflow count as 1e-17.  Not finite, or near overflow: key 0, the scan
// decides.  (The bound by the scan's own arithmetic read every pair's rows again
// and added 2 M terms one after the other on every lane: 768 us for 143k pairs,
// d 768, M 96; 5 now, with the same 107k pairs left out.)
__global__ __launch_bounds__(256) void k_ipbound_f32(BaseArgs b, const float* __restrict__ coarse,
                                                     const float* __restrict__ qn, const float* __restrict__ cn,
                                                     int nlist) {
  __shared__ float s_s[4], s_a[4];
  const size_t q = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const float* mx = reinterpret_cast<const float*>(b.iplo) + q * b.M;
  float s = 0.f, ab = 0.f;
  for (int m = tid; m < b.M; m += 256) {
    s += mx[m];
    ab += fabsf(mx[m]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_xor(s, off);
    ab += __shfl_xor(ab, off);
  }
  if (lane == 0) {
    s_s[tid >> 6] = s;
    s_a[tid >> 6] = ab;
  }
  __syncthreads();
  s = (s_s[0] + s_s[1]) + (s_s[2] + s_s[3]);
  ab = (s_a[0] + s_a[1]) + (s_a[2] + s_a[3]);
  const float u = (float)(b.d + b.dsub + 2 * b.M + 64) * 0x1p-23f;
  const float qq = qn[q];
  for (int j = tid; j < b.npmax; j += 256) {
    const size_t i = q * b.npmax + j;
    const int p = b.probes[i];
    if (p < 0) continue;
    const float mag = (sqrtf(qq) + 1e-17f) * (sqrtf(cn[p]) + 1e-17f) * 1.001f + ab;
    const float lb = (coarse[q * nlist + p] - s) - (mag * u + 1e-30f * (float)b.M);
    const bool ok = mag < 1e30f && qq < 1e37f && cn[p] < 1e37f && lb > -1e37f && lb < 1e37f;  // false for NaN
    b.pbase[i] = ok ? (int64_t)fkey(lb) : 0;
  }
}

// the same where the coarse distances are integer ones, computed
// with the scan's own FP32 arithmetic (a wave per pair): the pair's base
// term bf = sum over the subspaces (in order) of the FMA chain of -q_t c_t,
// then the in-order sum over the subspaces of the smallest LUT entry,
// bf - max_j dot_0j for subspace 0 and 0 - max_j dot_mj for the others
// (rounding is monotone, so these are the rows' smallest entries)
__global__ __launch_bounds__(256) void k_ipbase_f32(BaseArgs b) {
  const int lane = threadIdx.x & 63;
  const size_t i = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= (size_t)b.nq * b.npmax) return;
  const int p = b.probes[i];
  if (p < 0) return;
  const size_t q = i / b.npmax;
  const float* r = b.Q + q * b.d;
  const float* c = b.C + (size_t)p * b.d;
  float bf = 0.f;
  for (int m0 = 0; m0 < b.M; m0 += 64) {
    const int m = m0 + lane;
    float sq = 0.f;
    if (m < b.M)
      for (int t = 0; t < b.dsub; ++t) sq = fmaf(-r[m * b.dsub + t], c[m * b.dsub + t], sq);
    const int nm = b.M - m0 < 64 ? b.M - m0 : 64;
    for (int k = 0; k < nm; ++k) bf += __shfl(sq, k);  // in subspace order, the same on every lane
  }
  const float* mx = reinterpret_cast<const float*>(b.iplo) + q * b.M;
  float sb = 0.f;
  for (int m = 0; m < b.M; ++m) sb += (m == 0 ? bf : 0.f) - mx[m];
  if (lane == 0) b.pbase[i] = (int64_t)fkey(sb);
}

// LUT export (test hook), inner product: a pair's LUT is its query's table
// at its width (a workgroup per pair)
__global__ void k_export_ip(BaseArgs b, uint16_t* exq, int32_t* exs, int64_t* exb, int32_t* ext) {
  const size_t i = blockIdx.x;
  const int p = b.probes[i];
  if (p < 0) return;
  const size_t q = i / b.npmax;
  const int wi = (b.pbits[i] >> 2) - 1;
  const size_t tsz = (size_t)b.M * kKsub;
  if (threadIdx.x == 0) {
    exs[i] = b.ipsh[q * 4 + wi];
    exb[i] = b.pbase[i];
  }
  const uint16_t* slot = b.iptq + (q * 4 + wi) * tsz;
  const bool by = ip_bytes(b.gran, wi, b.M);
  for (size_t e = threadIdx.x; e < tsz; e += blockDim.x) {
    exq[i * tsz + e] = by ? reinterpret_cast<const uint8_t*>(slot)[e] : slot[e];
    if (ext) ext[i * tsz + e] = b.iptab[q * tsz + e];
  }
}

// inner product, integer policies: each query's table quantised at every
// width its pairs use: shift s from the query's span (smallest with
// (span + hf(s)) >> s <= 2^b - 1), entries (T - min_m + hf(s)) >> s as
// uint16, or as bytes in the first half of the table's slot (ip_bytes);
// eight entries per thread, read once and written at every width the query
// needs
__global__ void k_ipq(BaseArgs b) {
  // the pair bases: sum of the query's row minima - qi.ci (pbase held qi.ci)
  const size_t np = (size_t)b.nq * b.npmax;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < np; i += (size_t)gridDim.x * blockDim.x)
    if (b.probes[i] >= 0) b.pbase[i] = b.iplsum[i / b.npmax] - b.pbase[i];
  const size_t per = (size_t)b.M * kKsub / 8;
  const size_t n = (size_t)b.nq * per;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const size_t q = i / per;
    const int mask = b.ipmask[q];
    if (!mask) continue;
    const size_t e0 = (i - q * per) * 8;
    const int m = (int)(e0 >> 8);
    const int lo = b.iplo[q * b.M + m];
    const int32_t* T = b.iptab + q * b.M * kKsub + e0;
    const u32x4 t0 = *reinterpret_cast<const u32x4*>(T), t1 = *reinterpret_cast<const u32x4*>(T + 4);
    const int tv[8] = {(int)t0[0], (int)t0[1], (int)t0[2], (int)t0[3], (int)t1[0], (int)t1[1], (int)t1[2], (int)t1[3]};
    for (int wi = 0; wi < 4; ++wi) {
      if (!(mask & (1 << wi))) continue;
      const size_t qw = q * 4 + wi;
      const int sh = quant_shift(b.ipspan[q], b.gran ? b.M : 1, 4 * (wi + 1));
      const int off = (sh ? 1 << (sh - 1) : 0) - lo;
      if (e0 == 0) b.ipsh[qw] = sh;
      uint32_t v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = (uint32_t)((tv[k] + off) >> sh);
      uint16_t* slot = b.iptq + qw * ((size_t)b.M * kKsub);
      if (ip_bytes(b.gran, wi, b.M)) {
        *reinterpret_cast<u32x2*>(reinterpret_cast<uint8_t*>(slot) + e0) =
            (u32x2){v[0] | (v[1] << 8) | (v[2] << 16) | (v[3] << 24), v[4] | (v[5] << 8) | (v[6] << 16) | (v[7] << 24)};
      } else {
        *reinterpret_cast<u32x4*>(slot + e0) =
            (u32x4){v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
      }
    }
  }
}

// ------------------------------------------------------------------ pair bases, L2
// Lower bound of every (query, probed list) pair's estimates on L2, and its
// d' for the predictor.  Integer policies: the exact base, sum over the
// subspaces of min_j T[m][j] with T = |ri_m|^2 + (|cbi|^2 - 2 ri_m . cbi).
//
// A v_mfma_f32_32x32x16_bf16 takes 32 codewords as its rows and 32 pairs as
// its columns for one subspace: K holds the 8 dims (lanes 0-31 of either
// operand) and the base-256 digits of |cbi|^2 (lanes 32-63; the pair side
// holds their powers and an offset that keeps every sum positive, so that
// float bit patterns order as integers and two results take one v_min3).  A
// lane then holds 16 codewords of ONE pair: the minimum over the 256
// codewords needs one cross-lane step per subspace, and the pair operand is
// 16 bytes of the residual row as it sits in LDS (-2 ri in BF16, exact).
// Every product and sum is an integer below 2^24: exact in any order.
//
// kBaseNT threads, NPT tiles of 32 pairs; the subspaces go in chunks of
// kBaseCM, whose residuals the workgroup puts on the grid, then each wave
// takes subspaces of the chunk with its 8 codeword fragments (32 registers)
// kept over all pair tiles.  Bound by the matrix unit and the VALU minima,
// 32 clocks each per 1024 entries (17 us at 10000 x 32 pairs, d 128, M 16),
// and the residual rows read before them: 76 us measured, see launch_base_l2.
// 128 registers (four pair tiles: and 20 bytes of scratch per lane): two
// workgroups per CU, one on its rows while the other multiplies (161 registers,
// one workgroup: 104 us).
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kBaseCM = 16;   // subspaces per chunk
constexpr int kBaseNT = 512;  // threads

struct BaseL2Args {
  const float* Q;
  const float* C;
  const u32x4* bsw;      // MFMA B fragments of the grid codebook (k_prep_bsw)
  const int32_t* probes;
  int64_t* pbase;        // [nq][npmax]
  int64_t* dq2;          // [nq][npmax] squared norm of the grid residual
  int nq, d, M, dsub, npmax, grid_e, grid_kind;
};

constexpr int base_l2_row() { return kBaseCM * 16 + 16; }  // bytes of a residual row (padded: distinct banks)
inline size_t base_l2_lds(int npt) { return (size_t)npt * 32 * (base_l2_row() + 8 + 8 + 4 + 4); }

template <int NPT>
__global__ __launch_bounds__(kBaseNT, 4) void k_base_l2(BaseL2Args b) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int G = NPT * 32, ROW = base_l2_row(), NW = kBaseNT / 64, RU = NPT < 4 ? NPT : 4;
  unsigned long long* smin = reinterpret_cast<unsigned long long*>(lds + G * ROW);  // [G] sum of the minima
  int64_t* srr = reinterpret_cast<int64_t*>(smin + G);                              // [G] sum of |ri|^2
  int32_t* sp = reinterpret_cast<int32_t*>(srr + G);                                // [G] list of the pair, or -1
  int32_t* sq = sp + G;                                                             // [G] query of the pair
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = tid & 15, grp = tid >> 4;
  const size_t n = (size_t)b.nq * b.npmax, i0 = (size_t)blockIdx.x * G;
  for (int g = tid; g < G; g += kBaseNT) {
    const size_t i = i0 + g;
    sp[g] = i < n ? b.probes[i] : -1;
    sq[g] = i < n ? (int)(i / b.npmax) : 0;
    smin[g] = 0;
    srr[g] = 0;
  }
  const int ds = b.dsub;
  if (ds != 8 && ds != 4 && ds != 2) {
    // rows of other widths are written element by element: the padding stays zero
    for (int i = tid; i < G * ROW / 16; i += kBaseNT) reinterpret_cast<u32x4*>(lds)[i] = (u32x4){0u, 0u, 0u, 0u};
  }
  int64_t sum[NPT];
#pragma unroll
  for (int t = 0; t < NPT; ++t) sum[t] = 0;
  // pair side of the |cbi|^2 digits and the offset 64 * 65536 = 2^22 (the
  // codeword side holds 65536 there), above any 2 |ri . cbi| (at most 8 * 2 *
  // 448^2)
  const u32x4 aug = {0x43804780u, 0x42803F80u, 0u, 0u};  // BF16 65536, 256 | 1, 64 | 0
  constexpr int kOff = 1 << 22;
  for (int m0 = 0; m0 < b.M; m0 += kBaseCM) {
    const int cm = b.M - m0 < kBaseCM ? b.M - m0 : kBaseCM;
    const int cd4 = (cm * ds) >> 2, o4 = (m0 * ds) >> 2;  // M and the chunk are multiples of 4
    __syncthreads();  // the last chunk's rows are read (first chunk: the lists are in)
    // residuals onto the grid: sixteen lanes per pair, two 16-byte reads each
#pragma unroll RU
    for (int u = 0; u < G / (kBaseNT / 16) + (G < kBaseNT / 16); ++u) {
      const int g = grp + u * (kBaseNT / 16);
      if (g >= G) break;
      const int p = sp[g] < 0 ? 0 : sp[g];  // (absent pairs: any row, never written out)
      const float4* qr = reinterpret_cast<const float4*>(b.Q + (size_t)sq[g] * b.d) + o4;
      const float4* cr = reinterpret_cast<const float4*>(b.C + (size_t)p * b.d) + o4;
      int s2 = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t4 = l16 + 16 * h;
        if (t4 >= cd4) break;
        const float4 x = qr[t4], c = cr[t4];
        const int v0 = grid_val(x.x - c.x, b.grid_e, b.grid_kind), v1 = grid_val(x.y - c.y, b.grid_e, b.grid_kind);
        const int v2 = grid_val(x.z - c.z, b.grid_e, b.grid_kind), v3 = grid_val(x.w - c.w, b.grid_e, b.grid_kind);
        s2 += v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3;
        const uint32_t b0 = bf16_bits((float)(-2 * v0)), b1 = bf16_bits((float)(-2 * v1));
        const uint32_t b2 = bf16_bits((float)(-2 * v2)), b3 = bf16_bits((float)(-2 * v3));
        char* row = lds + g * ROW;
        if (ds == 8) {
          *reinterpret_cast<u32x2*>(row + t4 * 8) = (u32x2){b0 | (b1 << 16), b2 | (b3 << 16)};
        } else if (ds == 4) {
          *reinterpret_cast<u32x4*>(row + t4 * 16) = (u32x4){b0 | (b1 << 16), b2 | (b3 << 16), 0u, 0u};
        } else if (ds == 2) {
          *reinterpret_cast<u32x4*>(row + t4 * 32) = (u32x4){b0 | (b1 << 16), 0u, 0u, 0u};
          *reinterpret_cast<u32x4*>(row + t4 * 32 + 16) = (u32x4){b2 | (b3 << 16), 0u, 0u, 0u};
        } else {
          const uint32_t bv[4] = {b0, b1, b2, b3};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int t = 4 * t4 + k;
            *reinterpret_cast<uint16_t*>(row + (t / ds) * 16 + (t % ds) * 2) = (uint16_t)bv[k];
          }
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) s2 += __shfl_xor(s2, o, 16);
      if (l16 == 0) srr[g] += s2;
    }
    __syncthreads();
    for (int mi = wave; mi < cm; mi += NW) {
      const int m = m0 + mi;
      // codeword fragments of the subspace: 32 codewords per tile, dims in
      // lanes 0-31, digits in lanes 32-63
      const u32x4* src = b.bsw + (size_t)(m >> 1) * 1024 + (2 * (m & 1) + (lane >> 5)) * 16 + (lane & 15) +
                         ((lane >> 4) & 1) * 64;
      u32x4 cw[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) cw[t] = src[t * 128];
#pragma unroll
      for (int pt = 0; pt < NPT; ++pt) {
        u32x4 pr = aug;
        if (lane < 32) pr = *reinterpret_cast<const u32x4*>(lds + (pt * 32 + lane) * ROW + mi * 16);
        int run = 0x7FFFFFFF;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const f32x16 z = {};
          const f32x16 a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, cw[t]),
                                                                   __builtin_bit_cast(bf16x8, pr), z, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int v = __float_as_int(a[r]);
            run = v < run ? v : run;
          }
        }
        const int o = __shfl_xor(run, 32);
        sum[pt] += (int)__int_as_float(o < run ? o : run) - kOff;
      }
    }
  }
#pragma unroll
  for (int pt = 0; pt < NPT; ++pt)
    if (lane < 32) atomicAdd(&smin[pt * 32 + lane], (unsigned long long)sum[pt]);
  __syncthreads();
  for (int g = tid; g < G; g += kBaseNT)
    if (sp[g] >= 0) {
      b.pbase[i0 + g] = (int64_t)smin[g] + srr[g];
      b.dq2[i0 + g] = srr[g];
    }
}

// FP32 policy: a lower bound of every pair's in-order FP32 sums, as the key
// the queue compares with the phase-1 bound.  The FP32 LUT of a pair takes 8
// dependent FMAs per entry on the VALU, and most pairs need it only to be
// found dead (26 of 27 at 4999 x 32 pairs, d 128, M 16: the full scan of that
// batch took 2546 us and takes 190 without them; these bounds take 49).  Here
// |r|^2 + |c|^2 - 2 r . c of a 32 x 32 tile comes from two BF16 MFMAs of the
// operands split into high and low parts (lo . lo left out), with |c|^2 and
// |r|^2 in three pieces each; bound by the matrix unit, 64 clocks per 1024
// entries (9 us at that size), and by the residual rows read and split.
// Errors, in units of |r_m|^2 + max_j |c_mj|^2 of a subspace: the split
// 3 * 2^-18 (2 |r| |c| <= |r|^2 + |c|^2), |r|^2 from the rounded parts 2^-17,
// accumulation 20 terms * 2^-23 * 2, the scan's own entry 24 * 2^-24 and its
// sum M * 2^-23: together below 2^-15 + M * 2^-23, and twice that is taken
// off the sum.  A minimum by integer order takes a negative value nearest to
// zero, off by at most the same error.  A sum or slack that is not finite (or
// near overflow) gives key 0: the scan decides.  The scan still tests the
// exact bound of the pairs that pass.
struct BaseL2FArgs {
  const float* Q;
  const float* C;
  const u32x4* bswf;
  const int32_t* probes;
  int64_t* pbase;        // [nq][npmax] keys
  int nq, d, M, dsub, npmax;
};

constexpr int base_l2f_row() { return kBaseCM * 32 + 16; }  // high and low halves side by side, padded
constexpr int kBaseRr = kBaseCM + 1;                        // |r_m|^2 row, padded
inline size_t base_l2f_lds(int npt) {
  return (size_t)npt * 32 * (base_l2f_row() + kBaseRr * 4 + 4 * (kBaseNT / 64 + 3));
}

template <int NPT>
__global__ __launch_bounds__(kBaseNT, 4) void k_base_l2f(BaseL2FArgs b) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int G = NPT * 32, ROW = base_l2f_row(), NW = kBaseNT / 64, RU = NPT < 2 ? NPT : 2;
  float* rr = reinterpret_cast<float*>(lds + G * ROW);  // [G][kBaseRr]
  float* part = rr + G * kBaseRr;                       // [NW][G] sums of the waves
  float* srr = part + NW * G;                           // [G] sum of |r|^2
  int32_t* sp = reinterpret_cast<int32_t*>(srr + G);
  int32_t* sq = sp + G;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = tid & 15, grp = tid >> 4;
  const size_t n = (size_t)b.nq * b.npmax, i0 = (size_t)blockIdx.x * G;
  for (int g = tid; g < G; g += kBaseNT) {
    const size_t i = i0 + g;
    sp[g] = i < n ? b.probes[i] : -1;
    sq[g] = i < n ? (int)(i / b.npmax) : 0;
    srr[g] = 0.f;
  }
  const int ds = b.dsub;
  if (ds != 8 && ds != 4)  // element-wise rows: the padding stays zero
    for (int i = tid; i < G * ROW / 16; i += kBaseNT) reinterpret_cast<u32x4*>(lds)[i] = (u32x4){0u, 0u, 0u, 0u};
  float sum[NPT];
#pragma unroll
  for (int t = 0; t < NPT; ++t) sum[t] = 0.f;
  for (int m0 = 0; m0 < b.M; m0 += kBaseCM) {
    const int cm = b.M - m0 < kBaseCM ? b.M - m0 : kBaseCM;
    const int cd4 = (cm * ds) >> 2, o4 = (m0 * ds) >> 2;
    __syncthreads();
#pragma unroll RU
    for (int u = 0; u < NPT; ++u) {
      const int g = grp + u * (kBaseNT / 16);
      const int p = sp[g] < 0 ? 0 : sp[g];
      const float4* qr = reinterpret_cast<const float4*>(b.Q + (size_t)sq[g] * b.d) + o4;
      const float4* cr = reinterpret_cast<const float4*>(b.C + (size_t)p * b.d) + o4;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t4 = l16 + 16 * h;
        if (t4 >= cd4) break;
        const float4 x = qr[t4], c = cr[t4];
        const float v[4] = {-2.f * (x.x - c.x), -2.f * (x.y - c.y), -2.f * (x.z - c.z), -2.f * (x.w - c.w)};
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float r;
          hi[k] = bf16_rn(v[k], r);
          lo[k] = bf16_rn(r, r);
        }
        char* row = lds + g * ROW;
        if (ds == 8) {
          char* w = row + (t4 >> 1) * 32 + (t4 & 1) * 8;
          *reinterpret_cast<u32x2*>(w) = (u32x2){hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
          *reinterpret_cast<u32x2*>(w + 16) = (u32x2){lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
        } else if (ds == 4) {
          char* w = row + t4 * 32;
          *reinterpret_cast<u32x4*>(w) = (u32x4){hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16), 0u, 0u};
          *reinterpret_cast<u32x4*>(w + 16) = (u32x4){lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16), 0u, 0u};
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int t = 4 * t4 + k;
            char* w = row + (t / ds) * 32 + (t % ds) * 2;
            *reinterpret_cast<uint16_t*>(w) = (uint16_t)hi[k];
            *reinterpret_cast<uint16_t*>(w + 16) = (uint16_t)lo[k];
          }
        }
      }
    }
    __syncthreads();
    // |r_m|^2 from the split parts
    for (int e = tid; e < G * cm; e += kBaseNT) {
      const int g = e / cm, mi = e - g * cm;
      const u32x4 h = *reinterpret_cast<const u32x4*>(lds + g * ROW + mi * 32);
      const u32x4 l = *reinterpret_cast<const u32x4*>(lds + g * ROW + mi * 32 + 16);
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float a = __uint_as_float(h[k] << 16) + __uint_as_float(l[k] << 16);
        const float c = __uint_as_float(h[k] & 0xFFFF0000u) + __uint_as_float(l[k] & 0xFFFF0000u);
        s = fmaf(a, a, s);
        s = fmaf(c, c, s);
      }
      rr[g * kBaseRr + mi] = 0.25f * s;  // (the parts are those of -2 r)
    }
    __syncthreads();
    if (tid < G) {
      float s = srr[tid];
      for (int mi = 0; mi < cm; ++mi) s += rr[tid * kBaseRr + mi];
      srr[tid] = s;
    }
    for (int mi = wave; mi < cm; mi += NW) {
      int run[NPT];
#pragma unroll
      for (int t = 0; t < NPT; ++t) run[t] = 0x7FFFFFFF;
      // four codeword tiles at a time: their fragments stay in 32 registers
#pragma unroll
      for (int th = 0; th < 2; ++th) {
        const u32x4* src = b.bswf + (size_t)((m0 + mi) * 8 + th * 4) * 128 + lane;
        u32x4 c0[4], c1[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          c0[t] = src[t * 128];
          c1[t] = src[t * 128 + 64];
        }
#pragma unroll
        for (int pt = 0; pt < NPT; ++pt) {
          const int g = pt * 32 + (lane & 31);
          const u32x4 p0 = *reinterpret_cast<const u32x4*>(lds + g * ROW + mi * 32);
          float r = rr[g * kBaseRr + mi];
          const uint32_t r0 = bf16_rn(r, r), r1 = bf16_rn(r, r), r2 = bf16_rn(r, r);
          u32x4 p1 = {0x3F803F80u, 0x00003F80u | (r0 << 16), r1 | (r2 << 16), 0u};  // for the pieces of |c|^2: ones
          if (lane < 32) p1 = *reinterpret_cast<const u32x4*>(lds + g * ROW + mi * 32 + 16);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            f32x16 a = {};
            a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, c0[t]),
                                                        __builtin_bit_cast(bf16x8, p0), a, 0, 0, 0);
            a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, c1[t]),
                                                        __builtin_bit_cast(bf16x8, p1), a, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
              const int v = __float_as_int(a[k]);
              run[pt] = v < run[pt] ? v : run[pt];
            }
            // (an opaque step: reassociated into one tree, the minima would
            // keep every tile's accumulators alive)
            asm volatile("" : "+v"(run[pt]));
          }
        }
      }
#pragma unroll
      for (int pt = 0; pt < NPT; ++pt) {
        const int o = __shfl_xor(run[pt], 32);
        sum[pt] += __int_as_float(o < run[pt] ? o : run[pt]);
      }
    }
  }
#pragma unroll
  for (int pt = 0; pt < NPT; ++pt)
    if (lane < 32) part[wave * G + pt * 32 + lane] = sum[pt];
  __syncthreads();
  const float cbsum = *reinterpret_cast<const float*>(b.bswf + (size_t)b.M * 1024);
  for (int g = tid; g < G; g += kBaseNT)
    if (sp[g] >= 0) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += part[w * G + g];
      const float mag = srr[g] + cbsum;
      // (the absolute term covers squares that underflow)
      const float lb = s - (mag * (0x1p-14f + (float)b.M * 0x1p-22f) + (float)b.M * 1e-30f);
      const bool ok = mag < 1e37f && lb > -3e38f && lb < 3e38f;  // false for NaN
      b.pbase[i0 + g] = ok ? (int64_t)fkey(lb) : 0;
    }
}

// ------------------------------------------------------------------ host launchers
template <typename K>
static void* kaddr(K k) { return reinterpret_cast<void*>(k); }

// dynamic LDS limit of a kernel raised to `bytes` (only ever raised; the
// runtime call takes microseconds of a launch-bound search, so what a kernel
// has been given on a device is remembered)
static hipError_t set_lds(const void* fn, size_t bytes) {
  struct Slot {
    const void* fn;
    int dev;
    size_t bytes;
  };
  static std::mutex mu;
  static Slot slots[512];
  static int n = 0;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  Slot* s = nullptr;
  for (int i = 0; i < n && !s; ++i)
    if (slots[i].fn == fn && slots[i].dev == dev) s = &slots[i];
  if (s && bytes <= s->bytes) return hipSuccess;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  if (!s && n < 512) {
    s = &slots[n++];
    s->fn = fn;
    s->dev = dev;
  }
  if (s) s->bytes = bytes;
  return hipSuccess;
}

// workgroups per CU of a kernel at a block size and dynamic LDS (remembered
// likewise)
static hipError_t blocks_per_cu(int* out, const void* fn, int nt, size_t lds) {
  struct Slot {
    const void* fn;
    int dev, nt, blocks;
    size_t lds;
  };
  static std::mutex mu;
  static Slot slots[512];
  static int n = 0;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  for (int i = 0; i < n; ++i)
    if (slots[i].fn == fn && slots[i].dev == dev && slots[i].nt == nt && slots[i].lds == lds) {
      *out = slots[i].blocks;
      return hipSuccess;
    }
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(out, fn, nt, lds)) != hipSuccess) return e;
  if (n < 512) slots[n++] = Slot{fn, dev, nt, *out, lds};
  return hipSuccess;
}

hipError_t launch_prep_index(const amp_index* ix, hipStream_t st) {
  const DeviceIndex& dv = ix->dev;
  hipLaunchKernelGGL(k_sqnorm, dim3((ix->nlist + 3) / 4), dim3(256), 0, st, dv.centroids, ix->nlist,
                     ix->d, dv.cnorm);
  const int total = (ix->M / 2) * 16 * 64;
  hipLaunchKernelGGL(k_prep_cbi, dim3((ix->M * kKsub * 8 + 255) / 256), dim3(256), 0, st, dv.codebook, ix->M,
                     ix->dsub, ix->grid_e, ix->grid_kind, dv.cbi16);
  const size_t nc = (size_t)ix->nlist * ix->d;
  hipLaunchKernelGGL(k_qgrid, dim3((unsigned)std::min<size_t>((nc + 255) / 256, 65536)), dim3(256), 0, st,
                     dv.centroids, dv.ci16, nc, ix->grid_e, ix->grid_kind);
  hipLaunchKernelGGL(k_prep_bsw, dim3((total + 255) / 256), dim3(256), 0, st, dv.codebook, ix->M, ix->dsub,
                     ix->grid_e, ix->grid_kind, reinterpret_cast<u32x4*>(dv.bsw),
                     reinterpret_cast<u32x4*>(dv.bsw16), reinterpret_cast<u32x2*>(dv.bsw8));
  if (ix->metric == AMP_L2) {
    u32x4* f = reinterpret_cast<u32x4*>(dv.bswf);
    hipLaunchKernelGGL(k_prep_bswf, dim3((ix->M * 512 + 255) / 256), dim3(256), 0, st, dv.codebook, ix->M, ix->dsub, f);
    hipLaunchKernelGGL(k_prep_cbsum, dim3(1), dim3(256), 0, st, dv.codebook, ix->M, ix->dsub,
                       reinterpret_cast<float*>(f + (size_t)ix->M * 1024));
  }
  return hipGetLastError();
}

// dynamic LDS of a scan launch (lw_bits -1: the mixed-class kernel), the
// layout the kernel computes for itself
static size_t scan_lds_bytes(int lw_bits, int phase, int M, int d, int wpr, int nt) {
  const bool fp = lw_bits == 0;
  const int cw = lw_bits < 0 ? wpr : class_wpr(lw_bits, wpr);
  return (size_t)scan_lds_layout(unit_pairs(lw_bits, wpr), cw, M, d, fp, phase, nt).total;
}

int scan_wpr(int M, bool fp32, int lut_dtype, bool narrow) {
  return narrow ? 1 : kernel_wpr(scan_mt(fp32 ? 0 : 8, M, dt_of(lut_dtype)));
}

static int g_num_cu = 0;

// lwb < 0: every integer lane class in one launch (k_scan_mix).  A LUT tile
// so large that one 256-thread workgroup fills a CU's LDS leaves one wave
// per SIMD to hide the LDS and code-load latencies: the generic variant then
// runs 512-thread workgroups (two waves per SIMD on the same LUT;
// AMP_SCAN_WG512=0 keeps 256).
static hipError_t launch_scan(int lwb, int ph, int dt, int wpr, const ScanArgs& sa, int64_t max_units,
                              hipStream_t st) {
  const bool mix = lwb < 0;
  if (lwb == 0) dt = sa.metric == AMP_IP && wpr == 1 ? DT_TAB : DT_BF16;
  auto pick = [&](int nt) {
    return ph == 1 ? pick_scan_ph1(lwb, sa.M, dt, wpr, nt)
                   : (ph == 2 ? pick_scan_ph2(lwb, sa.M, dt, wpr, nt) : pick_scan_ph3(lwb, sa.M, dt, wpr, nt));
  };
  ScanFn fn = pick(kThreads);
  int nt = kThreads;
  // the queue packed units for `wpr` words per row: the variant must agree
  const int mt = scan_mt(mix ? 8 : lwb, sa.M, dt);
  if (!fn || variant_wpr(mt, scan_nr(mt, wpr)) != wpr) return hipErrorInvalidValue;
  size_t lds = scan_lds_bytes(lwb, ph, sa.M, sa.d, wpr, nt);
  hipError_t e = set_lds(kaddr(fn), lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = blocks_per_cu(&per_cu, kaddr(fn), nt, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) return hipErrorInvalidConfiguration;
  static const bool wg512 = [] {
    const char* v = getenv("AMP_SCAN_WG512");
    return !(v && v[0] == '0');
  }();
  if (per_cu == 1 && wg512) {
    ScanFn f2 = pick(2 * kThreads);
    if (f2) {
      const size_t l2 = scan_lds_bytes(lwb, ph, sa.M, sa.d, wpr, 2 * kThreads);
      int pc2 = 0;
      if ((e = set_lds(kaddr(f2), l2)) != hipSuccess)
        return e;
      if ((e = blocks_per_cu(&pc2, kaddr(f2), 2 * kThreads, l2)) != hipSuccess)
        return e;
      if (pc2 >= 1) {
        fn = f2;
        nt = 2 * kThreads;
        lds = l2;
        per_cu = pc2;
      }
    }
  }
  if (!g_num_cu) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&g_num_cu, hipDeviceAttributeMultiprocessorCount, dev);
  }
  // phase 3 (the re-run) usually has nothing to do: one workgroup per CU.  No
  // more workgroups than units: each claims from one counter before it finds
  // the queue drained (8 queries, nprobe 32, copied FP32 LUT of M 8: phases 1 and 2
  // in 22.8 and 26.9 us with the 2048 workgroups that fit the chip, in 9.4 and
  // 12.6 with 256, the pairs)
  const int64_t wgs = (int64_t)g_num_cu * (ph == 3 ? 1 : per_cu);
  hipLaunchKernelGGL(fn, dim3((unsigned)std::max<int64_t>(1, std::min(wgs, max_units))), dim3(nt), lds, st, sa);
  return hipGetLastError();
}

hipError_t launch_assign(const float* X, int64_t n, int dd, int ld, const float* C, int k, float* xn, float* cn,
                         int32_t* out_a, float* out_d, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sqnorm_ld, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, X, n, dd, ld, xn);
  hipLaunchKernelGGL(k_sqnorm_ld, dim3((unsigned)((k + 3) / 4)), dim3(256), 0, st, C, (int64_t)k, dd, dd, cn);
  hipLaunchKernelGGL(k_assign, dim3((unsigned)((n + CL_T - 1) / CL_T)), dim3(256), 0, st, X, xn, n, dd, ld, C, cn, k,
                     out_a, out_d);
  return hipGetLastError();
}

hipError_t launch_sqnorm(const float* X, int64_t n, int dd, float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sqnorm_ld, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, X, n, dd, dd, out);
  return hipGetLastError();
}

hipError_t launch_residual(const float* X, const int32_t* a, const float* C, int64_t n, int d, float* out,
                           hipStream_t st) {
  const int64_t total = n * d;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_residual, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X, a, C, n, d, out);
  return hipGetLastError();
}

// as many pairs per workgroup (128 at most: they share the codeword
// fragments, M * 8 KB from L2) as leave three workgroups for two CUs.  With
// 32 / 64 / 128 / 256 pairs: 110 / 87 / 76 / 76 us at 10000 x 32 pairs,
// d 128, M 16; 165 / 143 / 136 / 182 us at 1000 x 64, d 960, M 120 (500
// workgroups of 128); 211 / 166 / 145 / 144 us at 4096 x 8..128, d 96, M 24.
// (The 16x16x32 tiles before, with the residual's operand converted for every
// tile and a cross-lane reduction per 16 codewords: 231, 640 and 480 us, and
// the predictor read the same rows again: 41 -> 19, 96 -> 12, 194 -> 168 us.)
static int base_l2_npt(size_t n) {
  int npt = 4;
  while (npt > 1 && n < (size_t)npt * 32 * 384) npt >>= 1;
  return npt;
}

static hipError_t launch_base_l2(const BaseL2Args& b, hipStream_t st) {
  const size_t n = (size_t)b.nq * b.npmax;
  const int npt = base_l2_npt(n);
  auto fn = npt == 4 ? k_base_l2<4> : (npt == 2 ? k_base_l2<2> : k_base_l2<1>);
  const size_t lds = base_l2_lds(npt);
  const hipError_t e = set_lds(kaddr(fn), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fn, dim3((unsigned)((n + npt * 32 - 1) / (npt * 32))), dim3(kBaseNT), lds, st, b);
  return hipGetLastError();
}

static hipError_t launch_base_l2f(const BaseL2FArgs& b, hipStream_t st) {
  const size_t n = (size_t)b.nq * b.npmax;
  const int npt = base_l2_npt(n);
  auto fn = npt == 4 ? k_base_l2f<4> : (npt == 2 ? k_base_l2f<2> : k_base_l2f<1>);
  const size_t lds = base_l2f_lds(npt);
  const hipError_t e = set_lds(kaddr(fn), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fn, dim3((unsigned)((n + npt * 32 - 1) / (npt * 32))), dim3(kBaseNT), lds, st, b);
  return hipGetLastError();
}

hipError_t launch_search(const amp_index* ix, const Workspace& ws, const float* queries_in, const SearchDims& sd,
                         const ModelArgs& ma, const ModelArgs& clma, int64_t* out_ids, float* out_dist,
                         int64_t* out_qdist,
                         float* out_coarse, hipStream_t st, hipEvent_t* ev) {
  const DeviceIndex& dv = ix->dev;
  const bool fp32 = sd.policy == AMP_POLICY_FP32;
  const int ncls = fp32 ? 1 : kNCls;
  const int NB = ncls * sd.nlist;
  const size_t npairs = (size_t)sd.nq * sd.npmax;
  auto mark = [&](int i) { if (ev) (void)hipEventRecord(ev[i], st); };
  mark(0);
  const bool ipm = sd.metric == AMP_IP;
  const float* queries = sd.q_bf16 ? sd.q_conv : queries_in;
  // small batches: launches fused where latency and launch gaps are the cost
  const int64_t min_chunk = std::min(sd.chunk, sd.chunk1);
  const bool small_q = npairs <= (size_t)kSmallQueue && NB <= kSmallBuckets &&
                       (ix->max_list + min_chunk - 1) / min_chunk < (1 << 17);  // (32-bit unit offsets)
  const bool small_b = sd.nq <= kSmallBatch;
  {
    FrontArgs f{};
    f.cnt = reinterpret_cast<uint32_t*>(ws.cnt);
    f.ncnt = small_q ? 0 : (size_t)2 * kQSub * NB;
    f.counters = ws.counters;
    f.ncounters = (size_t)2 * (kNCls + 1) * kQueueSlot;
    f.flags = reinterpret_cast<uint32_t*>(ws.flags);
    f.work = ws.work;
    f.tau = ws.tau;
    f.ccount = ws.ccount;
    f.ipmask = ipm ? ws.ipmask : nullptr;
    f.ipspan = ws.ipspan;
    f.iplsum = ws.iplsum;
    f.kin = sd.k_dev;
    f.npin = sd.np_dev;
    f.kout = ws.kq;
    f.npout = ws.npq;
    f.kmax = sd.kmax;
    f.npmax = sd.npmax;
    f.q = queries_in;
    f.qb = sd.q_bf16;
    f.qw = sd.q_conv;
    // (coarse distances of L2; pair bounds of the FP32 policy under inner product)
    f.qn = sd.cl_policy == AMP_CL_FP32 && (sd.metric == AMP_L2 || (ipm && fp32)) ? ws.qnorm : nullptr;
    f.qi = ipm && !fp32 ? ws.qi16 : nullptr;  // (predictor, table build, pair bases)
    f.rows = f.qb || f.qn || f.qi;
    f.nq = sd.nq;
    f.d = sd.d;
    f.grid_e = sd.grid_e;
    f.grid_kind = sd.grid_kind;
    const unsigned fb = (unsigned)std::min<size_t>(std::max<size_t>(((size_t)sd.nq + 3) / 4, 64 + f.ncnt / 4096), 16384);
    hipLaunchKernelGGL(k_front, dim3(fb), dim3(256), 0, st, f);
    if (f.kin && sd.nq > kFrontSizes)
      hipLaunchKernelGGL(k_sizes, dim3((sd.nq + 255) / 256), dim3(256), 0, st, f);
  }
  // CL
  float* coarse = out_coarse ? out_coarse : ws.coarse;
  if (sd.cl_policy != AMP_CL_FP32) {
    // integer cluster locating on 8-bit codes (fixed or adaptive operand
    // widths): order keys of the exact integer distances
    const hipError_t e = launch_cl(ix, ws, queries, sd, clma, ws.coarse, st);
    if (e != hipSuccess) return e;
    coarse = ws.coarse;
  } else if (sd.metric == AMP_L1) {
    hipLaunchKernelGGL(k_coarse_l1, dim3((sd.nlist + CL_T - 1) / CL_T, (sd.nq + CL_T - 1) / CL_T), dim3(256), 0,
                       st, queries, dv.centroids, coarse, sd.nq, sd.nlist, sd.d);
  } else {
    const dim3 g((sd.nlist + CL_T - 1) / CL_T, (sd.nq + CL_T - 1) / CL_T);
    const bool vec = sd.d % 4 == 0 && ((reinterpret_cast<uintptr_t>(queries) | reinterpret_cast<uintptr_t>(dv.centroids)) & 15) == 0;
    // (64-wide K chunks measured the same as 32 at 4096 x 2048 x 768)
    if (vec)
      hipLaunchKernelGGL((k_coarse<CL_K, true>), g, dim3(256), 0, st, queries, dv.centroids, ws.qnorm, dv.cnorm, coarse,
                         sd.nq, sd.nlist, sd.d, sd.metric);
    else
      hipLaunchKernelGGL((k_coarse<CL_K, false>), g, dim3(256), 0, st, queries, dv.centroids, ws.qnorm, dv.cnorm,
                         coarse, sd.nq, sd.nlist, sd.d, sd.metric);
  }
  mark(1);
  int np2 = 1;
  while (np2 < sd.nlist) np2 <<= 1;
  // (a wave per query counts a row by itself, a workgroup splits it: one query
  // over 1024 lists 13.7 against 7.8 us; whole searches 102 against 96 us for
  // one query, 260 / 252 for 1024, 294 / 287 for 2048, 368 / 367 for 4096, 575 /
  // 580 for 10000; over 256 lists they are even at 256 to 1024 queries and 241 /
  // 249 at 4096.  Workgroups take four times the waves, which counts beside
  // another stream's search: 2000 queries on three streams, 300 lists 122.7 / 123.8
  // us, 512 lists 143.3 / 144.9 and, FP32 under L1, 821 / 857, 1024 lists 204.6 /
  // 203.9; 1000 queries even, 300 queries over 512 lists 74.4 / 73.9)
  const int topn_wg = sd.nlist > 512 ? 2048 : 1024;
  if (sd.npmax <= 64 && sd.nlist <= 1024 && (sd.nq > topn_wg || sd.nlist <= 256)) {
    const dim3 g((sd.nq + 3) / 4), b(256);
    const int32_t* npq = ws.npq ? ws.npq : nullptr;
    if (sd.nlist <= 64)
      hipLaunchKernelGGL(k_topn_wave<1>, g, b, 0, st, coarse, sd.nlist, sd.nq, npq, sd.npconst, sd.npmax, ws.probes);
    else if (sd.nlist <= 128)
      hipLaunchKernelGGL(k_topn_wave<2>, g, b, 0, st, coarse, sd.nlist, sd.nq, npq, sd.npconst, sd.npmax, ws.probes);
    else if (sd.nlist <= 256)
      hipLaunchKernelGGL(k_topn_wave<4>, g, b, 0, st, coarse, sd.nlist, sd.nq, npq, sd.npconst, sd.npmax, ws.probes);
    else if (sd.nlist <= 512)
      hipLaunchKernelGGL(k_topn_wave<8>, g, b, 0, st, coarse, sd.nlist, sd.nq, npq, sd.npconst, sd.npmax, ws.probes);
    else
      hipLaunchKernelGGL(k_topn_wave<16>, g, b, 0, st, coarse, sd.nlist, sd.nq, npq, sd.npconst, sd.npmax, ws.probes);
  } else if (sd.nlist <= 4096) {
    const int32_t* npq = ws.npq ? ws.npq : nullptr;
    const size_t lds = np2 * sizeof(uint64_t);
    if (sd.nlist <= 1024)
      hipLaunchKernelGGL(k_topn_wg<4>, dim3(sd.nq), dim3(256), lds, st, coarse, sd.nlist, npq, sd.npconst, sd.npmax,
                         ws.probes);
    else if (sd.nlist <= 2048)
      hipLaunchKernelGGL(k_topn_wg<8>, dim3(sd.nq), dim3(256), lds, st, coarse, sd.nlist, npq, sd.npconst, sd.npmax,
                         ws.probes);
    else
      hipLaunchKernelGGL(k_topn_wg<16>, dim3(sd.nq), dim3(256), lds, st, coarse, sd.nlist, npq, sd.npconst,
                         sd.npmax, ws.probes);
  } else {
    hipLaunchKernelGGL(k_topn, dim3(sd.nq), dim3(256), np2 * sizeof(uint64_t), st, coarse, sd.nlist, np2,
                       ws.npq ? ws.npq : nullptr, sd.npconst, sd.npmax, ws.probes);
  }
  mark(2);
  const int dt = dt_of(sd.lut_dtype);
  // lower bounds of the pairs' estimates (integer policies: the exact bases):
  // the full scan's queue is built after the phase-1 bound and leaves out the
  // pairs whose bound exceeds it.  (The FP32 policy under L1 tests its bound
  // inside the scan, after its LUT.)
  const bool early = (!fp32 || sd.metric != AMP_L1) && !sd.noskip;
  // L2, exact LUT builds: the base kernel reads every pair's rows and leaves
  // d' for the predictor, so it runs first (in the rank array, which the
  // queue fills later); the caller's stage times are put in order again
  const bool base_first = sd.metric == AMP_L2 && !fp32 && dt != DT_F8 && early;
  if (base_first) {
    BaseL2Args bl;
    bl.Q = queries;
    bl.C = dv.centroids;
    bl.bsw = reinterpret_cast<const u32x4*>(dv.bsw);
    bl.probes = ws.probes;
    bl.pbase = ws.pbase;
    bl.dq2 = reinterpret_cast<int64_t*>(ws.rank);
    bl.nq = sd.nq;
    bl.d = sd.d;
    bl.M = sd.M;
    bl.dsub = sd.dsub;
    bl.npmax = sd.npmax;
    bl.grid_e = sd.grid_e;
    bl.grid_kind = sd.grid_kind;
    const hipError_t e = launch_base_l2(bl, st);
    if (e != hipSuccess) return e;
    mark(3);
  }
  // PPM
  PairArgs pa;
  pa.Q = queries;
  pa.C = dv.centroids;
  pa.qi16 = (ipm && !fp32) ? ws.qi16 : nullptr;
  pa.ci16 = dv.ci16;
  const bool pdot = ipm && !fp32 && sd.policy == AMP_POLICY_ADAPTIVE;
  pa.dq2_in = base_first ? reinterpret_cast<const int64_t*>(ws.rank) : nullptr;
  pa.dot_out = pdot ? ws.pbase : nullptr;
  pa.ipmask = pdot ? ws.ipmask : nullptr;
  pa.probes = ws.probes;
  pa.radq = dv.radq;
  pa.offsets = dv.offsets;
  pa.xbits = ws.xbits;
  pa.pbits = ws.pbits;
  pa.nq = sd.nq;
  pa.d = sd.d;
  pa.npmax = sd.npmax;
  pa.grid_e = sd.grid_e;
  pa.grid_kind = sd.grid_kind;
  pa.metric = sd.metric;
  pa.policy = sd.policy;
  pa.fixed_bits = sd.fixed_bits;
  pa.lane_sel_M = sd.M;
  pa.allowed = sd.allowed_mask;
  pa.margin = sd.margin;
  pa.lg_npp = 0;
  while ((1 << pa.lg_npp) < sd.npmax) ++pa.lg_npp;
  // threads per pair: more for batches too small to fill the chip (about
  // 2^17 threads), at most 64 and at most one query per workgroup
  pa.lg_T = 0;
  while (pa.lg_T < 6 && pa.lg_npp + pa.lg_T < 8 && ((int64_t)sd.nq << (pa.lg_npp + pa.lg_T + 1)) <= (1 << 17))
    ++pa.lg_T;
  const int qpb = 256 >> (pa.lg_npp + pa.lg_T);
  hipLaunchKernelGGL(k_pairs, dim3((sd.nq + qpb - 1) / qpb), dim3(256), 0, st, pa, ma);
  mark(base_first ? 4 : 3);
  hipError_t err = hipSuccess;
  if (!base_first) {
    BaseArgs ba;
    ba.Q = queries;
    ba.C = dv.centroids;
    ba.bsw = reinterpret_cast<const u32x4*>(dv.bsw);
    ba.bsw16 = reinterpret_cast<const u32x4*>(dv.bsw16);
    ba.bsw8 = reinterpret_cast<const u32x2*>(dv.bsw8);
    ba.cbi16 = dv.cbi16;
    ba.ci16 = dv.ci16;
    ba.probes = ws.probes;
    ba.pbase = ws.pbase;
    ba.qi16 = ws.qi16;
    ba.iptab = ws.iptab;
    ba.iplo = ws.iplo;
    ba.ipspan = ws.ipspan;
    ba.iplsum = ws.iplsum;
    ba.iptq = ws.iptq;
    ba.ipsh = ws.ipsh;
    ba.ipmask = ws.ipmask;
    ba.pbits = ws.pbits;
    ba.codebook = dv.codebook;
    ba.nq = sd.nq;
    ba.d = sd.d;
    ba.M = sd.M;
    ba.dsub = sd.dsub;
    ba.npmax = sd.npmax;
    ba.grid_e = sd.grid_e;
    ba.grid_kind = sd.grid_kind;
    ba.metric = sd.metric;
    ba.gran = sd.gran;
    if (fp32 && sd.metric == AMP_L2 && early) {
      BaseL2FArgs bf;
      bf.Q = queries;
      bf.C = dv.centroids;
      bf.bswf = reinterpret_cast<const u32x4*>(dv.bswf);
      bf.probes = ws.probes;
      bf.pbase = ws.pbase;
      bf.nq = sd.nq;
      bf.d = sd.d;
      bf.M = sd.M;
      bf.dsub = sd.dsub;
      bf.npmax = sd.npmax;
      if ((err = launch_base_l2f(bf, st)) != hipSuccess) return err;
    } else if (ipm && fp32) {
      // the queries' FP32 dot-product tables, their row maxima, the pairs'
      // FP32 lower bounds
      static_assert(kMaxDsub == 8, "a table kernel per subspace width");
      constexpr decltype(&k_iptab_f32<1>) kTab[kMaxDsub] = {k_iptab_f32<1>, k_iptab_f32<2>, k_iptab_f32<3>,
                                                            k_iptab_f32<4>, k_iptab_f32<5>, k_iptab_f32<6>,
                                                            k_iptab_f32<7>, k_iptab_f32<8>};
      const auto tab = kTab[sd.dsub - 1];
      // (y ends at 65535 workgroups, 2.1M queries; subspaces on x, so that
      // neighbouring workgroups write neighbouring rows: 1024 queries, d 768, M 96,
      // 35.8 us, with the query groups on x 37.4)
      const unsigned tg = (unsigned)((sd.nq + kTabF - 1) / kTabF), tz = (tg + 65534) / 65535;
      hipLaunchKernelGGL(tab, dim3((unsigned)sd.M, (tg + tz - 1) / tz, tz), dim3(256), 0, st, ba);
      if (sd.cl_policy == AMP_CL_FP32)
        hipLaunchKernelGGL(k_ipbound_f32, dim3((unsigned)sd.nq), dim3(256), 0, st, ba, coarse, ws.qnorm, dv.cnorm,
                           sd.nlist);
      else
        hipLaunchKernelGGL(k_ipbase_f32, dim3((unsigned)((npairs + 3) / 4)), dim3(256), 0, st, ba);
    } else if (ipm) {
      // the pairs' qi.ci and the widths each query needs, then the queries'
      // tables with their minima (and the pair bases), then the quantised tables
      const size_t tlds = base_lds_layout(kTabQ, sd.M, sd.d).total;
      auto fn = dt == DT_F16 ? k_iptab<DT_F16> : (dt == DT_F8 ? k_iptab<DT_F8> : k_iptab<DT_BF16>);
      if ((err = set_lds(kaddr(fn), tlds)) != hipSuccess)
        return err;
      // (adaptive: the predictor pass wrote qi.ci and the width masks)
      if (sd.policy != AMP_POLICY_ADAPTIVE)
        hipLaunchKernelGGL(k_ipbase, dim3((unsigned)sd.nq), dim3(256), 0, st, ba);
      // (at least four m-pairs, one per wave, and no more workgroups than twice the chip)
      const int groups = (sd.nq + kTabQ - 1) / kTabQ, ys = std::max(1, std::min(512 / groups, sd.M / 8));
      const int mps = (((sd.M / 2 + ys - 1) / ys) + 3) & ~3;
      hipLaunchKernelGGL(fn, dim3(groups, (sd.M / 2 + mps - 1) / mps), dim3(kThreads), tlds, st, ba, mps);
      const size_t nq8 = (size_t)sd.nq * sd.M * kKsub / 8;
      hipLaunchKernelGGL(k_ipq, dim3((unsigned)std::min<size_t>((nq8 + 255) / 256, 1 << 20)), dim3(256), 0, st, ba);
    } else if (early && !fp32) {
      // FP8 build: every pair's LUT minima, as many pairs per workgroup as fit
      // 64 KB of residual rows (128 at most): they share the B fragments.  L1
      // shares nothing: 32 pairs, for enough workgroups to spread over the chip
      // (whole searches with 32 / 128, us alone and on three streams: 700 queries,
      // nprobe 32, M 16, d 80, 436 / 502 and 267 / 306; 8000, nprobe 16, M 16, d 64,
      // 1535 / 1760 and 1264 / 1304; 2000, nprobe 32, d 64, 4 bits, 850 / 851 and
      // 580 / 546; M 96, d 384, 3600 / 3757 and 3314 / 3488, there with 64)
      int G = sd.metric == AMP_L1 ? 32 : 128;
      while (G > 8 && (size_t)G * ri_stride(sd.d) * 2 > 65536) G >>= 1;
      ba.G = G;
      const size_t blds = base_lds_layout(G, sd.M, sd.d).total;
      auto fn = sd.metric == AMP_L1 ? k_base<true> : k_base<false>;
      if ((err = set_lds(kaddr(fn), blds)) != hipSuccess)
        return err;
      hipLaunchKernelGGL(fn, dim3((unsigned)((npairs + G - 1) / G)), dim3(kThreads), blds, st, ba);
    }
    mark(4);
  }
  // queue
  QueueArgs qa;
  qa.probes = ws.probes;
  qa.pbits = ws.pbits;
  qa.kq = ws.kq;
  qa.kconst = sd.kconst;
  qa.offsets = dv.offsets;
  qa.lorder = dv.lorder;
  qa.lpos = dv.lpos;
  qa.cnt = ws.cnt;
  qa.rank = ws.rank;
  qa.pairoff = ws.pairoff;
  qa.unitoff = ws.unitoff;
  qa.sorted = ws.sorted;
  qa.units = ws.units;
  qa.flags = ws.flags;
  qa.nq = sd.nq;
  qa.npmax = sd.npmax;
  qa.nlist = sd.nlist;
  qa.M = sd.M;
  qa.ncls = ncls;
  qa.gran = sd.gran;
  qa.wpr = sd.wpr;
  qa.chunk[0] = sd.chunk1;
  qa.chunk[1] = sd.chunk;
  qa.max_units = sd.max_units;
  qa.pbase = nullptr;
  qa.fkeys = 0;
  qa.all_offsets = getenv("AMP_STATS") != nullptr;
  qa.tau = ws.tau;
  qa.work = nullptr;
  const int qb = (int)((npairs + 255) / 256);
  // one build of the queue phases [ph0, ph1)
  auto build_queue = [&](int ph0, int ph1) -> hipError_t {
    QueueArgs q = qa;
    q.ph0 = ph0;
    q.ph1 = ph1;
    if (ph1 > 1 && early) {
      q.pbase = ws.pbase;
      q.fkeys = fp32 ? 1 : 0;
      q.work = sd.want_work ? ws.work : nullptr;
    }
    if (small_q) {
      // (few pairs and buckets: four waves to a barrier)
      const int nt = npairs <= 256 && NB <= 1024 ? 256 : 1024;
      const size_t qlds = (size_t)NB * 8 + npairs * 4;
      auto fn = npairs <= (size_t)nt ? k_queue_small<1>
                                     : (npairs <= 2048 ? k_queue_small<2> : k_queue_small<4>);
      const hipError_t e = set_lds(kaddr(fn), qlds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(fn, dim3(1), dim3(nt), qlds, st, q, fp32 ? 1 : 0);
      return hipGetLastError();
    }
    hipLaunchKernelGGL(k_qhist, dim3(qb), dim3(256), 0, st, q);
    hipLaunchKernelGGL(k_qtot, dim3(((ph1 - ph0) * NB + 255) / 256), dim3(256), 0, st, q, fp32 ? 1 : 0);
    if (NB <= kFewBuckets) {
      hipLaunchKernelGGL(k_qscan_few, dim3(1), dim3(1024), 0, st, q);
    } else {
      const size_t slds = (size_t)NB * 4;
      const hipError_t e = set_lds(kaddr(k_qscan), slds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(k_qscan, dim3(1), dim3(1024), slds, st, q);
    }
    hipLaunchKernelGGL(k_qscatter, dim3(qb), dim3(256), 0, st, q);
    hipLaunchKernelGGL(k_qunits, dim3(512), dim3(256), 0, st, q, fp32 ? 1 : 0);
    return hipGetLastError();
  };
  if ((err = build_queue(0, early ? 1 : 2)) != hipSuccess) return err;
  mark(5);
  // LC + DC, phase 1 then phase 2
  ScanArgs sa;
  sa.Q = queries;
  sa.C = dv.centroids;
  sa.codebook = dv.codebook;
  sa.bsw = reinterpret_cast<const u32x4*>(dv.bsw);
  sa.bsw16 = reinterpret_cast<const u32x4*>(dv.bsw16);
  sa.bsw8 = reinterpret_cast<const u32x2*>(dv.bsw8);
  sa.cbi16 = dv.cbi16;
  sa.codes = dv.codes;
  sa.ids = dv.ids;
  sa.offsets = dv.offsets;
  sa.kq = ws.kq;
  sa.pbits = ws.pbits;
  sa.tau = ws.tau;
  sa.ccount = ws.ccount;
  sa.ckey = ws.ckey;
  sa.cid = ws.cid;
  sa.flags = ws.flags;
  sa.nq = sd.nq;
  sa.d = sd.d;
  sa.M = sd.M;
  sa.dsub = sd.dsub;
  sa.nlist = sd.nlist;
  sa.npmax = sd.npmax;
  sa.grid_e = sd.grid_e;
  sa.grid_kind = sd.grid_kind;
  sa.metric = sd.metric;
  sa.gran = sd.gran;
  sa.noskip = sd.noskip;
  sa.kconst = sd.kconst;
  sa.kmax = sd.kmax;
  sa.chunk = sd.chunk;  // per phase below
  sa.capq = sd.capq;
  sa.tau_id = nullptr;
  sa.nrerun = nullptr;
  sa.work = nullptr;
  sa.steal = sd.queue;
  sa.iptab = ws.iptab;
  sa.iplo = ws.iplo;
  sa.iptq = ws.iptq;
  sa.ipsh = ws.ipsh;
  sa.pbase_g = ws.pbase;
  sa.tab_out = nullptr;
  // the lane classes run one after another on the caller's stream, each a
  // persistent kernel over its own unit range.  (Running them concurrently
  // on separate streams was measured slower on the mid-size workload: scan
  // phase 2 took 1.86 ms against 1.50 ms serially.)
  for (int ph = 1; ph <= 2; ++ph) {
    sa.sorted = ws.sorted + (ph == 2 ? npairs : 0);
    sa.unitoff = ws.unitoff + (ph == 2 ? (NB + 1) : 0);
    sa.units = ws.units + (ph == 2 ? sd.max_units : 0);
    sa.chunk = ph == 2 ? sd.chunk : sd.chunk1;
    int sa_lwb;
    if (fp32 || sd.policy == AMP_POLICY_FIXED) {
      // one lane class holds every pair: its own kernel
      const int c = fp32 ? 0 : lane_class(sd.M, sd.fixed_bits, sd.gran);
      sa.cls = c;
      sa.counter = ws.counters + ((ph - 1) * (kNCls + 1) + c) * kQueueSlot;
      sa_lwb = fp32 ? 0 : lane_bits(c, sd.gran, sd.M);
    } else {
      sa.cls = -1;
      sa.counter = ws.counters + ((ph - 1) * (kNCls + 1) + kNCls) * kQueueSlot;
      sa_lwb = sd.gran ? kLwMixSub : kLwMix;
    }
    ScanArgs sp = sa;
    sp.work = (ph == 2 && sd.want_work) ? ws.work : nullptr;
    // (units of one pair and list chunk at the most)
    const int64_t most = (int64_t)npairs * ((ix->max_list + sa.chunk - 1) / sa.chunk);
    if ((err = launch_scan(sa_lwb, ph, dt, sd.wpr, sp, most, st)) != hipSuccess) return err;
    if (ph == 1) {
      // phase-1 minima -> per-query bound, buffer emptied for the candidates
      if (small_b) {
        const size_t tlds = sd.capq * 8 + 4 * (256 + 2);
        if ((err = set_lds(kaddr(k_tau_small), tlds)) != hipSuccess) return err;
        hipLaunchKernelGGL(k_tau_small, dim3(sd.nq), dim3(256), tlds, st, ws.ccount, ws.ckey, ws.tau, ws.kq,
                           sd.kconst, sd.capq, ws.flags + 1);
      } else {
        hipLaunchKernelGGL(k_tau_wave, dim3((sd.nq + 3) / 4), dim3(256), 0, st, ws.ccount, ws.ckey, ws.tau, ws.kq,
                           sd.kconst, sd.nq, sd.capq, ws.flags + 1);
        // keys + digit counts + selection + list of the queries to select in
        const size_t tlds = sd.capq * 8 + 4 * (256 + 2 + 1 + 256);
        if ((err = set_lds(kaddr(k_tau), tlds)) != hipSuccess) return err;
        hipLaunchKernelGGL(k_tau, dim3(sd.nq < 1024 ? sd.nq : 1024), dim3(256), tlds, st, ws.ccount, ws.ckey, ws.tau,
                           ws.kq, sd.kconst, sd.nq, sd.capq);
      }
      if (early && (err = build_queue(1, 2)) != hipSuccess) return err;  // the full scan's queue: live pairs only
    }
    mark(5 + ph);
    if (ph == 2) {
      // (timed with the merge stage: the phase-2 stage is its scan alone)
      // up to two re-runs of phase 2 for queries whose candidates overflowed,
      // each with a tighter bound (the scan kernels return at once when no
      // query takes part); each re-run shrinks a query's candidate count by
      // about k / capq
      const size_t rlds = sd.capq * 16 + 4 * (256 + 2 + 1 + 256);  // keys, ids, digit counts, selection, query list
      err = set_lds(kaddr(k_retry), rlds);
      if (err != hipSuccess) return err;
      ScanArgs sr = sa;
      sr.tau_id = ws.tau_id;
      sr.sorted = ws.sorted;
      sr.units = ws.units;
      RetryArgs ra{ws.ccount, ws.ckey, ws.cid, ws.tau, ws.tau_id, ws.kq, sd.kconst, sd.nq, (kNCls + 1) * kQueueSlot,
                   sd.capq, nullptr, ws.counters + (kNCls + 1) * kQueueSlot, ws.units, ws.sorted};
      QueueArgs qr = qa;
      if (early) {
        qr.pbase = ws.pbase;
        qr.fkeys = fp32 ? 1 : 0;
      }
      for (int rr = 0; rr < sd.reruns; ++rr) {
        sr.nrerun = ra.nrerun = ws.flags + 1 + rr;  // a unit count per round
        hipLaunchKernelGGL(k_retry, dim3(sd.nq < 256 ? sd.nq : 256), dim3(256), rlds, st, ra, qr);
        // phase 3: the phase-2 scan's re-run (its own kernel symbol)
        if ((err = launch_scan(sa_lwb, 3, dt, sd.wpr, sr, most, st)) != hipSuccess) return err;
      }
    }
  }
  // TS
  MergeArgs ma2;
  ma2.ccount = ws.ccount;
  ma2.ckey = ws.ckey;
  ma2.cid = ws.cid;
  ma2.kq = ws.kq;
  ma2.flags = ws.flags;
  ma2.out_ids = out_ids;
  ma2.out_dist = out_dist;
  ma2.out_qdist = out_qdist;
  ma2.kconst = sd.kconst;
  ma2.kmax = sd.kmax;
  ma2.fp32 = fp32 ? 1 : 0;
  ma2.h2 = ldexpf(1.f, sd.metric == AMP_L1 ? sd.grid_e : 2 * sd.grid_e);  // L1 estimates are in units of h
  ma2.capq = sd.capq;
  const size_t mlds = merge_select_lds(sd.capq), flds = sd.capq * 16;
  if (small_b) {
    const size_t slds = std::max(mlds, flds);
    if ((err = set_lds(kaddr(k_merge_small), slds)) != hipSuccess) return err;
    hipLaunchKernelGGL(k_merge_small, dim3(sd.nq), dim3(256), slds, st, ma2);
  } else {
    if ((err = set_lds(kaddr(k_merge), mlds)) != hipSuccess) return err;
    if ((err = set_lds(kaddr(k_merge_full), flds)) != hipSuccess) return err;
    hipLaunchKernelGGL(k_merge_wave, dim3((sd.nq + 3) / 4), dim3(256), 0, st, ma2, sd.nq);
    hipLaunchKernelGGL(k_merge, dim3(sd.nq < 1024 ? sd.nq : 1024), dim3(256), mlds, st, ma2, sd.nq);
    hipLaunchKernelGGL(k_merge_full, dim3(sd.nq < 512 ? sd.nq : 512), dim3(256), flds, st, ma2, sd.nq);
  }
  if (sd.lut_export) {
    // test hook: every pair's LUT as the search builds it
    const amp_lut_export* ex = sd.lut_export;
    BaseArgs eb{};
    eb.Q = queries;
    eb.C = dv.centroids;
    eb.bsw = reinterpret_cast<const u32x4*>(dv.bsw);
    eb.bsw16 = reinterpret_cast<const u32x4*>(dv.bsw16);
    eb.bsw8 = reinterpret_cast<const u32x2*>(dv.bsw8);
    eb.probes = ws.probes;
    eb.pbase = ws.pbase;
    eb.iptab = ws.iptab;
    eb.iptq = ws.iptq;
    eb.ipsh = ws.ipsh;
    eb.pbits = ws.pbits;
    eb.nq = sd.nq;
    eb.d = sd.d;
    eb.M = sd.M;
    eb.dsub = sd.dsub;
    eb.npmax = sd.npmax;
    eb.grid_e = sd.grid_e;
    eb.grid_kind = sd.grid_kind;
    eb.metric = sd.metric;
    eb.gran = sd.gran;
    if (ipm) {
      hipLaunchKernelGGL(k_export_ip, dim3((unsigned)npairs), dim3(256), 0, st, eb, ex->q, ex->shift, ex->base, ex->t);
    } else {
      const size_t elds = base_lds_layout(kBaseExport, sd.M, sd.d).total;
      auto fn = dt == DT_F16 ? k_export<DT_F16> : (dt == DT_F8 ? k_export<DT_F8> : k_export<DT_BF16>);
      if ((err = set_lds(kaddr(fn), elds)) != hipSuccess)
        return err;
      hipLaunchKernelGGL(fn, dim3((unsigned)((npairs + kBaseExport - 1) / kBaseExport)), dim3(kThreads), elds, st, eb,
                         ex->q, ex->shift, ex->base, ex->t);
    }
  }
  if (sd.out_status) hipLaunchKernelGGL(k_status, dim3(1), dim3(64), 0, st, ws.flags, sd.out_status);
  mark(8);
  return hipGetLastError();
}

}  // namespace amp

// index-build kernels and launchers
#include "build_kernels.inc"
