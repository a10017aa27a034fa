// Index-build kernels: the residual codebook's k-means runs for every
// subspace side by side on the device, the encoder writes code bytes, and the
// per-list radius is gathered where the residuals are.  All of them give the
// bits of the sequential definition (build.cpp): nearest centroid in FP32 with
// ties to the lower index, means as FP64 sums over the members in row order.
#include "build_kernels.h"
#include "device_common.h"

namespace amp {

// rows [n][d] of a sample: x - c_a at FP32, gathered by row number
__global__ void k_gather_residual(const float* __restrict__ X, const int32_t* __restrict__ a,
                                  const float* __restrict__ C, const int32_t* __restrict__ rows, int64_t n, int d,
                                  float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * d) return;
  const int64_t j = i / d;
  const int t = (int)(i - j * d), r = rows[j];
  out[i] = X[(size_t)r * d + t] - C[(size_t)a[r] * d + t];
}

// Nearest of 256 codewords in each of G subspaces of dd <= 8 dims: row r of
// subspace g is X + r ld + g dd, its codewords C[g] [256][dd] with squared
// norms cn[g].  A wave keeps the subspace's codewords in registers (16 tiles
// of 16, FP32 MFMA 16x16x4, one or two steps of K) and walks over tiles of 16
// rows; a lane holds 4 rows x 16 codewords and its running minimum, merged
// across the 16 lanes of a row by (distance, index).  The distance is the
// k_assign expression cn - 2 x.c in the same order of products (K beyond dd
// adds exact zeros).  Bound by the VALU comparisons, 4 per distance: 65536 rows
// x 24 subspaces in 50 us, where a launch and a copy per subspace took 35 us
// and 300 us of host time each.
constexpr int kSubRows = 1024;  // rows of a workgroup (4 waves)
template <int KS, bool CODES>
__global__ __launch_bounds__(256) void k_assign_sub(const float* __restrict__ X, int64_t n, int dd, int ld,
                                                    const float* __restrict__ C, const float* __restrict__ cn,
                                                    int32_t* __restrict__ out_a, uint8_t* __restrict__ out_c) {
  const int g = blockIdx.y, G = gridDim.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, kg = lane >> 4;
  const float* Cg = C + (size_t)g * kKsub * dd;
  float b[16][KS], nrm[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int j = 16 * t + col;
#pragma unroll
    for (int k = 0; k < KS; ++k) b[t][k] = 4 * k + kg < dd ? Cg[j * dd + 4 * k + kg] : 0.f;
    nrm[t] = cn[g * kKsub + j];
  }
  const int64_t r0 = (int64_t)blockIdx.x * kSubRows;
  for (int64_t rt = r0 + 16 * wave; rt < r0 + kSubRows && rt < n; rt += 64) {
    float a[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k)
      a[k] = rt + col < n && 4 * k + kg < dd ? X[(size_t)(rt + col) * ld + g * dd + 4 * k + kg] : 0.f;
    float best[4] = {3.4e38f, 3.4e38f, 3.4e38f, 3.4e38f};
    int bi[4] = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KS; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], b[t][k], acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = nrm[t] - 2.f * acc[i];
        if (v < best[i]) {  // (ascending codewords: ties keep the lower)
          best[i] = v;
          bi[i] = 16 * t + col;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        const float ov = __shfl_xor(best[i], o, 16);
        const int oi = __shfl_xor(bi[i], o, 16);
        // (no distance below the start value: index 0, as the sequential scan leaves it)
        if (ov < best[i] || (ov == best[i] && oi < bi[i])) {
          best[i] = ov;
          bi[i] = oi;
        }
      }
      const int64_t r = rt + 4 * kg + i;
      if (col == i && r < n) {
        if (CODES) out_c[(size_t)r * G + g] = (uint8_t)bi[i];
        else out_a[(size_t)g * n + r] = bi[i];
      }
    }
  }
}

// ------------------------------------------------------------------ rows grouped by cluster
// Stable counting sort of n rows by one 8-bit digit of their cluster, G
// groups side by side: counts per block of kSortRows rows, one scan per
// group, and a scatter that ranks equal digits by wave ballots in row order.
constexpr int kSortRows = 1024;
__global__ __launch_bounds__(256) void k_group_hist(const int32_t* __restrict__ key, const int32_t* __restrict__ in,
                                                    int n, int shift, int32_t* __restrict__ hist) {
  __shared__ int32_t h[256];
  const int g = blockIdx.y, nb = gridDim.x;
  h[threadIdx.x] = 0;
  __syncthreads();
  for (int u = 0; u < kSortRows / 256; ++u) {
    const int i = blockIdx.x * kSortRows + u * 256 + threadIdx.x;
    if (i < n) {
      const int r = in ? in[(size_t)g * n + i] : i;
      atomicAdd(&h[(key[(size_t)g * n + r] >> shift) & 255], 1);
    }
  }
  __syncthreads();
  hist[((size_t)g * 256 + threadIdx.x) * nb + blockIdx.x] = h[threadIdx.x];
}
// exclusive scan of a group's 256 nb counts (digit major), in place
__global__ __launch_bounds__(1024) void k_group_scan(int32_t* __restrict__ hist, int nb) {
  __shared__ int32_t s_w[16];
  int32_t* h = hist + (size_t)blockIdx.x * 256 * nb;
  const int total = 256 * nb, per = (total + 1023) / 1024, b0 = threadIdx.x * per;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int sum = 0;
  for (int i = b0; i < b0 + per && i < total; ++i) sum += h[i];
  int inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(inc, o);
    if (lane >= o) inc += v;
  }
  if (lane == 63) s_w[wv] = inc;
  __syncthreads();
  for (int w = 0; w < wv; ++w) inc += s_w[w];
  int x = inc - sum;
  for (int i = b0; i < b0 + per && i < total; ++i) {
    const int c = h[i];
    h[i] = x;
    x += c;
  }
}
__global__ __launch_bounds__(256) void k_group_scatter(const int32_t* __restrict__ key, const int32_t* __restrict__ in,
                                                       int n, int shift, const int32_t* __restrict__ hist,
                                                       int32_t* __restrict__ out) {
  __shared__ int32_t s_base[256], s_cnt[4][256];
  const int g = blockIdx.y, nb = gridDim.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  s_base[tid] = hist[((size_t)g * 256 + tid) * nb + blockIdx.x];
  for (int w = 0; w < 4; ++w) s_cnt[w][tid] = 0;
  __syncthreads();
  for (int u = 0; u < kSortRows / 256; ++u) {
    const int i = blockIdx.x * kSortRows + u * 256 + tid;
    const bool on = i < n;
    const int r = on ? (in ? in[(size_t)g * n + i] : i) : 0;
    const int dg = on ? (key[(size_t)g * n + r] >> shift) & 255 : 0;
    uint64_t peers = __ballot(on);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint64_t m = __ballot((dg >> b) & 1);
      peers &= (dg >> b) & 1 ? m : ~m;
    }
    const int rank = __popcll(peers & ((1ull << lane) - 1));
    if (on && rank == 0) s_cnt[wv][dg] = __popcll(peers);
    __syncthreads();
    if (on) {
      int pos = s_base[dg] + rank;
      for (int w = 0; w < wv; ++w) pos += s_cnt[w][dg];
      out[(size_t)g * n + pos] = r;
    }
    __syncthreads();
    int c = 0;
    for (int w = 0; w < 4; ++w) {
      c += s_cnt[w][tid];
      s_cnt[w][tid] = 0;
    }
    s_base[tid] += c;
    __syncthreads();
  }
}

// New centroids: FP64 sum of each cluster's members in row order times
// 1 / count, one thread per (cluster, dim); order [G][n] holds the rows by
// cluster (a cluster's range by binary search).  A cluster without members
// keeps its centroid and raises its group's flag.
__global__ void k_means_step(const float* __restrict__ X, int n, int dd, int ld, int k,
                             const int32_t* __restrict__ key, const int32_t* __restrict__ order,
                             double* __restrict__ C, float* __restrict__ Cf, int32_t* __restrict__ empty) {
  const int g = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)k * dd) return;
  const int c = (int)(i / dd), t = (int)(i - (int64_t)c * dd);
  const int32_t* a = key + (size_t)g * n;
  const int32_t* o = order + (size_t)g * n;
  auto first = [&](int v) {  // first position whose cluster is at least v
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (a[o[mid]] < v) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  const int j0 = first(c), j1 = first(c + 1);
  double* dst = C + ((size_t)g * k + c) * dd + t;
  if (j1 == j0) {
    if (t == 0) empty[g] = 1;
    return;
  }
  const float* x = X + (size_t)g * dd + t;
  double acc = 0.0;
  int j = j0;
  for (; j + 8 <= j1; j += 8) {  // eight loads in flight ahead of the dependent additions
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[(size_t)o[j + u] * ld];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = __dadd_rn(acc, (double)v[u]);
  }
  for (; j < j1; ++j) acc = __dadd_rn(acc, (double)x[(size_t)o[j] * ld]);
  const double m = __dmul_rn(acc, __ddiv_rn(1.0, (double)(j1 - j0)));
  *dst = m;
  Cf[((size_t)g * k + c) * dd + t] = (float)m;
}

// largest squared residual norm of every list (FP64, dims in order), as the
// bits of a non-negative double, and the largest residual (with vecs: also
// vector) magnitude of all rows, as FP32 bits
__global__ void k_radius(const float* __restrict__ X, const float* __restrict__ R, const int32_t* __restrict__ a,
                         int64_t n, int d, int vecs, unsigned long long* __restrict__ rad2,
                         uint32_t* __restrict__ amax) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float mx = 0.f;
  if (r < n) {
    double s2 = 0.0;
    for (int t = 0; t < d; ++t) {
      const float v = R[(size_t)r * d + t];
      s2 = __dadd_rn(s2, __dmul_rn((double)v, (double)v));
      mx = fabsf(v) > mx ? fabsf(v) : mx;
      if (vecs) {
        const float x = fabsf(X[(size_t)r * d + t]);
        mx = x > mx ? x : mx;
      }
    }
    // (a NaN norm never exceeds the host's running maximum either)
    if (s2 == s2) atomicMax(&rad2[a[r]], (unsigned long long)__double_as_longlong(s2));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if ((threadIdx.x & 63) == 0 && mx > 0.f) atomicMax(amax, __float_as_uint(mx));
}

// ------------------------------------------------------------------ launchers
hipError_t launch_gather_residual(const float* X, const int32_t* a, const float* C, const int32_t* rows, int64_t n,
                                  int d, float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_residual, dim3((unsigned)((n * d + 255) / 256)), dim3(256), 0, st, X, a, C, rows, n, d,
                     out);
  return hipGetLastError();
}

hipError_t launch_assign_sub(const float* X, int64_t n, int dd, int ld, int G, const float* C, const float* cn,
                             int32_t* out_a, uint8_t* out_c, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const dim3 g((unsigned)((n + kSubRows - 1) / kSubRows), (unsigned)G);
  if (dd <= 4) {
    if (out_c) hipLaunchKernelGGL((k_assign_sub<1, true>), g, dim3(256), 0, st, X, n, dd, ld, C, cn, out_a, out_c);
    else hipLaunchKernelGGL((k_assign_sub<1, false>), g, dim3(256), 0, st, X, n, dd, ld, C, cn, out_a, out_c);
  } else {
    if (out_c) hipLaunchKernelGGL((k_assign_sub<2, true>), g, dim3(256), 0, st, X, n, dd, ld, C, cn, out_a, out_c);
    else hipLaunchKernelGGL((k_assign_sub<2, false>), g, dim3(256), 0, st, X, n, dd, ld, C, cn, out_a, out_c);
  }
  return hipGetLastError();
}

size_t group_hist_words(int n, int G) { return (size_t)G * 256 * ((n + kSortRows - 1) / kSortRows); }

hipError_t launch_means(const float* X, int n, int dd, int ld, int G, int k, const int32_t* key, int32_t* order,
                        int32_t* order2, int32_t* hist, double* C, float* Cf, int32_t* empty, hipStream_t st) {
  const int nb = (n + kSortRows - 1) / kSortRows;
  const int32_t* in = nullptr;
  int32_t* out = order;
  for (int shift = 0; shift == 0 || (k - 1) >> shift; shift += 8) {  // k <= 256: one pass; else two
    hipLaunchKernelGGL(k_group_hist, dim3(nb, G), dim3(256), 0, st, key, in, n, shift, hist);
    hipLaunchKernelGGL(k_group_scan, dim3(G), dim3(1024), 0, st, hist, nb);
    hipLaunchKernelGGL(k_group_scatter, dim3(nb, G), dim3(256), 0, st, key, in, n, shift, hist, out);
    in = out;
    out = out == order ? order2 : order;
  }
  hipLaunchKernelGGL(k_means_step, dim3((unsigned)(((int64_t)k * dd + 255) / 256), G), dim3(256), 0, st, X, n, dd, ld,
                     k, key, in, C, Cf, empty);
  return hipGetLastError();
}

hipError_t launch_radius(const float* X, const float* R, const int32_t* a, int64_t n, int d, bool vecs,
                         unsigned long long* rad2, uint32_t* amax, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_radius, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, X, R, a, n, d, vecs ? 1 : 0, rad2,
                     amax);
  return hipGetLastError();
}

}  // namespace amp
