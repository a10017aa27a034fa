// Launchers of the index-build kernels (build_kernels.inc; squared norms:
// kernels.hip).
#pragma once
#include "amp_internal.h"

namespace amp {

// squared norms of n contiguous rows of dd floats
hipError_t launch_sqnorm(const float* X, int64_t n, int dd, float* out, hipStream_t st);
// rows of a sample as residuals: out [n][d] = X[rows[j]] - C[a[rows[j]]]
hipError_t launch_gather_residual(const float* X, const int32_t* a, const float* C, const int32_t* rows, int64_t n,
                                  int d, float* out, hipStream_t st);
// nearest of 256 codewords in each of G subspaces of dd <= 8 dims (row r of
// subspace g at X + r ld + g dd; C [G][256][dd], cn [G][256]): out_a [G][n] or
// the code bytes out_c [n][G]
hipError_t launch_assign_sub(const float* X, int64_t n, int dd, int ld, int G, const float* C, const float* cn,
                             int32_t* out_a, uint8_t* out_c, hipStream_t st);
// one k-means update of G groups (rows as above, key [G][n] their clusters):
// C [G][k][dd] the means in FP64, Cf the same in FP32; empty[g] = 1 where a
// cluster has no member (its centroid stays).  Scratch: order, order2 (k > 256)
// [G][n], hist group_hist_words
size_t group_hist_words(int n, int G);
hipError_t launch_means(const float* X, int n, int dd, int ld, int G, int k, const int32_t* key, int32_t* order,
                        int32_t* order2, int32_t* hist, double* C, float* Cf, int32_t* empty, hipStream_t st);
// per list the largest |R row|^2 (FP64 bits), and the largest magnitude of R
// (vecs: and X) as FP32 bits, both raised from their present values
hipError_t launch_radius(const float* X, const float* R, const int32_t* a, int64_t n, int d, bool vecs,
                         unsigned long long* rad2, uint32_t* amax, hipStream_t st);

}  // namespace amp
