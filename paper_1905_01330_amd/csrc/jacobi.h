// Jacobi sweeps over the Gram matrix of a matrix's columns (jacobi.hip)
#pragma once

#include "internal.h"

namespace tn {

constexpr int kJacB = 16;   // columns of a block; a block pair is one eigenproblem of order 32

// columns (padded) that a sweep takes: whole block pairs
inline int64_t jac_padded(int64_t c) { return (c + 2 * kJacB - 1) / (2 * kJacB) * (2 * kJacB); }
// matrices are read through 2^31-byte buffers
inline bool jac_fits(int64_t rows, int64_t cp) { return cp <= 4096 && rows * cp < (int64_t)1 << 28; }
// doubles of scratch: two Gram matrices, the sweep's rotations and two rounds' rotations
inline size_t jac_scratch_doubles(int64_t cp) { return (size_t)(3 * cp * cp + 2 * (cp / (2 * kJacB)) * 4 * kJacB * kJacB); }

// The Gram matrix of x's columns (column c of x at x + c rows; cp columns) in
// the order perm into the scratch, and into *ctl a count that is zero where
// every pair is orthogonal: |g_ij| <= tol sigma_i sigma_j (sigma: the columns' norms).
int32_t jac_gram(const double* x, int rows, int cp, const double* sigma, const int* perm, double tol, double* scratch,
                 int* ctl, hipStream_t st);
// One sweep over all pairs from that Gram matrix: x2 = x(:, perm) J, v2 = v(:, perm) J (v: cp x cp).
// Its kernels leave at once where *ctl is zero, so that a sweep can be issued
// before the count is known to the host; x2 and v2 are undefined then.
int32_t jac_sweep(const double* x, const double* v, double* x2, double* v2, int rows, int cp, const int* perm,
                  double tol, double* scratch, const int* ctl, hipStream_t st);

}  // namespace tn
