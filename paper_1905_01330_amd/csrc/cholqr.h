// QR of a site by Cholesky factorisation with a certificate (cholqr.hip)
#pragma once

#include "internal.h"

namespace tn {

// The largest |E| that certifies a site of up to kMaxEn columns, 2^-35, as
// bits; beyond, it falls as 1 / n.  The neglected terms are |E|_2^2 <= (n max
// |E|)^2 <= 2^-52 from kMaxEn columns on, an FP64 rounding at the very worst,
// and below that width less (2^-61 or so for errors of random signs).
constexpr uint64_t kMaxE = (uint64_t)(1023 - 35) << 52;
constexpr int kMaxEn = 512;
// ebits: the bits of max |E| max(1, n / kMaxEn) (a NaN's are larger than any
// number's); kernels
// of the Householder path take it as `cert` (null: run) and leave at once
// where the site is certified
__device__ __forceinline__ bool chol_certified(const uint64_t* ebits) { return ebits && *ebits <= kMaxE; }

// the factor L of two diagonal blocks in turn, each with the sums of squares of
// its 64 x 64 entries and of R's, eight parts each
constexpr size_t kCholLinv = 2 * (64 * 64 + 16);   // doubles

// x (dk x cols, row-major) = r (dk x dk upper triangular, zero below) a
int32_t chol_absorb(const double* r, const double* a, double* x, int dk, int cols, hipStream_t st);
// Q1, R1 and U of x (m x n, row-major, overwritten; m >= n), the certificate
// into ebits, and R = (I + U) R1 into r where it holds.  g, r1, u, r: n x n;
// q1: m x n; linv: kCholLinv doubles.
int32_t chol_qr(double* x, int m, int n, double* g, double* r1, double* u, double* q1, double* linv, uint64_t* ebits,
                double* r, hipStream_t st);
// site = Q1 (I - U) where the certificate holds
int32_t chol_q(const double* q1, const double* u, double* site, int m, int n, uint64_t* ebits, hipStream_t st);

}  // namespace tn
