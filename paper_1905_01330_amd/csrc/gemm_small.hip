// Contractions whose contracted and one free extent are both tiny (an MPO
// acting on a bond pair, a 2-index gate): C[m, n] = sum_k A[m, k] B[k, n]
// with K <= 32 and N <= 16.  No matrix-core tile fits such a shape; the
// work is reading A and writing C once, so it is bound by HBM.  B lives in
// LDS, each thread owns one row m (consecutive m are the unit-stride index
// when there is one) and keeps its N sums in FP64.
#include "internal.h"

namespace tn {

constexpr int kSmallK = 32, kSmallN = 16;

__device__ inline float small_bf16(float x) { return (float)(__bf16)x; }

// K and N up to 8: the offsets of k and n come with
// the arguments, a row's values are all in flight before the operand's are in
// LDS, and the sums are unrolled.  A row's time is the latency of one load
// then, not of K.  131072 rows, K = N = 6 (the operator step of a two-site
// update at bond 256): 10.6 us before, 7.7 now, with its result laid out along
// the rows; 10^6 rows, K = N = 4, 20.1 and 10.0.  (With 16 by 16 sums, or a
// loop over a thread's rows, the operand moves into registers and costs waves:
// 10^6 rows, K = N = 10, 38 -> 177 us.)
constexpr int kTab = 8;
constexpr int64_t kTabRows = 65536 * 256;   // a row a thread
struct SmallDesc {
  const float* a;
  const float* b;
  float* c;
  int32_t M, K, N;
  Group gm;
  int64_t ka[kTab], kb[kTab], bn[kTab], cn[kTab];
};
__global__ void __launch_bounds__(256) gemm_small_table_kernel(const SmallDesc d, int bf16_round) {
  __shared__ double sb[kTab][kTab];
  const int K = d.K, N = d.N;
  const int m = blockIdx.x * 256 + threadIdx.x;
  int64_t om[2];
  group_offsets<2>(d.gm, (uint32_t)(m < d.M ? m : d.M - 1), om, 0);
  float av[kTab];
#pragma unroll
  for (int k = 0; k < kTab; ++k)
    if (k < K) av[k] = d.a[om[0] + d.ka[k]];
  if (threadIdx.x < kTab * kTab) {
    const int k = threadIdx.x / kTab, n = threadIdx.x % kTab;
    if (k < K && n < N) {
      const float v = d.b[d.kb[k] + d.bn[n]];
      sb[k][n] = (double)(bf16_round ? small_bf16(v) : v);
    }
  }
  __syncthreads();
  if (m >= d.M) return;
  double acc[kTab];
#pragma unroll
  for (int n = 0; n < kTab; ++n) acc[n] = 0.0;
#pragma unroll
  for (int k = 0; k < kTab; ++k)
    if (k < K) {
      const double a = (double)(bf16_round ? small_bf16(av[k]) : av[k]);
#pragma unroll
      for (int n = 0; n < kTab; ++n)
        if (n < N) acc[n] += a * sb[k][n];
    }
#pragma unroll
  for (int n = 0; n < kTab; ++n)
    if (n < N) d.c[om[1] + d.cn[n]] = (float)acc[n];
}

// PRELOAD: a row's K values are loaded before the first is used (for grids
// too small to hide one load at a time behind other waves; a full chip
// hides it, and there the extra registers would cost waves)
template <bool PRELOAD>
__global__ void __launch_bounds__(256) gemm_small_kernel(const GemmDesc d, int bf16_round) {
  __shared__ float sb[kSmallK * kSmallN];
  __shared__ int64_t ka[kSmallK];
  __shared__ int64_t cn[kSmallN];
  const int K = d.K, N = d.N;
  for (int e = threadIdx.x; e < K * N; e += blockDim.x) {
    const int k = e / N, n = e % N;
    int64_t ok[2], on[2];
    group_offsets<2>(d.gk, (uint32_t)k, ok, 0);
    group_offsets<2>(d.gn, (uint32_t)n, on, 0);
    float v = d.b[ok[1] + on[0]];
    sb[e] = bf16_round ? small_bf16(v) : v;
  }
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    int64_t ok[2];
    group_offsets<2>(d.gk, (uint32_t)k, ok, 0);
    ka[k] = ok[0];
  }
  for (int n = threadIdx.x; n < N; n += blockDim.x) {
    int64_t on[2];
    group_offsets<2>(d.gn, (uint32_t)n, on, 0);
    cn[n] = on[1];
  }
  __syncthreads();
  const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
  for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < d.M; m += nthreads) {
    int64_t om[2];
    group_offsets<2>(d.gm, (uint32_t)m, om, 0);
    double acc[kSmallN];
#pragma unroll
    for (int n = 0; n < kSmallN; ++n) acc[n] = 0.0;
    if constexpr (PRELOAD) {
      float av[kSmallK];
#pragma unroll
      for (int k = 0; k < kSmallK; ++k) av[k] = k < K ? d.a[om[0] + ka[k]] : 0.0f;
#pragma unroll
      for (int k = 0; k < kSmallK; ++k) {
        if (k < K) {
          const float a = bf16_round ? small_bf16(av[k]) : av[k];
#pragma unroll
          for (int n = 0; n < kSmallN; ++n)
            if (n < N) acc[n] += (double)a * (double)sb[k * N + n];
        }
      }
    } else {
      for (int k = 0; k < K; ++k) {
        float a = d.a[om[0] + ka[k]];
        if (bf16_round) a = small_bf16(a);
#pragma unroll
        for (int n = 0; n < kSmallN; ++n)
          if (n < N) acc[n] += (double)a * (double)sb[k * N + n];
      }
    }
#pragma unroll
    for (int n = 0; n < kSmallN; ++n)
      if (n < N) d.c[om[1] + cn[n]] = (float)acc[n];
  }
}

bool gemm_small_fits(const GemmDesc& d) {
  const bool n_small = d.K <= kSmallK && d.N <= kSmallN;
  const bool m_small = d.K <= kSmallK && d.M <= kSmallN;
  return d.batch == 1 && !d.a_scale_bits && !d.c_absmax && (n_small || m_small) && (int64_t)d.M * d.N >= 4096;
}

int32_t launch_gemm_small(const GemmDesc& d0, int32_t prec, hipStream_t st) {
  GemmDesc d = d0;
  if (!(d.K <= kSmallK && d.N <= kSmallN)) {
    // C^T = B^T A^T: the small free extent becomes N
    std::swap(d.a, d.b);
    std::swap(d.M, d.N);
    std::swap(d.gm, d.gn);
    for (int i = 0; i < d.gk.n; ++i) std::swap(d.gk.s[0][i], d.gk.s[1][i]);
  }
  int64_t blocks = (d.M + 255) / 256;
  blocks = blocks < 1 ? 1 : (blocks > 65536 ? 65536 : blocks);
  const int bf = prec == TN_PREC_BF16 ? 1 : 0;
  if (d.K <= kTab && d.N <= kTab && d.M <= kTabRows) {
    SmallDesc t{};
    t.a = d.a;
    t.b = d.b;
    t.c = d.c;
    t.M = d.M;
    t.K = d.K;
    t.N = d.N;
    t.gm = d.gm;
    for (int k = 0; k < d.K; ++k) {
      int64_t o[2];
      group_offsets<2>(d.gk, (uint32_t)k, o, 0);
      t.ka[k] = o[0];
      t.kb[k] = o[1];
    }
    for (int n = 0; n < d.N; ++n) {
      int64_t o[2];
      group_offsets<2>(d.gn, (uint32_t)n, o, 0);
      t.bn[n] = o[0];
      t.cn[n] = o[1];
    }
    hipLaunchKernelGGL(gemm_small_table_kernel, dim3((unsigned)blocks), dim3(256), 0, st, t, bf);
  } else if (blocks < 256)
    hipLaunchKernelGGL(gemm_small_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, d, bf);
  else
    hipLaunchKernelGGL(gemm_small_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, d, bf);
  return hip_check(hipGetLastError(), "small gemm launch");
}

}  // namespace tn
