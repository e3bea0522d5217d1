// Left-canonical gauge of an MPS in FP64 on the GPU: successive QR
// factorisations.  For site k the carried triangular factor is absorbed first
// (X = R_{k-1} A_k viewed as (D_k d) x D_{k+1}), X is factorised, and
// diag(R) >= 0.
//
// From kCholMin columns on a site is first factorised by Cholesky
// (cholqr.hip); where its certificate holds, the Householder kernels below
// leave at once, otherwise they do the site from the start.
//
// Householder (Golub and Van Loan, "Matrix Computations", 5.1-5.2): X is
// factorised in place, the thin Q is accumulated backwards from [I; 0], and
// signs are fixed.  X and Q are kept column-major so every reflector and
// column update reads contiguous memory.  Up to 2048 rows the factorisation
// is blocked in the compact WY form (Schreiber and Van Loan; Golub and Van
// Loan 5.2.3): one workgroup factorises a panel of 16 columns held in
// registers (one workgroup reduction per column, row conditions as selects so
// the unrolled panel stays short) and forms the panel's triangular factor T
// from the Gram matrix of its reflectors; I - V T^T V^T is applied to the
// columns of the panels after it on the matrix cores, a panel's columns a
// workgroup (the next panel's by that panel's own); Q is accumulated panel by
// panel in reverse with I - V T V^T.  All panels and updates of a matrix are
// tasks of one launch.  Taller matrices take one reflector launch and one
// update launch per column.
#include <algorithm>
#include <cmath>
#include <vector>

#include "cholqr.h"

namespace tn {

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

__device__ inline double block_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

// Xc[b * m + (i * d + s)] = sum_l R[i, l] A[l, s, b]     (R: dk x dk row-major,
// upper triangular: the sum starts at l = i, so a row block skips the l
// blocks below it).  The 64 x 64 result tile goes through LDS so that the
// column-major stores run along i.
__global__ void __launch_bounds__(256) absorb_kernel(const double* __restrict__ r, const double* __restrict__ a,
                                                     double* __restrict__ xc, int dk, int d, int dn,
                                                     uint32_t* ctr, int ctr_words, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  // the task counters of the factorisation that follows
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = threadIdx.x; i < ctr_words; i += 256) ctr[i] = 0;
  __shared__ double sr[64][17];
  __shared__ double sa[16][65];
  __shared__ double so[64][65];
  const int m = dk * d;
  const int p = d * dn;            // columns of A viewed (dk, d*dn)
  const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double acc[4][4] = {};
  for (int l0 = i0; l0 < dk; l0 += 16) {
    for (int e = threadIdx.x; e < 64 * 16; e += 256) {
      int ii = e / 16, ll = e % 16;
      sr[ii][ll] = (i0 + ii < dk && l0 + ll < dk) ? r[(int64_t)(i0 + ii) * dk + l0 + ll] : 0.0;
      int l2 = e / 64, jj = e % 64;
      sa[l2][jj] = (l0 + l2 < dk && j0 + jj < p) ? a[(int64_t)(l0 + l2) * p + j0 + jj] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int ll = 0; ll < 16; ++ll)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = fma(sr[ty * 4 + u][ll], sa[ll][tx * 4 + v], acc[u][v]);
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) so[ty * 4 + u][tx * 4 + v] = acc[u][v];
  __syncthreads();
  // consecutive threads take consecutive i of one column j = (s, b)
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int jl = e / 64, il = e % 64;
    const int i = i0 + il, j = j0 + jl;
    if (i < dk && j < p) {
      const int s = j / dn, b = j - s * dn;
      xc[(int64_t)b * m + i * d + s] = so[il][jl];
    }
  }
}

// reflector for column j of the column-major m x n matrix X (LAPACK larfg convention)
__global__ void __launch_bounds__(256) reflector_kernel(double* xc, double* tau, int m, int j, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  __shared__ double red[4];
  double* col = xc + (int64_t)j * m;
  double s = 0.0;
  for (int i = j + 1 + threadIdx.x; i < m; i += blockDim.x) s += col[i] * col[i];
  const double sigma = block_sum(s, red);
  const double alpha = col[j];
  __syncthreads();
  if (sigma == 0.0) {
    if (threadIdx.x == 0) tau[j] = 0.0;
    return;
  }
  const double beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
  const double scale = 1.0 / (alpha - beta);
  for (int i = j + 1 + threadIdx.x; i < m; i += blockDim.x) col[i] *= scale;
  if (threadIdx.x == 0) {
    tau[j] = (beta - alpha) / beta;
    col[j] = beta;
  }
}

// apply H_j = I - tau v v^T (v_j = 1, v_i = X[i, j] below) to columns c0.. of Y (m rows, column-major)
__global__ void __launch_bounds__(256) reflect_cols_kernel(const double* __restrict__ xc, const double* __restrict__ tau,
                                                           double* y, int m, int j, int c0, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  __shared__ double red[4];
  const double t = tau[j];
  if (t == 0.0) return;
  const double* v = xc + (int64_t)j * m;
  double* col = y + (int64_t)(c0 + blockIdx.x) * m;
  double s = threadIdx.x == 0 ? col[j] : 0.0;
  for (int i = j + 1 + threadIdx.x; i < m; i += blockDim.x) s += v[i] * col[i];
  const double w = block_sum(s, red) * t;
  if (threadIdx.x == 0) col[j] -= w;
  for (int i = j + 1 + threadIdx.x; i < m; i += blockDim.x) col[i] -= w * v[i];
}

// ---- blocked path (m <= kQrThreads * kQrRows) --------------------------------

constexpr int kQrThreads = 512;   // threads per workgroup; thread t owns rows t + 512 q
constexpr int kQrRows = 4;        // rows per thread
constexpr int kQrNb = 16;         // panel width
constexpr int kQrCb = 4;          // columns of a product with Q per workgroup
constexpr int kQrWaves = kQrThreads / 64;

// x from lane (this lane xor M) of the wavefront.  Within a 16-lane row (M <
// 16) a DPP move on each 32-bit half: quad permutations for M = 1, 2, the
// row rotation by 8 for M = 8, and for M = 4 the rotation by 4 or by 12 as
// the lane's bit 2 is set or clear; across rows a lane exchange through the
// LDS crossbar.
template <int CTRL>
__device__ __forceinline__ double qr_dpp(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

template <int M>
__device__ __forceinline__ double qr_xor_lane(double x) {
  if constexpr (M == 1) return qr_dpp<0xB1>(x);         // quad_perm [1, 0, 3, 2]
  else if constexpr (M == 2) return qr_dpp<0x4E>(x);    // quad_perm [2, 3, 0, 1]
  else if constexpr (M == 4) {
    // row_ror n: lane i reads lane (i - n) mod 16 of its row
    const double below = qr_dpp<0x124>(x);              // row_ror 4: lane i - 4
    const double above = qr_dpp<0x12C>(x);              // row_ror 12: lane i + 4
    return (threadIdx.x & 4) ? below : above;
  } else if constexpr (M == 8) return qr_dpp<0x128>(x);  // row_ror 8: lane i xor 8
  else return __shfl_xor(x, M, 64);
}

// x of lane L (a constant) in every lane
template <int L>
__device__ __forceinline__ double qr_read_lane(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)v, L);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), L);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

template <int NV, int I = 0>
__device__ __forceinline__ void qr_broadcast(double t, double (&v)[NV]) {
  if constexpr (I < NV) {
    v[I] = qr_read_lane<I>(t);
    qr_broadcast<NV, I + 1>(t, v);
  }
}

// Wavefront reduce-scatter of N partial values (N a power of two <= 64):
// lane l returns the sum over the 64 lanes of value l % N.  Each halving step
// sends one half of the remaining values to the partner lane and keeps the
// other half (N - 1 exchanges in all, instead of 6 N for N separate sums).
template <int N, int H>
__device__ __forceinline__ void qr_halve(double (&v)[N], int lane) {
  if constexpr (H >= 1) {
    const bool up = (lane & H) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double send = up ? v[i] : v[i + H];
      const double keep = up ? v[i + H] : v[i];
      v[i] = keep + qr_xor_lane<H>(send);
    }
    qr_halve<N, H / 2>(v, lane);
  }
}

// r summed over the lane groups that differ in bits N, 2N, ... 32
template <int MK>
__device__ __forceinline__ void qr_xor_tail(double& r) {
  if constexpr (MK < 64) {
    r += qr_xor_lane<MK>(r);
    qr_xor_tail<MK * 2>(r);
  }
}

template <int N>
__device__ inline double qr_reduce_scatter(double (&v)[N]) {
  const int lane = threadIdx.x & 63;
  qr_halve<N, N / 2>(v, lane);
  double r = v[0];
  qr_xor_tail<N>(r);
  return r;
}

// Workgroup sum of v[0..NV) returned to every thread.  P (a power of two >=
// NV) values per wavefront go through red[buf] (two buffers used in turn, so
// one barrier per reduction suffices: a wavefront can only write a buffer
// again after every wavefront has passed the barrier of the reduction that
// read it last).
template <int NV, int P>
__device__ inline void qr_block_sum(double (&v)[NV], double (*red)[kQrWaves * 64], int& buf) {
  double w[P];
#pragma unroll
  for (int i = 0; i < P; ++i) w[i] = i < NV ? v[i] : 0.0;
  const double r = qr_reduce_scatter<P>(w);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane < P) red[buf][wave * P + lane] = r;
  __syncthreads();
  // lane i < NV of every wavefront adds the wavefronts' partial sums of value
  // i (in wavefront order), and every lane takes value i from lane i: eight
  // LDS reads per lane instead of eight per value
  double t = 0.0;
  if (lane < NV) {
#pragma unroll
    for (int wv = 0; wv < kQrWaves; ++wv) t += red[buf][wv * P + lane];
  }
  qr_broadcast<NV>(t, v);
  buf ^= 1;
}

// The reflector of panel column J (a template argument, so the register
// panel is only indexed by constants) and its update of the panel columns to
// its right, the same reflector as reflector_kernel + reflect_cols_kernel with
// one workgroup reduction: the products of column J with itself and the
// columns to its right below row gj, s_c = sum x_J x_c, give both the norm
// (c = J) and, with row gj's entries y_c and v = [1; x_J scale],
// v^T x_c = y_c + scale s_c.  (Two reductions, the second over the scaled
// column: a 512 x 512 split's factorisation and the rest 0.7 ms slower, of
// 25.3.)  Row conditions are selects, not branches, to keep the
// unrolled panel short.
template <int J, int NR>
__device__ __forceinline__ void qr_panel_step(double (&x)[NR][kQrNb], double (*red)[kQrWaves * 64],
                                              double (*top)[kQrNb], int& buf, double* tau, int m, int r0, int j0, int nb) {
  if constexpr (J < kQrNb) {
    if (J < nb) {
      constexpr int NW = kQrNb - J;
      const int gj = j0 + J;
      // A column of values near 1e-150 (what is left of dependent columns)
      // would lose its norm to underflow and the reflector its orthogonality:
      // its products are then formed again with the column scaled by 2^700,
      // which leaves v and tau as they are.
      double s[NW], unit = 1.0, sigma, alpha;
      int at;
      for (;;) {
#pragma unroll
        for (int c = 0; c < NW; ++c) s[c] = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
          const int row = r0 + threadIdx.x + kQrThreads * q;
          const double xv = row > gj && row < m ? unit * x[q][J] : 0.0;
          s[0] += xv * xv;
#pragma unroll
          for (int c = 1; c < NW; ++c) s[c] += xv * x[q][J + c];
          if (row == gj) {
#pragma unroll
            for (int c = 0; c < NW; ++c) top[buf][c] = x[q][J + c];
          }
        }
        at = buf;
        qr_block_sum<NW, (NW > 8 ? 16 : NW > 4 ? 8 : NW > 2 ? 4 : NW > 1 ? 2 : 1)>(s, red, buf);
        sigma = s[0];
        alpha = unit * top[at][0];
        if (unit != 1.0 || !(alpha * alpha + sigma < 1e-240)) break;
        unit = 0x1p700;
      }
      double t = 0.0;
      if (sigma != 0.0) {   // the same in every thread
        double beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
        double scale = 1.0 / (alpha - beta);
        t = (beta - alpha) / beta;
        double w[NW];
#pragma unroll
        for (int c = 1; c < NW; ++c) w[c] = t * (top[at][c] + scale * s[c]);
        if (unit != 1.0) {
          beta *= 0x1p-700;
          scale *= unit;
        }
#pragma unroll
        for (int q = 0; q < NR; ++q) {
          const int row = r0 + threadIdx.x + kQrThreads * q;
          const double v = row > gj && row < m ? x[q][J] * scale : (row == gj ? 1.0 : 0.0);
          x[q][J] = row > gj && row < m ? v : (row == gj ? beta : x[q][J]);
#pragma unroll
          for (int c = 1; c < NW; ++c) x[q][J + c] -= w[c] * v;
        }
      }
      if (threadIdx.x == 0) tau[gj] = t;
    }
    qr_panel_step<J + 1, NR>(x, red, top, buf, tau, m, r0, j0, nb);
  }
}

// Factorise columns j0 .. j0+nb-1 (rows j0..m-1) of the column-major X in
// place, then form the panel's triangular factor (LAPACK larft, forward,
// columnwise): H_0 ... H_{nb-1} = I - V T V^T with T[j][j] = tau_j and
// T[0:j, j] = -tau_j T[0:j, 0:j] (V[:, 0:j]^T v_j); T row-major 16 x 16.
struct QrPanelSmem {
  double red[2][kQrWaves * 64];
  double top[2][kQrNb];
  double gram[kQrNb * kQrNb];
  double tl[kQrNb * kQrNb];
  double stage[kQrWaves][64][kQrNb + 1];   // a wave's 64 rows, between a row a lane and the matrix cores' layouts
  double part[kQrWaves][kQrNb * kQrNb];    // the waves' shares of a 16 x 16 sum
};
typedef double qr_d4_t __attribute__((ext_vector_type(4)));
// a wave's LDS accesses are served in order; the compiler must keep them so
__device__ __forceinline__ void qr_wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ void qr_stage(double (*st)[kQrNb + 1], const double (&v)[kQrNb]) {
  qr_wave_order();
#pragma unroll
  for (int c = 0; c < kQrNb; ++c) st[threadIdx.x & 63][c] = v[c];
  qr_wave_order();
}
// A^T B of a wave's 64 rows, operands as qr_rows reads them.  Sixteen rows a
// chain: summed in a tree as far as the matrix cores' own order allows
// (64 in one chain: |Q R - X| of a factorisation 1.2 times as large).
__device__ __forceinline__ qr_d4_t qr_products(const double (&a)[16], const double (&b)[16]) {
  qr_d4_t w[4] = {};
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) w[kk & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], b[kk], w[kk & 3], 0, 0, 0);
  return (w[0] + w[1]) + (w[2] + w[3]);
}
// the staged rows as a right operand (or, transposed, a left one) of a sum
// over the rows: k = 4 kk + lane / 16, column lane % 16
__device__ __forceinline__ void qr_rows(const double (*st)[kQrNb + 1], double (&o)[16]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) o[kk] = st[4 * kk + (lane >> 4)][lane & 15];
}

// A matrix (below 2^31 bytes) as a raw buffer: a thread's row is a vector
// offset, a column a scalar one, and a row past the matrix an offset past the
// buffer, which reads zero and is not written.  (Addresses of 16 columns each
// would take the registers that a panel of four rows a thread needs.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t qr_rsrc(const double* xc) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(xc), (short)0, (int)0x80000000, 0x00020000);
}
__device__ __forceinline__ uint32_t qr_row(int m, int r0, int q) {
  const int row = r0 + threadIdx.x + kQrThreads * q;
  return row < m ? (uint32_t)row * 8u : 0x80000000u;
}
// columns c0 .. c0 + nb - 1 at this thread's row q (rows from r0 on), zero past the matrix
__device__ __forceinline__ void qr_columns(double (&x)[kQrNb], __amdgpu_buffer_rsrc_t rs, int m, int r0, int c0, int nb, int q) {
  const uint32_t row = qr_row(m, r0, q);
#pragma unroll
  for (int c = 0; c < kQrNb; ++c)
    x[c] = __builtin_bit_cast(
        double, __builtin_amdgcn_raw_buffer_load_b64(rs, c < nb ? row : 0x80000000u, c < nb ? (c0 + c) * m * 8 : 0, 0));
}
__device__ __forceinline__ void qr_store(const double (&x)[kQrNb], __amdgpu_buffer_rsrc_t rs, int m, int r0, int c0, int nb,
                                         int q) {
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  const uint32_t row = qr_row(m, r0, q);
#pragma unroll
  for (int c = 0; c < kQrNb; ++c)
    if (c < nb) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, x[c]), rs, row, (c0 + c) * m * 8, 0);
}

// Panel j0 (whole, reflectors in X, factor T) applied to the columns c0 .. c0 +
// nb - 1, rows from j0 on: x -= V T^T (V^T x) on the matrix cores; f(q, x) with
// the result at this thread's row q.  The next panel's own workgroup does it
// for that panel's columns (by other workgroups it was 7 us and a second
// exchange of data of a panel's 60 us at 512 x 512).  Bound by the latency of a
// workgroup's loads; each application also costs a release and an acquire of
// the caches, so a task takes a panel's 16 columns.  With four columns a task,
// summed by vector instructions, the applications were longer than the panels
// from 1024 rows on: 2048 x 1024 7.1 -> 4.2 ms (4.9 with a launch a panel and a
// launch an application), 1024 x 1024 4.5 -> 2.7, 512 x 512 1.38 -> 1.09.  Up
// to two rows a thread x is read once and held between the two products, and
// the reflectors are read ahead of them; with four the registers hold neither.
template <int NR, class F>
__device__ __forceinline__ void qr_block(__amdgpu_buffer_rsrc_t rs, const double* __restrict__ tf, int m, int j0, int c0,
                                         int nb, QrPanelSmem& sm, F&& f) {
  constexpr bool HOLD = NR <= 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, lk = lane >> 4;
  auto st = sm.stage[wave];
  double t[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) t[kk] = tf[(j0 / kQrNb) * kQrNb * kQrNb + (4 * kk + lk) * kQrNb + l15];
  auto reflectors = [&](int q, double (&v)[kQrNb]) {
    qr_columns(v, rs, m, j0, j0, kQrNb, q);
    const int at = threadIdx.x + kQrThreads * q;   // row j0 + at: column c is 1 at c, X below it, 0 above
#pragma unroll
    for (int c = 0; c < kQrNb; ++c) v[c] = at > c ? v[c] : at == c ? 1.0 : 0.0;
  };
  double v[kQrNb], x[HOLD ? NR : 1][kQrNb];
  qr_d4_t w = {};
  auto sum = [&](const double (&y)[kQrNb]) {
    double a[16], b[16];
    qr_stage(st, v);
    qr_rows(st, a);
    qr_stage(st, y);
    qr_rows(st, b);
    w += qr_products(a, b);
  };
  if constexpr (HOLD) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      qr_columns(x[q], rs, m, j0, c0, nb, q);
      reflectors(q, v);
      sum(x[q]);
    }
  } else {
#pragma unroll 1
    for (int q = 0; q < NR; ++q) {
      reflectors(q, v);
      qr_columns(x[0], rs, m, j0, c0, nb, q);
      sum(x[0]);
    }
  }
  // FP64 16x16x4 result: lane (column l15) register r holds row 4 r + lk,
  // which is the next product's right operand as it stands
#pragma unroll
  for (int r = 0; r < 4; ++r) sm.part[wave][r * 64 + lane] = w[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    w[r] = 0.0;
#pragma unroll
    for (int wv = 0; wv < kQrWaves; ++wv) w[r] += sm.part[wv][r * 64 + lane];
  }
  qr_d4_t w2 = {};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) w2 = __builtin_amdgcn_mfma_f64_16x16x4f64(t[kk], w[kk], w2, 0, 0, 0);
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    double(&y)[kQrNb] = x[HOLD ? q : 0];
    if (NR > 1) reflectors(q, v);
    if (!HOLD) qr_columns(y, rs, m, j0, c0, nb, q);
    qr_stage(st, v);
    constexpr int AHEAD = HOLD ? 4 : 1;   // 16-row blocks read at a time
    double a[AHEAD][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i % AHEAD == 0) {
#pragma unroll
        for (int h = 0; h < AHEAD; ++h)
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) a[h][kk] = st[16 * (i + h) + l15][4 * kk + lk];
        qr_wave_order();
      }
      qr_d4_t o = {};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) o = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i % AHEAD][kk], w2[kk], o, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) st[16 * i + 4 * r + lk][l15] = o[r];
    }
    qr_wave_order();
#pragma unroll
    for (int c = 0; c < kQrNb; ++c) y[c] -= st[lane][c];
    f(q, y);
    if (!HOLD) __builtin_amdgcn_sched_barrier(0);   // one row's loads at a time: the registers hold no more
  }
}

// (ahead: the panel before it is applied first, and its rows are held too)
template <int NR>
__device__ inline void qr_panel(double* xc, double* tau, double* tf, int m, int j0, int nb, bool ahead, QrPanelSmem& sm) {
  auto& red = sm.red;
  auto& gram = sm.gram;
  auto& tl = sm.tl;
  const int r0 = ahead ? j0 - kQrNb : j0;   // rows above are done
  int buf = 0;
  double x[NR][kQrNb];
  const __amdgpu_buffer_rsrc_t rs = qr_rsrc(xc);
  if (ahead) {
    qr_block<NR>(rs, tf, m, r0, j0, nb, sm, [&](int q, const double (&y)[kQrNb]) {
#pragma unroll
      for (int c = 0; c < kQrNb; ++c) x[q][c] = y[c];
    });
  } else {
#pragma unroll
    for (int q = 0; q < NR; ++q) qr_columns(x[q], rs, m, r0, j0, nb, q);
  }
  qr_panel_step<0, NR>(x, red, sm.top, buf, tau, m, r0, j0, nb);
#pragma unroll
  for (int q = 0; q < NR; ++q) qr_store(x[q], rs, m, r0, j0, nb, q);
  // the reflectors in place of the panel: v_c is 1 at row j0 + c, X below it,
  // 0 above (and 0 in the columns past nb)
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int row = r0 + threadIdx.x + kQrThreads * q;
#pragma unroll
    for (int c = 0; c < kQrNb; ++c) {
      const int gc = j0 + c;
      x[q][c] = (c >= nb || row >= m) ? 0.0 : (row == gc ? 1.0 : (row > gc ? x[q][c] : 0.0));
    }
  }
  // Gram matrix of the reflectors, on the matrix cores
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    qr_d4_t g = {};
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      double o[16];
      qr_stage(sm.stage[wave], x[q]);
      qr_rows(sm.stage[wave], o);
      g += qr_products(o, o);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) sm.part[wave][r * 64 + lane] = g[r];
    __syncthreads();
    if (threadIdx.x < kQrNb * kQrNb) {
      double t = 0.0;
#pragma unroll
      for (int wv = 0; wv < kQrWaves; ++wv) t += sm.part[wv][threadIdx.x];
      gram[threadIdx.x] = t;
    }
    __syncthreads();
  }
  // lane i builds row i of T: T[i][j] needs only T[i][i..j-1] (its own row)
  if (threadIdx.x < kQrNb) {
    const int i = threadIdx.x;
    double row[kQrNb];
#pragma unroll
    for (int j = 0; j < kQrNb; ++j) {
      const double tj = j < nb ? tau[j0 + j] : 0.0;
      double v = 0.0;   // row[l] is zero for l < i
#pragma unroll
      for (int l = 0; l < j; ++l) v += row[l] * gram[l * kQrNb + j];
      row[j] = i < j ? -tj * v : i == j ? tj : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kQrNb; ++j) tl[i * kQrNb + j] = row[j];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kQrNb * kQrNb; e += kQrThreads) tf[(j0 / kQrNb) * kQrNb * kQrNb + e] = tl[e];
}

// reflector j of the panel at this thread's rows (from r0 on): 1 at row j0+j, X below, 0 above
template <int NR>
__device__ inline void qr_load_v(const double* __restrict__ xc, int m, int r0, int j0, int nb, int j, double (&v)[NR]) {
  const int gj = j0 + j;
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int row = r0 + threadIdx.x + kQrThreads * q;
    v[q] = j >= nb ? 0.0 : (row == gj ? 1.0 : ((row > gj && row < m) ? xc[(int64_t)gj * m + row] : 0.0));
  }
}

// Y (this workgroup's kQrCb columns, thread t's rows r0 + t + 512 q in yv) times
// the panel j0 .. j0+nb-1 (reflectors in X, triangular factor T) for products
// with Q: Y -= V T (V^T Y) (H_0 ... H_{nb-1} Y)
struct QrApplySmem {
  double red[kQrWaves * kQrNb * kQrCb];
  double sw[kQrNb * kQrCb], sw2[kQrNb * kQrCb], st[kQrNb * kQrNb];
};
template <int NR>
__device__ inline void qr_apply(const double* __restrict__ xc, const double* __restrict__ tf, int m, int r0, int j0, int nb,
                                double (&yv)[NR][kQrCb], QrApplySmem& sm) {
  constexpr int NW = kQrNb * kQrCb;   // 64 entries of W = V^T Y
  for (int e = threadIdx.x; e < kQrNb * kQrNb; e += kQrThreads) sm.st[e] = tf[(j0 / kQrNb) * kQrNb * kQrNb + e];
  double w[NW];
#pragma unroll
  for (int j = 0; j < kQrNb; ++j) {
    double v[NR];
    qr_load_v(xc, m, r0, j0, nb, j, v);
#pragma unroll
    for (int c = 0; c < kQrCb; ++c) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NR; ++q) s += v[q] * yv[q][c];
      w[j * kQrCb + c] = s;
    }
  }
  const double r = qr_reduce_scatter<NW>(w);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  sm.red[wave * NW + lane] = r;
  __syncthreads();
  if (threadIdx.x < NW) {
    double t = 0.0;
#pragma unroll
    for (int wv = 0; wv < kQrWaves; ++wv) t += sm.red[wv * NW + threadIdx.x];
    sm.sw[threadIdx.x] = t;
  }
  __syncthreads();
  if (threadIdx.x < NW) {
    const int j = threadIdx.x / kQrCb, c = threadIdx.x % kQrCb;
    double t = 0.0;
#pragma unroll
    for (int l = 0; l < kQrNb; ++l) t += sm.st[j * kQrNb + l] * sm.sw[l * kQrCb + c];
    sm.sw2[threadIdx.x] = t;
  }
  __syncthreads();
#pragma unroll 2
  for (int j = 0; j < kQrNb; ++j) {
    double v[NR];
    qr_load_v(xc, m, r0, j0, nb, j, v);
#pragma unroll
    for (int c = 0; c < kQrCb; ++c) {
      const double w2 = sm.sw2[j * kQrCb + c];
#pragma unroll
      for (int q = 0; q < NR; ++q) yv[q][c] -= v[q] * w2;
    }
  }
}

template <int NR>
__device__ inline void qr_load_y(const double* y, int m, int r0, int cb0, int ncols, double (&yv)[NR][kQrCb]) {
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int row = r0 + threadIdx.x + kQrThreads * q;
#pragma unroll
    for (int c = 0; c < kQrCb; ++c) yv[q][c] = (row < m && cb0 + c < ncols) ? y[(int64_t)(cb0 + c) * m + row] : 0.0;
  }
}
template <int NR>
__device__ inline void qr_store_y(double* y, int m, int r0, int cb0, int ncols, const double (&yv)[NR][kQrCb]) {
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int row = r0 + threadIdx.x + kQrThreads * q;
    if (row < m) {
#pragma unroll
      for (int c = 0; c < kQrCb; ++c)
        if (cb0 + c < ncols) y[(int64_t)(cb0 + c) * m + row] = yv[q][c];
    }
  }
}

// The whole factorisation in one launch.  The workgroup that is first does the
// panels, one after the other (its code and its own panel stay close; dealt to
// any workgroup they took 49 us each at 512 x 512, so 44, and now 34), each with the
// panel before it applied to its own columns.  The tasks of the others are the
// applications of panel p to the columns of a panel past p + 1, in the order of
// p, taken from a counter.  An application waits for its panel and for the last
// application to its columns, which has a smaller number and so has been taken
// by a running workgroup.  A panel waits for the applications of all but the
// last panel to its columns; while these have not been taken the panels'
// workgroup takes tasks itself, so every wait ends whatever share of the grid
// is resident.
// ctr: the task counter, the number of finished panels, the number of
// workgroups begun, and per panel the number of panels applied to its columns
// (zero at the start).
__host__ __device__ inline int qr_panels(int n) { return (n + kQrNb - 1) / kQrNb; }

__device__ inline void qr_wait(const uint32_t* flag, uint32_t want) {
  if (threadIdx.x == 0)
    while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) __builtin_amdgcn_s_sleep(4);
}
__device__ inline void qr_acquire() {
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}
__device__ inline void qr_signal(uint32_t* flag, uint32_t value) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(kQrThreads) qr_factor_kernel(double* xc, double* tau, double* tf, int m, int n,
                                                               uint32_t* ctr, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  __shared__ QrPanelSmem sm;
  __shared__ int s_task;
  const int panels = qr_panels(n);
  uint32_t* done = ctr + 1;
  uint32_t* applied = ctr + 3;
  // panel p's applications: panels p + 2 and on
  auto count = [&](int p) { return max(panels - p - 2, 0); };
  auto apply = [&](int p, int g) {
    const int j0 = p * kQrNb, c0 = g * kQrNb, nb = min(n - c0, kQrNb);
    qr_wait(done, (uint32_t)(p + 1));
    qr_wait(applied + g, (uint32_t)p);
    qr_acquire();
    const __amdgpu_buffer_rsrc_t rs = qr_rsrc(xc);
    auto store = [&](int q, const double (&y)[kQrNb]) { qr_store(y, rs, m, j0, c0, nb, q); };
    if (m - j0 <= kQrThreads) qr_block<1>(rs, tf, m, j0, c0, nb, sm, store);
    else if (m - j0 <= 2 * kQrThreads) qr_block<2>(rs, tf, m, j0, c0, nb, sm, store);
    else qr_block<kQrRows>(rs, tf, m, j0, c0, nb, sm, store);
    qr_signal(applied + g, (uint32_t)(p + 1));
  };
  if (threadIdx.x == 0) s_task = (int)atomicAdd(ctr + 2, 1u);
  __syncthreads();
  const bool first = s_task == 0;
  // tasks base .. base + count(p) - 1 are panel p's
  int p = 0, base = 0, q = first ? 0 : panels;
  for (;;) {
    __syncthreads();
    if (q < panels) {
      // the next panel, as soon as all tasks that it needs have been taken
      int need = 0;   // tasks up to panel q - 2's for its columns
      for (int i = 0; i < q - 2; ++i) need += count(i);
      if (q >= 2) ++need;
      if (threadIdx.x == 0) {
        uint32_t t = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_task = -1;
        while ((int)t < need) {
          if (__hip_atomic_compare_exchange_strong(ctr, &t, t + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT)) {
            s_task = (int)t;
            break;
          }
        }
      }
      __syncthreads();
      if (s_task < 0) {
        const int j0 = q * kQrNb;
        if (q > 1) qr_wait(applied + q, (uint32_t)(q - 1));
        qr_acquire();
        const int nb = n - j0 < kQrNb ? n - j0 : kQrNb, rows = m - (q > 0 ? j0 - kQrNb : 0);
        if (rows <= kQrThreads) qr_panel<1>(xc, tau, tf, m, j0, nb, q > 0, sm);
        else if (rows <= 2 * kQrThreads) qr_panel<2>(xc, tau, tf, m, j0, nb, q > 0, sm);
        else qr_panel<kQrRows>(xc, tau, tf, m, j0, nb, q > 0, sm);
        ++q;
        qr_signal(done, (uint32_t)q);
        continue;
      }
    } else {
      if (threadIdx.x == 0) s_task = (int)atomicAdd(ctr, 1u);
      __syncthreads();
    }
    const int task = s_task;
    while (p < panels && task >= base + count(p)) base += count(p++);
    if (p >= panels) return;
    apply(p, p + 2 + task - base);
  }
}

// Y := Q Y (eye: Y = Q [I; 0]), kQrCb columns a workgroup, all panels from the
// last (eye: from the first that reaches the columns) with Y in registers
template <int NR>
__global__ void __launch_bounds__(kQrThreads) qr_form_kernel(const double* __restrict__ xc, const double* __restrict__ tf,
                                                             double* y, int m, int n, int ncols, bool eye,
                                                             const uint64_t* cert) {
  if (chol_certified(cert)) return;
  __shared__ QrApplySmem sm;
  const int cb0 = blockIdx.x * kQrCb;
  double yv[NR][kQrCb];
  if (eye) {
#pragma unroll
    for (int q = 0; q < NR; ++q)
#pragma unroll
      for (int c = 0; c < kQrCb; ++c) yv[q][c] = (int)threadIdx.x + kQrThreads * q == cb0 + c ? 1.0 : 0.0;
  } else {
    qr_load_y<NR>(y, m, 0, cb0, ncols, yv);
  }
  const int last = (n - 1) / kQrNb;
  for (int p = eye ? min(last, cb0 / kQrNb) : last; p >= 0; --p) {
    __syncthreads();
    qr_apply<NR>(xc, tf, m, 0, p * kQrNb, min(kQrNb, n - p * kQrNb), yv, sm);
  }
  qr_store_y<NR>(y, m, 0, cb0, ncols, yv);
}

__global__ void qr_reset_kernel(uint32_t* ctr, int words) {
  for (int i = threadIdx.x; i < words; i += blockDim.x) ctr[i] = 0;
}

__global__ void eye_kernel(double* qc, int m, int n, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  const int64_t total = (int64_t)m * n;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t c = e / m, i = e - c * m;
    qc[e] = (i == c) ? 1.0 : 0.0;
  }
}

// site[i, s, b] = Q[(i d + s), b] * sign(R[b, b]);  R_next[r, c] = sign(R[r, r]) * R[r, c] (upper)
// Q with column signs so that diag(R) >= 0, written over the site
__global__ void finalize_q_kernel(const double* __restrict__ xc, const double* __restrict__ qc, double* site, int m,
                                  int n, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  const int64_t total = (int64_t)m * n;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t row = e / n, b = e - row * n;   // row-major site index (row = i*d + s)
    double sg = xc[b * m + b] < 0.0 ? -1.0 : 1.0;
    site[e] = qc[b * m + row] * sg;
  }
}

// R with row signs (diag(R) >= 0), row-major, for the next site's absorb
__global__ void finalize_r_kernel(const double* __restrict__ xc, double* rnext, int m, int n, const uint64_t* cert) {
  if (chol_certified(cert)) return;
  const int64_t tr = (int64_t)n * n;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < tr; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t r = e / n, c = e - r * n;
    double sg = xc[r * m + r] < 0.0 ? -1.0 : 1.0;
    rnext[e] = (c >= r) ? sg * xc[c * m + r] : 0.0;
  }
}

__global__ void lognorm_kernel(const double* r, double* out) {
  if (threadIdx.x == 0) out[0] = log(r[0]);
}

__global__ void one_kernel(double* r) {
  if (threadIdx.x == 0) r[0] = 1.0;
}

static unsigned blocks_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 16384));
}

// Householder QR of a column-major m x n matrix (m >= n) for other callers:
// the blocked path only (m <= 2048), factorised in place (R in the upper
// triangle, the reflectors below), T factors in tf; and the product Q y.
bool householder_qr_fits(int64_t m) { return m <= (int64_t)kQrThreads * kQrRows; }

// the panels' T factors, then the task counters of the factorisation
static size_t qr_tf_doubles(int64_t n) { return (size_t)((n + kQrNb - 1) / kQrNb) * kQrNb * kQrNb; }
static size_t qr_ctr_words(int64_t n) { return 3 + (size_t)qr_panels((int)n); }
size_t householder_tf_doubles(int64_t n) { return qr_tf_doubles(n) + (qr_ctr_words(n) + 1) / 2; }

// a workgroup for the panels and one for every task of the widest application
static int qr_grid(int n) { return std::min(256, qr_panels(n)); }

// Y := Q Y or Q [I; 0], the rows 1, 2 or 4 a thread as in the factorisation (a
// panel's rows start at its first; with 4 a thread throughout, 512 x 512 took
// 2.49 ms to factorise and 0.38 ms here, with 2 then 1 1.91, now 1.09, and 0.21)
static void launch_form(const double* xc, const double* tf, double* y, int m, int n, int ncols, bool eye,
                        const uint64_t* cert, hipStream_t st) {
  const dim3 grid((unsigned)((ncols + kQrCb - 1) / kQrCb)), blk(kQrThreads);
  if (m <= kQrThreads) hipLaunchKernelGGL(qr_form_kernel<1>, grid, blk, 0, st, xc, tf, y, m, n, ncols, eye, cert);
  else if (m <= 2 * kQrThreads) hipLaunchKernelGGL(qr_form_kernel<2>, grid, blk, 0, st, xc, tf, y, m, n, ncols, eye, cert);
  else hipLaunchKernelGGL(qr_form_kernel<kQrRows>, grid, blk, 0, st, xc, tf, y, m, n, ncols, eye, cert);
}

int32_t householder_qr(double* xc, int m, int n, double* tau, double* tf, hipStream_t st) {
  uint32_t* ctr = reinterpret_cast<uint32_t*>(tf + qr_tf_doubles(n));
  hipLaunchKernelGGL(qr_reset_kernel, dim3(1), dim3(256), 0, st, ctr, (int)qr_ctr_words(n));
  hipLaunchKernelGGL(qr_factor_kernel, dim3((unsigned)qr_grid(n)), dim3(kQrThreads), 0, st, xc, tau, tf, m, n, ctr,
                     (const uint64_t*)nullptr);
  return hip_check(hipGetLastError(), "householder qr");
}

// y (m x ncols, column-major) := Q y, the panels applied last to first
int32_t householder_apply_q(const double* xc, int m, int n, const double* tf, double* y, int ncols, hipStream_t st) {
  launch_form(xc, tf, y, m, n, ncols, false, nullptr, st);
  return hip_check(hipGetLastError(), "householder apply");
}

// Sites of at least this many columns are factorised by Cholesky first
// (cholqr.hip); below, the two panels of Householder cost less than its ten
// launches.  Chains of 26 (1024: 24) sites of two states, all certified /
// Householder alone / every site's certificate failing after the attempt: bond
// 32 1.46 / 1.92 / 2.68 ms, 64 1.55 / 3.06 / 3.83, 256 2.47 / 8.4 / 9.75, 1024
// 5.3 / 28.4 / 33.0.
constexpr int kCholMin = 32;

// X, Q and T come in two sets, used by alternate sites: a site's Q is formed
// on the side stream while the next site is factorised
struct QrLayout {
  size_t x[2], q[2], r, tau, tf[2], g, r1, u[2], linv, ebits, total;
};

static int32_t qr_check(int32_t n, const tn_tensor* sites, QrLayout& L) {
  if (n < 1 || !sites) return fail(TN_ERR_INVALID_ARGUMENT, "need n_sites >= 1 and sites");
  int64_t mx = 1, mr = 1;
  int64_t prev = 1;
  for (int k = 0; k < n; ++k) {
    char nm[32];
    snprintf(nm, sizeof(nm), "sites[%d]", k);
    TN_TRY(check_tensor(&sites[k], nm, TN_F64));
    const tn_tensor& t = sites[k];
    if (t.rank != 3) return fail(TN_ERR_SHAPE_MISMATCH, "%s must be rank 3", nm);
    if (t.stride[2] != 1 || t.stride[1] != t.shape[2] || t.stride[0] != t.shape[1] * t.shape[2])
      return fail(TN_ERR_UNSUPPORTED, "%s must be contiguous", nm);
    if (t.shape[0] != prev) return fail(TN_ERR_SHAPE_MISMATCH, "bond %d does not match", k);
    if (t.shape[2] > t.shape[0] * t.shape[1])
      return fail(TN_ERR_UNSUPPORTED, "%s: D_k+1 > d * D_k (wider than the row space)", nm);
    mx = std::max(mx, t.shape[0] * t.shape[1] * t.shape[2]);
    mr = std::max(mr, t.shape[2] * t.shape[2]);
    prev = t.shape[2];
  }
  if (sites[0].shape[0] != 1 || prev != 1) return fail(TN_ERR_SHAPE_MISMATCH, "boundary bonds must be 1");
  size_t o = 0;
  for (int h = 0; h < 2; ++h) {
    L.x[h] = o;
    o += al256(mx * 8);
    L.q[h] = o;
    o += al256(mx * 8);
    L.tf[h] = o;
    o += al256(householder_tf_doubles(4096) * 8);
  }
  L.r = o;
  o += al256(std::max<int64_t>(mr, 1) * 8);
  L.tau = o;
  o += al256(4096 * 8);
  // Cholesky path: the Gram matrix, R1, U and the certificate per set
  for (size_t* p : {&L.g, &L.r1, &L.u[0], &L.u[1]}) {
    *p = o;
    o += al256(std::max<int64_t>(mr, 1) * 8);
  }
  L.linv = o;
  o += al256(kCholLinv * 8);
  L.ebits = o;
  o += al256(2 * 8);
  L.total = o;
  int64_t maxn = 1;
  for (int k = 0; k < n; ++k) maxn = std::max(maxn, sites[k].shape[2]);
  if (maxn > 4096) return fail(TN_ERR_UNSUPPORTED, "bond dimension above 4096");
  return TN_OK;
}

}  // namespace tn

using namespace tn;

extern "C" {

int32_t tn_mps_left_canonicalize_workspace(int32_t n_sites, const tn_tensor* sites, size_t* bytes) {
  if (!bytes) return fail(TN_ERR_INVALID_ARGUMENT, "bytes is NULL");
  QrLayout L;
  TN_TRY(qr_check(n_sites, sites, L));
  *bytes = L.total;
  return TN_OK;
}

int32_t tn_mps_left_canonicalize(int32_t n_sites, tn_tensor* sites, double* lognorm, void* workspace, size_t ws_bytes,
                                 void* stream) {
  QrLayout L;
  TN_TRY(qr_check(n_sites, sites, L));
  if (!lognorm) return fail(TN_ERR_INVALID_ARGUMENT, "lognorm is NULL");
  if (!workspace || ws_bytes < L.total) return fail(TN_ERR_WORKSPACE_TOO_SMALL, "workspace needs %zu bytes", L.total);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  double* r = reinterpret_cast<double*>(ws + L.r);
  double* tau = reinterpret_cast<double*>(ws + L.tau);
  // Site k's factorisation and R run on the caller's stream; its Q (the
  // reflectors applied to [I; 0]) and the write-back run on the side stream,
  // overlapping site k+1's factorisation, whose one-workgroup panels leave
  // most of the chip idle.  Site k+2 reuses site k's X, Q and T only after
  // that Q is done (event per set); the call ends joined on the caller's stream.
  hipStream_t side = st;
  TN_TRY(side_stream(side));
  StreamMark factored, formed[2];
  hipLaunchKernelGGL(one_kernel, dim3(1), dim3(64), 0, st, r);
  int32_t rc = TN_OK;
  for (int k = 0; k < n_sites && rc == TN_OK; ++k) {
    const int h = k & 1;
    double* xc = reinterpret_cast<double*>(ws + L.x[h]);
    double* qc = reinterpret_cast<double*>(ws + L.q[h]);
    double* tf = reinterpret_cast<double*>(ws + L.tf[h]);
    const int dk = (int)sites[k].shape[0], d = (int)sites[k].shape[1], dn = (int)sites[k].shape[2];
    const int m = dk * d, n = dn;
    double* a = static_cast<double*>(sites[k].data);
    rc = formed[h].wait(st);   // site k-2's Q no longer reads this set
    if (rc != TN_OK) break;
    // Cholesky first: the site's X and Q1 take the places of the Householder
    // path's, which then forms its own X again, or leaves at once where the
    // certificate holds
    uint64_t* cert = nullptr;
    double* u = reinterpret_cast<double*>(ws + L.u[h]);
    if (n >= kCholMin && (int64_t)m * n < (1 << 28)) {
      cert = reinterpret_cast<uint64_t*>(ws + L.ebits) + h;
      rc = chol_absorb(r, a, xc, dk, d * dn, st);
      if (rc == TN_OK)
        rc = chol_qr(xc, m, n, reinterpret_cast<double*>(ws + L.g), reinterpret_cast<double*>(ws + L.r1), u, qc,
                     reinterpret_cast<double*>(ws + L.linv), cert, r, st);
      if (rc != TN_OK) break;
    }
    dim3 g((unsigned)((d * dn + 63) / 64), (unsigned)((dk + 63) / 64));
    hipLaunchKernelGGL(absorb_kernel, g, dim3(256), 0, st, r, a, xc, dk, d, dn,
                       reinterpret_cast<uint32_t*>(tf + qr_tf_doubles(n)), (int)qr_ctr_words(n), cert);
    const bool blocked = m <= kQrThreads * kQrRows;
    if (blocked) {
      hipLaunchKernelGGL(qr_factor_kernel, dim3((unsigned)qr_grid(n)), dim3(kQrThreads), 0, st, xc, tau, tf, m, n,
                         reinterpret_cast<uint32_t*>(tf + qr_tf_doubles(n)), cert);
    } else {
      for (int j = 0; j < n; ++j) {
        hipLaunchKernelGGL(reflector_kernel, dim3(1), dim3(256), 0, st, xc, tau, m, j, cert);
        if (j + 1 < n) hipLaunchKernelGGL(reflect_cols_kernel, dim3(n - j - 1), dim3(256), 0, st, xc, tau, xc, m, j, j + 1, cert);
      }
    }
    hipLaunchKernelGGL(finalize_r_kernel, dim3(blocks_for((int64_t)n * n)), dim3(256), 0, st, xc, r, m, n, cert);
    // Q: on the side stream for the blocked path; the column path's Q needs
    // tau, which the next site overwrites, so it stays on the caller's stream
    hipStream_t qs = blocked ? side : st;
    if (blocked) {
      rc = factored.set(st);
      if (rc == TN_OK) rc = factored.wait(side);
    }
    if (rc == TN_OK && cert) rc = chol_q(qc, u, a, m, n, cert, qs);
    if (rc != TN_OK) break;
    if (blocked) {
      launch_form(xc, tf, qc, m, n, n, true, cert, qs);
    } else {
      hipLaunchKernelGGL(eye_kernel, dim3(blocks_for((int64_t)m * n)), dim3(256), 0, qs, qc, m, n, cert);
      for (int j = n - 1; j >= 0; --j)
        hipLaunchKernelGGL(reflect_cols_kernel, dim3(n - j), dim3(256), 0, qs, xc, tau, qc, m, j, j, cert);
    }
    hipLaunchKernelGGL(finalize_q_kernel, dim3(blocks_for((int64_t)m * n)), dim3(256), 0, qs, xc, qc, a, m, n, cert);
    rc = hip_check(hipGetLastError(), "canonicalize");
    const int32_t set = formed[h].set(qs);
    if (rc == TN_OK) rc = set;
  }
  // join: every Q written back before the call's later work on the caller's stream
  for (const StreamMark& q : formed) {
    const int32_t joined = q.wait(st);
    if (rc == TN_OK) rc = joined;
  }
  TN_TRY(rc);
  hipLaunchKernelGGL(lognorm_kernel, dim3(1), dim3(64), 0, st, r, lognorm);
  return hip_check(hipGetLastError(), "lognorm");
}

}  // extern "C"
