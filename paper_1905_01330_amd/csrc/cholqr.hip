// QR of a site by Cholesky factorisation, for the left-canonical gauge: the
// tall matrix X (m x n, row-major, as a site is stored) is orthogonalised by
// its Gram matrix, R1^T R1 = X^T X and Q1 = X R1^-1 (the triangle is unique
// with a positive diagonal, so R and Q are those of the Householder
// factorisation), and corrected once: with E = Q1^T Q1 - I and U its upper
// triangle with half the diagonal,
//   Q = Q1 (I - U),  R = (I + U) R1
// are exact to second order in E (Yamamoto, Nakatsukasa, Yanagisawa and
// Fukaya, ETNA 44, 2015, for the two passes; the second one's factor is
// I + U + O(E^2)).
//
// Certificate: max |E| is taken over the computed Q1^T Q1.  Up to kMaxE (less
// for more than kMaxEn columns) the neglected terms stay below an FP64
// rounding; above it, or with a NaN (a pivot that is not positive, an
// overflow), the site is left to the Householder kernels.  Both sets of kernels
// are always launched and look at the certificate on the device: no host
// synchronisation, capturable.
//
// Everything is FP64 matrix-core work on the whole chip, 64 columns at a
// time; the Householder panels are a chain of one workgroup's reductions over
// the rows, one a column.  A chain of 28 sites of two states and bond 1024:
// 58.1 ms by Householder panels, 8.4 ms here.
#include "cholqr.h"

namespace tn {

typedef double d64x4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// products

enum CholOp { C_ABSORB, C_GRAM, C_DEFECT, C_TRIANGLE, C_Q };

struct CholGemm {
  const double* a;
  const double* b;
  const double* base;   // C_TRIANGLE: R1, C_Q: Q1
  double* c;
  int M, N, K, lda, ldb, ldc;
  uint64_t* ebits;
};

// a raw buffer of 2^31 bytes
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chol_rsrc(const double* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), (short)0, (int)0x80000000, 0x00020000);
}

// C with
//   C_ABSORB:   C = A B, A upper triangular (K from the row)
//   C_GRAM:     C = A^T B, the upper triangle's tiles
//   C_DEFECT:   U of A^T B - I, and max |E| into ebits
//   C_TRIANGLE: C = base + A B, all triangles upper, zero below (where certified)
//   C_Q:        C = base - A B, B upper triangular (where certified)
// A workgroup of eight waves owns a tile of 16 NB squared and cuts K over its
// waves, 16 k a wave and turn.  The operands go from memory straight into the
// matrix cores' registers, up to two turns ahead: no barrier before the sums.
// An instruction reads whole lines: four rows of 128 bytes where k is the
// outer index, 16 rows of 32 bytes in two halves where it is the inner one (a
// lane's four k are neighbours, the same four in both operands).  Bound by
// what a compute unit reads, 17 to 20 KB a us (the matrix cores would take
// twice that), so by the tile's side.  At 1024 columns, 2048 rows: the Gram
// matrix's triangle 94 us in tiles of 48, A B 76 to 82 and base - A B beside
// it in tiles of 64 (a site's absorb, Q and Gram 258 us staged through LDS in
// 32 x 64 tiles, 198 here; the defect 105 and 83, the triangle 47 and 30).
template <int OP, int NB>
__global__ void __launch_bounds__(512) chol_gemm_kernel(const CholGemm p) {
  constexpr bool TN = OP == C_GRAM || OP == C_DEFECT;   // A stored k x m
  constexpr bool TRI = OP == C_TRIANGLE || OP == C_Q;   // R1's blocks below the diagonal are not written: B reads zero there
  constexpr int T = 16 * NB, D = NB < 4 ? 2 : 1;   // turns in flight: 256 registers a wave
  __shared__ double red[8][4 * NB][64];
  __shared__ uint64_t smax[8];
  if constexpr (TRI) {
    if (!chol_certified(p.ebits)) return;
  }
  // the longest sums first
  const int m0 = (int)blockIdx.y * T, n0 = (int)(TRI ? gridDim.x - 1 - blockIdx.x : blockIdx.x) * T;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, lk = lane >> 4;
  if (TN && n0 + T <= m0) {
    // U's other half is zero: reads past the end of a row of it meet zeros of
    // the other operand, which what the workspace held before need not survive
    if constexpr (OP == C_DEFECT)
      for (int e = threadIdx.x; e < T * T; e += 512) {
        const int m = m0 + e / T, n = n0 + e % T;
        if (m < p.M && n < p.N) p.c[(int64_t)m * p.ldc + n] = 0.0;
      }
    return;
  }
  int kb = 0, ke = p.K;
  if (OP == C_ABSORB || OP == C_TRIANGLE) kb = m0;
  if (TRI) ke = min(p.K, n0 + T);
  // Raw buffers of exactly a matrix (below 2^31 bytes): what lies past it reads
  // zero, so no load has a guard, behind which the loads of a turn would wait
  // for each other.  Columns past M or N read the next row's values and are
  // not stored; A's k past K, where they run along a row, meet B's zeros.
  auto rsrc = [](const double* q, int64_t count) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(q), (short)0, (int)(count * 8), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t qa = rsrc(p.a, (int64_t)(TN ? p.K : p.M) * p.lda), qb = rsrc(p.b, (int64_t)p.K * p.ldb);
  typedef double d2_t __attribute__((ext_vector_type(2)));
  constexpr int NA = TN ? 4 : NB;
  uint32_t oa[NA], ob[4];   // byte offsets of the next turn
  const int k0 = kb + wave * 16 + 4 * lk;
  int kt = k0;
#pragma unroll
  for (int j = 0; j < 4; ++j) ob[j] = ((uint32_t)(k0 + j) * (uint32_t)p.ldb + (uint32_t)(n0 + l15)) * 8u;
#pragma unroll
  for (int j = 0; j < NA; ++j)
    oa[j] = TN ? ((uint32_t)(k0 + j) * (uint32_t)p.lda + (uint32_t)(m0 + l15)) * 8u
               : ((uint32_t)(m0 + 16 * j + l15) * (uint32_t)p.lda + (uint32_t)k0) * 8u;
  const uint32_t ia = 128u * 8u * (TN ? (uint32_t)p.lda : 1u), ib = 128u * 8u * (uint32_t)p.ldb;
  double a[D][NB][4], b[D][NB][4];
  auto load = [&](double (&xa)[NB][4], double (&xb)[NB][4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        uint32_t at = ob[j] + 128u * t;
        if constexpr (TRI) at = kt + j <= n0 + 16 * t + l15 ? at : 0x80000000u;
        xb[t][j] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(qb, at, 0, 0));
      }
    if constexpr (TN) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < NB; ++t)
          xa[t][j] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(qa, oa[j] + 128u * t, 0, 0));
    } else {
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
          const d2_t v = __builtin_bit_cast(d2_t, __builtin_amdgcn_raw_buffer_load_b128(qa, oa[t] + 8u * j, 0, 0));
          xa[t][j] = v[0];
          xa[t][j + 1] = v[1];
        }
    }
    kt += 128;
#pragma unroll
    for (int j = 0; j < 4; ++j) ob[j] += ib;
#pragma unroll
    for (int j = 0; j < NA; ++j) oa[j] += ia;
  };
  d64x4_t acc[NB][NB] = {};
  const int turns = (ke - kb + 127) / 128;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load(a[d], b[d]);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int turn = 0; turn < turns; turn += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int y = 0; y < NB; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][x][j], b[d][y][j], acc[x][y], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);   // a set's loads in one place, a turn ahead of their use
      load(a[d], b[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the waves' sums, a row of blocks at a time: wave w adds registers w and w + 8
  // FP64 16x16x4 result: lane (column l15) register r holds row 4 r + lk
  uint64_t emax = 0;
#pragma unroll
  for (int x = 0; x < NB; ++x) {
    if (x > 0) __syncthreads();
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][4 * y + r][lane] = acc[x][y][r];
    __syncthreads();
    for (int e = wave; e < 4 * NB; e += 8) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) v += red[w][e][lane];
      const int m = m0 + 16 * x + 4 * (e & 3) + lk, n = n0 + 16 * (e >> 2) + l15;
      if (m >= p.M || n >= p.N) continue;
      const int64_t at = (int64_t)m * p.ldc + n;
      if constexpr (OP == C_DEFECT) {
        if (m == n) v -= 1.0;
        if (n >= m) emax = max(emax, (uint64_t)__double_as_longlong(fabs(v)));
        v = n > m ? v : n == m ? 0.5 * v : 0.0;
      } else if constexpr (OP == C_TRIANGLE) {
        v = n >= m ? p.base[at] + v : 0.0;
      } else if constexpr (OP == C_Q) {
        v = p.base[at] - v;
      }
      p.c[at] = v;
    }
  }
  if constexpr (OP == C_DEFECT) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) emax = max(emax, (uint64_t)__shfl_xor((unsigned long long)emax, o, 64));
    if (lane == 0) smax[wave] = emax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int w = 1; w < 8; ++w) emax = max(emax, smax[w]);
      // by the width, towards the limit of kMaxEn columns (a NaN stays one)
      emax = __double_as_longlong(fabs(__longlong_as_double(emax) * max(1.0, p.N * (1.0 / kMaxEn))));
      atomicMax((unsigned long long*)p.ebits, (unsigned long long)emax);
    }
  }
}

// ---------------------------------------------------------------------------
// blocked Cholesky with the triangular solve of X carried along: step k takes
// the 64 columns of block k out of the trailing columns of G and X,
//   P_j = L G_kj (L = R_kk^-T), Q_t = X_tk L^T, G_ij -= P_i^T P_j, X_tj -= Q_t P_j.
// One launch a step; a workgroup owns one 64 x 64 tile (i, j) of G or (t, j)
// of X and forms the P and Q it needs itself (three products of 64^3; the
// matrix cores of the chip are idle otherwise, and a launch less costs more
// than they do).  The tile (k + 1, k + 1) then factorises its result for the
// next step.

// Q_t = X_tk L^T leaves a residual X_tk - Q_t R_kk of the rounding of L times
// the condition of the block R_kk, which no correction by E takes back.  Where
// |R_kk|_F |L|_F, 64 for an orthogonal block, is above kRefine, X's tiles
// therefore solve for it once more, Q_t += (X_tk - Q_t R_kk) L^T.  Sites of 33
// to 100 columns and conditions to 300: |Q R - X| up to 11 sqrt(n) eps of a
// column without it, 0.8 with it, 0.6 by Householder; Q up to five times as far
// from the exact one as Householder's, and as near with it.  Sites near an
// isometry take none.
constexpr double kRefine = 128.0;

constexpr int kCb = 64;                  // block
constexpr int kCholSlot = kCb * kCb + 16;   // doubles of one block's L and sums
constexpr int kPk = 66;                  // LDS pitch of operands read along k (rows 16 bytes apart mod 256)
constexpr int kPn = 80;                  // pitch of operands read along the other index
constexpr int kCholThreads = 512;

struct CholStep {
  double* g;        // n x n
  double* x;        // m x n
  double* q;        // Q1, m x n
  double* r;        // R1, n x n
  double* linv;     // L of the current block (64 x 64) and its sums; the next one's go to linv2
  double* linv2;
  uint64_t* ebits;
  int m, n, k, nb, tr;   // rows, columns, step (-1: factorise block 0), column blocks, row blocks of X
};

// 64 x 64 product of two LDS operands, waves of 16 rows x 32 columns:
// A at a + row * ar + k * ak, B at b + k * bk + col * bc
__device__ __forceinline__ void chol_product(const double* a, int ar, int ak, const double* b, int bk, int bc,
                                             d64x4_t (&acc)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, lk = lane >> 4;
  const double* pa = a + ((wave & 3) * 16 + l15) * ar + lk * ak;
  const double* pb = b + lk * bk + ((wave >> 2) * 32 + l15) * bc;
  acc[0] = acc[1] = d64x4_t{};
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) {
    const double av = pa[4 * kk * ak];
#pragma unroll
    for (int q = 0; q < 2; ++q)
      acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, pb[4 * kk * bk + 16 * q * bc], acc[q], 0, 0, 0);
  }
}

// f(row, column, value) over a wave's results
template <class F>
__device__ __forceinline__ void chol_each(const d64x4_t (&acc)[2], F&& f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) f((wave & 3) * 16 + 4 * r + (lane >> 4), (wave >> 2) * 32 + 16 * q + (lane & 15), acc[q][r]);
}

__device__ __forceinline__ double chol_lane(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

template <int CTRL>
__device__ __forceinline__ double chol_dpp(double x) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false));
}
// the sum over a wave, in every lane
__device__ __forceinline__ double chol_wave_sum(double x) {
  x += chol_dpp<0x128>(x);   // row_ror 8, 4, 2, 1
  x += chol_dpp<0x124>(x);
  x += chol_dpp<0x122>(x);
  x += chol_dpp<0x121>(x);
  return (chol_lane(x, 0) + chol_lane(x, 16)) + (chol_lane(x, 32) + chol_lane(x, 48));
}

// R and L = R^-T of the 64 x 64 matrix in tm (pitch kPn, upper triangle read):
// R back into tm, L into ym (pitch kPn).  Blocks of 16: the first wave
// eliminates the diagonal block and updates the next one, straight on to its
// elimination, while the others take the rest of the trailing rows as 16 x 16
// products; block rows by four waves.  The elimination has a column a lane,
// with the identity's columns on the next sixteen lanes ([G I] turns into
// [R L]); its chain from pivot to pivot is 1 / sqrt (the hardware's estimate
// and one step of third order; NaN where a pivot is not positive and finite,
// which fails the certificate), the row, and the next pivot from its own lane.
// (All in turn, two steps of second order: 5700 of 8200 cycles a block of 16
// in the elimination, 33000 in all; now 4500 and 24500.)
__device__ __forceinline__ void chol_factor(double* tm, double* ym, double* dm) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, lk = lane >> 4;
  for (int e = threadIdx.x; e < 64 * 64; e += kCholThreads) ym[(e >> 6) * kPn + (e & 63)] = (e >> 6) == (e & 63) ? 1.0 : 0.0;
  // C (16 x 16) = A^T-or-A B, A at a + k * ak + row * ar, B at b + k * kPn + col
  auto block = [&](const double* a, int ar, int ak, const double* b) {
    d64x4_t c = {};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(4 * kk + lk) * ak + l15 * ar], b[(4 * kk + lk) * kPn + l15], c, 0, 0, 0);
    return c;
  };
  for (int b = 0; b < 4; ++b) {
    const int r0 = 16 * b;
    if (wave == 0) {
      double g[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        g[i] = lane < 16 ? tm[(r0 + i) * kPn + r0 + lane] : (i == l15 ? 1.0 : 0.0);
      double d = chol_lane(g[0], 0);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        double y = __builtin_amdgcn_rsq(d);
        const double e = fma(-(d * y), y, 1.0);
        y = fma(y * e, fma(0.375, e, 0.5), y);
        const double r = g[k] * y;
        g[k] = r;
        if (k < 15) d = chol_lane(fma(-r, r, g[k + 1]), k + 1);
#pragma unroll
        for (int i = k + 1; i < 16; ++i) g[i] = fma(-chol_lane(r, i), r, g[i]);
      }
      if (lane < 16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) tm[(r0 + i) * kPn + r0 + lane] = i <= lane ? g[i] : 0.0;
      } else if (lane < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i) dm[i * 18 + l15] = i >= l15 ? g[i] : 0.0;
      }
    }
    __syncthreads();
    // block row b: R_b,cb = D T_b,cb (cb > b), L_b,cb = D Y_b,cb (cb <= b), a wave its own block
    if (wave < 4) {
      double* row = (wave > b ? tm : ym) + r0 * kPn + 16 * wave;
      const d64x4_t c = block(dm, 18, 1, row);
#pragma unroll
      for (int r = 0; r < 4; ++r) row[(4 * r + lk) * kPn + l15] = c[r];
    }
    __syncthreads();
    // trailing rows ib > b: T_ib,cb -= R_b,ib^T R_b,cb (cb >= ib), Y_ib,cb -= R_b,ib^T L_b,cb (cb <= b)
    int job = 0;
    for (int ib = b + 1; ib < 4; ++ib)
      for (int cb = 0; cb < 4; ++cb) {
        if (cb > b && cb < ib) continue;
        const int who = ib == b + 1 && cb == ib ? 0 : 1 + job++ % 7;
        if (who != wave) continue;
        double* src = (cb > b ? tm : ym) + r0 * kPn + 16 * cb;
        double* dst = (cb > b ? tm : ym) + 16 * ib * kPn + 16 * cb;
        const d64x4_t u = block(tm + r0 * kPn + 16 * ib, 1, kPn, src);
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(4 * r + lk) * kPn + l15] -= u[r];
      }
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kCholThreads) chol_step_kernel(const CholStep p) {
  __shared__ double sl[64 * kPk];           // L of the step
  __shared__ double s1[64 * kPn], s2[64 * kPn];
  __shared__ double dm[16 * 18];
  const int n = p.n, k0 = p.k * kCb;
  int id = blockIdx.x;
  if (p.k < 0) {   // block 0 only
    if (threadIdx.x == 0) *p.ebits = 0;
    for (int e = threadIdx.x; e < 64 * 64; e += kCholThreads) {
      const int i = e >> 6, j = e & 63;
      s1[i * kPn + j] = i < n && j < n ? (j >= i ? p.g[(int64_t)i * n + j] : 0.0) : (i == j ? 1.0 : 0.0);
    }
    __syncthreads();
  } else {
    // tile of the trailing columns: (i, j) of G, i <= j, then (t, j) of X
    const int left = p.nb - 1 - p.k, tri = left * (left + 1) / 2;
    const bool in_g = id < tri;
    int ti, tj;
    if (in_g) {
      tj = (int)((sqrtf(8.0f * id + 1.0f) - 1.0f) * 0.5f);
      while ((tj + 1) * (tj + 2) / 2 <= id) ++tj;
      while (tj * (tj + 1) / 2 > id) --tj;
      ti = id - tj * (tj + 1) / 2;
    } else {
      id -= tri;
      ti = id % p.tr;
      tj = id / p.tr;
    }
    const int j0 = (p.k + 1 + tj) * kCb;                              // columns of the tile
    const int i0 = in_g ? (p.k + 1 + ti) * kCb : ti * kCb;            // its rows
    const bool solve_only = left == 0;                                // the last block: Q alone
    // 64 x 64 blocks of rows r0.. and columns c0.., zero past the matrix: all
    // loads, then all stores
    auto fetch = [&](const double* src, int rows, int r0, int c0, double (&v)[8]) {
      const __amdgpu_buffer_rsrc_t rs = chol_rsrc(src);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = r0 + (threadIdx.x >> 6) + 8 * e, j = c0 + (threadIdx.x & 63);
        v[e] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                              rs, i < rows && j < n ? (uint32_t)(i * n + j) * 8u : 0x80000000u, 0, 0));
      }
    };
    auto put = [&](double* dst, int pitch, const double (&v)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) dst[((threadIdx.x >> 6) + 8 * e) * pitch + (threadIdx.x & 63)] = v[e];
    };
    double vl[8], v1[8], v2[8], vc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) vl[e] = p.linv[threadIdx.x + kCholThreads * e];
    double fl = 0.0, fr = 0.0;   // |L|_F^2, |R_kk|_F^2
    if (!in_g) {
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        fl += p.linv[kCb * kCb + w];
        fr += p.linv[kCb * kCb + 8 + w];
      }
    }
    if (!solve_only) fetch(p.g, n, k0, j0, v1);
    if (!in_g) fetch(p.x, p.m, i0, k0, v2);
    else if (ti != tj) fetch(p.g, n, k0, i0, v2);
    put(sl, kPk, vl);
    if (!solve_only) put(s1, kPn, v1);
    if (!in_g) put(s2, kPk, v2);
    else if (ti != tj) put(s2, kPn, v2);
    __syncthreads();
    // the tile itself, in the layout of the products' results
    if (!solve_only) {
      const __amdgpu_buffer_rsrc_t rs = chol_rsrc(in_g ? p.g : p.x);
      const int rows = in_g ? n : p.m, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + (wave & 3) * 16 + 4 * r + (lane >> 4), j = j0 + (wave >> 2) * 32 + 16 * q + (lane & 15);
          vc[4 * q + r] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                                         rs, i < rows && j < n ? (uint32_t)(i * n + j) * 8u : 0x80000000u, 0, 0));
        }
    }
    d64x4_t pj[2], pi[2];
    if (!solve_only) chol_product(sl, kPk, 1, s1, kPn, 1, pj);                    // P_j = L G_kj
    if (!in_g) chol_product(s2, kPk, 1, sl, 1, kPk, pi);                          // Q_t = X_tk L^T
    else if (ti != tj) chol_product(sl, kPk, 1, s2, kPn, 1, pi);                  // P_i
    __syncthreads();
    if (!in_g && fl * fr > kRefine * kRefine) {
      // a thread reads and writes its own entries of s2: X, Q, then the residual
      double vr[8], vx[8];
      fetch(p.r, n, k0, k0, vr);
      int at = 0;
      chol_each(pi, [&](int r, int c, double v) {
        vx[at++] = s2[r * kPk + c];
        s2[r * kPk + c] = v;
      });
      put(s1, kPn, vr);
      __syncthreads();
      d64x4_t t[2];
      chol_product(s2, kPk, 1, s1, kPn, 1, t);   // Q_t R_kk
      __syncthreads();
      at = 0;
      chol_each(t, [&](int r, int c, double v) { s2[r * kPk + c] = vx[at++] - v; });
      __syncthreads();
      chol_product(s2, kPk, 1, sl, 1, kPk, t);
#pragma unroll
      for (int q = 0; q < 2; ++q) pi[q] += t[q];
      __syncthreads();
    }
    if (!solve_only) chol_each(pj, [&](int r, int c, double v) { s1[r * kPn + c] = v; });
    if (!in_g) {
      chol_each(pi, [&](int r, int c, double v) {
        s2[r * kPk + c] = v;
        if (tj == 0 && i0 + r < p.m && k0 + c < n) p.q[(int64_t)(i0 + r) * n + k0 + c] = v;
      });
      if (solve_only) return;
    } else if (ti != tj) {
      chol_each(pi, [&](int r, int c, double v) { s2[r * kPn + c] = v; });
    } else {
      // the diagonal tiles write their columns of block row k of R
      chol_each(pj, [&](int r, int c, double v) {
        if (k0 + r < n && j0 + c < n) p.r[(int64_t)(k0 + r) * n + j0 + c] = v;
      });
    }
    __syncthreads();
    d64x4_t u[2];
    if (in_g) chol_product(ti == tj ? s1 : s2, 1, kPn, s1, kPn, 1, u);            // P_i^T P_j
    else chol_product(s2, kPk, 1, s1, kPn, 1, u);                                 // Q_t P_j
    double* c = in_g ? p.g : p.x;
    const int rows = in_g ? n : p.m;
    const bool next = in_g && ti == 0 && tj == 0;
    if (next) __syncthreads();   // s1 is read until here
    int at = 0;
    chol_each(u, [&](int r, int cc, double v) {
      const double y = vc[at++] - v;
      const bool inside = i0 + r < rows && j0 + cc < n;
      if (inside) c[(int64_t)(i0 + r) * n + j0 + cc] = y;
      // the next diagonal block, bordered by the identity past the last column
      if (next) s1[r * kPn + cc] = inside ? (cc >= r ? y : 0.0) : (r == cc ? 1.0 : 0.0);
    });
    if (!next) return;
    __syncthreads();
  }
  chol_factor(s1, s2, dm);
  const int d0 = (p.k + 1) * kCb;
  double fl = 0.0, fr = 0.0;
  for (int e = threadIdx.x; e < 64 * 64; e += kCholThreads) {
    const int i = e >> 6, j = e & 63;
    const double l = j <= i ? s2[i * kPn + j] : 0.0, r = j >= i ? s1[i * kPn + j] : 0.0;
    p.linv2[e] = l;
    if (d0 + i < n && d0 + j < n) p.r[(int64_t)(d0 + i) * n + d0 + j] = r;
    fl += l * l;
    fr += r * r;
  }
  fl = chol_wave_sum(fl);
  fr = chol_wave_sum(fr);
  if ((threadIdx.x & 63) == 0) {
    p.linv2[kCb * kCb + (threadIdx.x >> 6)] = fl;
    p.linv2[kCb * kCb + 8 + (threadIdx.x >> 6)] = fr;
  }
}

// ---------------------------------------------------------------------------

// Tiles of 32, 48 or 64, whichever has the busiest compute unit read least:
// a tile's bytes go with its side, and they bound it
template <int OP>
static void chol_gemm(const CholGemm& p, hipStream_t st) {
  auto load = [&](int64_t t) {
    const int64_t tm = (p.M + t - 1) / t, tn = (p.N + t - 1) / t;
    const int64_t tiles = OP == C_GRAM || OP == C_DEFECT || OP == C_TRIANGLE ? tm * (tm + 1) / 2 : tm * tn;
    return (tiles + 255) / 256 * t;
  };
  auto grid = [&](int t) { return dim3((unsigned)((p.N + t - 1) / t), (unsigned)((p.M + t - 1) / t)); };
  const int64_t l2 = load(32), l3 = load(48), l4 = load(64);
  if (l2 <= l3 && l2 <= l4) hipLaunchKernelGGL((chol_gemm_kernel<OP, 2>), grid(32), dim3(512), 0, st, p);
  else if (l3 <= l4) hipLaunchKernelGGL((chol_gemm_kernel<OP, 3>), grid(48), dim3(512), 0, st, p);
  else hipLaunchKernelGGL((chol_gemm_kernel<OP, 4>), grid(64), dim3(512), 0, st, p);
}

int32_t chol_absorb(const double* r, const double* a, double* x, int dk, int cols, hipStream_t st) {
  chol_gemm<C_ABSORB>({r, a, nullptr, x, dk, cols, dk, dk, cols, cols, nullptr}, st);
  return hip_check(hipGetLastError(), "absorb");
}

int32_t chol_qr(double* x, int m, int n, double* g, double* r1, double* u, double* q1, double* linv, uint64_t* ebits,
                double* r, hipStream_t st) {
  chol_gemm<C_GRAM>({x, x, nullptr, g, n, n, m, n, n, n, nullptr}, st);
  CholStep s;
  s.g = g;
  s.x = x;
  s.q = q1;
  s.r = r1;
  s.ebits = ebits;
  s.m = m;
  s.n = n;
  s.nb = (n + kCb - 1) / kCb;
  s.tr = (m + kCb - 1) / kCb;
  for (int k = -1; k < s.nb; ++k) {
    s.k = k;
    s.linv = linv + (k & 1) * kCholSlot;
    s.linv2 = linv + ((k + 1) & 1) * kCholSlot;
    const int left = s.nb - 1 - k;
    const int tiles = k < 0 ? 1 : left == 0 ? s.tr : left * (left + 1) / 2 + s.tr * left;
    hipLaunchKernelGGL(chol_step_kernel, dim3((unsigned)tiles), dim3(kCholThreads), 0, st, s);
  }
  chol_gemm<C_DEFECT>({q1, q1, nullptr, u, n, n, m, n, n, n, ebits}, st);
  chol_gemm<C_TRIANGLE>({u, r1, r1, r, n, n, n, n, n, n, ebits}, st);
  return hip_check(hipGetLastError(), "cholesky qr");
}

int32_t chol_q(const double* q1, const double* u, double* site, int m, int n, uint64_t* ebits, hipStream_t st) {
  chol_gemm<C_Q>({q1, u, q1, site, m, n, n, n, n, n, ebits}, st);
  return hip_check(hipGetLastError(), "cholesky q");
}

}  // namespace tn
