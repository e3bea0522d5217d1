// Jacobi sweeps for the node split that rotate the Gram matrix of the columns
// and not the columns themselves.
//
// A sweep of one-sided Jacobi is a chain of rotations, each taken from dot
// products over the rows and applied to them: at 512 columns 127 launches of
// 14.5 us, seven dependent steps each, 1.84 ms.  Here a sweep
//   1. forms G = X^T X once (jac_gram),
//   2. walks through all pairs of 16-column blocks by the circle method, a
//      launch a round (jac_round_kernel): the 32 x 32 subproblem of every
//      block pair is rotated in LDS by one workgroup, its rotations J are
//      collected, and G <- J^T G J, Js <- Js J run as matrix-core products,
//   3. applies the collected rotations, X <- X Js and V <- V Js, as products
//      on the whole chip (jac_gemm_kernel).
// The chain is one LDS step a rotation (0.45 us) and a launch a round (5.5 us
// beside its steps): 31 rounds of 13 and 20 us at 512 columns, 0.48 ms a sweep
// with the products and the check; 512 x 512 as a whole 24.9 -> 6.6 ms, 1000 x 1000
// 77 -> 17.8 ms.
//
// Accuracy.  G is formed anew from the columns before each sweep, and the
// columns' orthogonality is judged on it with the same bound as the
// column-wise sweeps use (|g_ij| <= tol |x_i| |x_j|); within a sweep G only
// chooses the angles.  A rotation is applied as x - s (y + u x),
// y + s (x - u y) with u = tan(angle / 2), s = 2 u / (1 + u^2): what it
// rounds is proportional to s, so the small rotations of the late sweeps do
// not wear the orthogonality of V (1e-14 after ten sweeps over 512 columns;
// 4e-13 with c x - s y).  Columns are taken in the order of their norms, and
// J is then graded like them, which keeps small columns accurate next to
// large ones through the products.
#include <type_traits>

#include "jacobi.h"

namespace tn {

namespace {

typedef double d64x4_t __attribute__((ext_vector_type(4)));

constexpr int kJacP = 2 * kJacB;
constexpr int kJacJ = kJacP * kJacP;

// round `round` of the circle method over nb blocks (even): the blocks of pair `pair`
__device__ __forceinline__ void jac_blocks(int nb, int round, int pair, int& p, int& q) {
  const int m = nb - 1, hi = round + pair, lo = round - pair;   // round < m, pair < nb / 2
  p = pair == 0 ? m : hi >= m ? hi - m : hi;
  q = lo < 0 ? lo + m : lo;
}
// and the pair and half (0: first) that block x has in it
__device__ __forceinline__ void jac_where(int nb, int round, int x, int& pair, int& half) {
  const int m = nb - 1;
  const int d = x - round, i = d < 0 ? d + m : d;   // x < m, else unused
  pair = x == m || i == 0 ? 0 : i < nb / 2 ? i : m - i;
  half = x == m ? 0 : i == 0 || i >= nb / 2 ? 1 : 0;
}

// Rotation by the angle that annihilates a_pq: s = sin(angle) and
// u = tan(angle / 2).  With cos(2 angle) = |d| / r, r^2 = d^2 + b^2, the angle
// is taken in single precision from values scaled to one (1e-7 of a_pq stays,
// where convergence is quadratic anyway), but for its factor b: between columns
// of very different norms the angle is far below the smallest float.
// s = 2 u / (1 + u^2) belongs to u to double precision, one step from
// (1 + cos(angle)) / 2 = 1 / (1 + u^2).  Whether to rotate is asked of the
// scaled values too: the products of entries of small columns would vanish.
__device__ __forceinline__ void jac_angle(double app, double aqq, double apq, double tol2, double& s, double& u) {
  const double d = aqq - app, b = 2.0 * apq;
  // 2^-(exponent of the larger); entries of G are at most 1
  const int e = max(__double2hiint(d) & 0x7ff00000, __double2hiint(b) & 0x7ff00000);
  const double scale = __hiloint2double(0x7fe00000 - e, 0);
  const double bs = b * scale;
  // (where d and b are far below the entries their scaled product is infinite, and that is orthogonal)
  const bool rot = bs * bs > 4.0 * tol2 * fabs((app * scale) * (aqq * scale));
  const float fd = fabsf((float)(d * scale)), fb = (float)bs;
  const float y = __builtin_amdgcn_rsqf(fd * fd + fb * fb);
  const float half = 0.5f + 0.5f * (fd * y);
  const float z = __builtin_amdgcn_rsqf(half);
  const float c1 = 1.0f + half * z;   // 1 + cos(angle)
  const float h = 0.5f * y * z * __builtin_amdgcn_rcpf(c1);
  u = rot ? __hiloint2double(__double2hiint(bs) ^ (__double2hiint(d) & 0x80000000), __double2loint(bs)) * (double)h : 0.0;
  const double w = 1.0 + u * u;
  double r = rot ? (double)(0.5f * c1) : 1.0;
  const double f = 1.0 - w * r;
  r += r * (f + f * f);
  s = 2.0 * u * r;
}
// x of lane `lk` of the lane's row of 16 (lk: the row)
__device__ __forceinline__ int jac_bcast(int x) {
  int r = x;
  r = __builtin_amdgcn_update_dpp(r, x, 0x150, 0x1, 0xf, false);   // row_newbcast:0 in row 0, ...
  r = __builtin_amdgcn_update_dpp(r, x, 0x151, 0x2, 0xf, false);
  r = __builtin_amdgcn_update_dpp(r, x, 0x152, 0x4, 0xf, false);
  r = __builtin_amdgcn_update_dpp(r, x, 0x153, 0x8, 0xf, false);
  return r;
}
__device__ __forceinline__ double jac_bcast(double x) {
  return __hiloint2double(jac_bcast(__double2hiint(x)), jac_bcast(__double2loint(x)));
}
__device__ __forceinline__ void jac_rotate(double& x, double& y, double s, double u) {
  const double a = x - s * (y + u * x), b = y + s * (x - u * y);
  x = a;
  y = b;
}

struct JacRound {
  const double* g;      // G before the last round's rotations (round 0: as formed)
  double* gnext;
  const double* jlast;  // the last round's rotations, one 32 x 32 a pair
  double* jthis;
  double* js;           // cp x cp, row-major: the order's permutation and the sweep's rotations so far
  const int* perm;
  const int* ctl;       // zero: nothing to rotate
  int cp, nb, round, rounds;
  double tol2;
};

// Columns h of a pair's 32 x 32 rotations as a matrix-core operand (as the
// right one, or transposed as the left one)
__device__ __forceinline__ void jac_cols(const double* j, int h, int l15, int lk, double (&o)[8]) {
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) o[kk] = j[(4 * kk + lk) * kJacP + 16 * h + l15];
}
// The 32 x 32 block T of g at block rows (pa, qa) and block columns (pb, qb) as a left operand
__device__ __forceinline__ void jac_tile(const double* g, int cp, int pa, int qa, int pb, int qb, int l15, int lk,
                                         double (&a)[2][8]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      a[t][kk] = g[(int64_t)((t ? qa : pa) * kJacB + l15) * cp + (kk >> 2 ? qb : pb) * kJacB + 4 * (kk & 3) + lk];
}
// S = T Jb.  As a matrix-core result (lane: column l15, register r of tile t:
// row 16 t + 4 r + lk) it is the next product's operand as it stands.
__device__ __forceinline__ void jac_right(const double (&a)[2][8], const double (&b)[8], d64x4_t (&s)[2]) {
  s[0] = s[1] = d64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
#pragma unroll
    for (int t = 0; t < 2; ++t) s[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t][kk], b[kk], s[t], 0, 0, 0);
}
// Ja^T S
__device__ __forceinline__ d64x4_t jac_left(const double (&a)[8], const d64x4_t (&s)[2]) {
  d64x4_t o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) o = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], s[kk >> 2][kk & 3], o, 0, 0, 0);
  return o;
}

// One round.  The first nb / 2 workgroups each take a block pair of this
// round: its 32 x 32 part of G after the last round (three products of the
// last round's G and J), the rotations in LDS, J out.  The others apply the
// last round's rotations to G and Js meanwhile, two waves to a 32 x 32 tile,
// so a round lasts as long as its subproblems.  The launch after the last
// round only completes Js.
// Every fourth round takes all pairs of its 32 columns (31 steps), the others
// those between the two blocks (16 steps): the blocks' own pairs need a visit
// now and then only (512 Gaussian columns: 10 sweeps, as with all pairs each
// time; 12 with one such round a sweep).
__global__ void __launch_bounds__(256) jac_round_kernel(const JacRound p) {
  constexpr int P = 48;   // LDS pitch: two rows of 16 doubles fill the banks
  __shared__ double A[2][kJacP][P], J[2][kJacP][P];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, lk = lane >> 4;
  const int np = p.nb / 2, first = p.round < p.rounds ? np : 0;
  const int gate = *p.ctl;   // looked at behind the loads
  if ((int)blockIdx.x >= first) {
    const int tiles = p.cp / kJacP;
    int w = ((int)blockIdx.x - first) * 4 + wave;
    if (gate == 0) return;
    if (p.round == 0) {   // Js: the permutation
      if (w < p.cp)
        for (int c = lane; c < p.cp; c += 64) p.js[(int64_t)w * p.cp + c] = p.perm[c] == w ? 1.0 : 0.0;
      return;
    }
    if (w < 2 * np * tiles) {   // rows 16 (w % ...) of Js, columns of a pair
      const int pair = w / (2 * tiles), row0 = (w - pair * 2 * tiles) * kJacB;
      int pb, qb;
      jac_blocks(p.nb, p.round - 1, pair, pb, qb);
      const double* jb = p.jlast + pair * kJacJ;
      double a[8], b[2][8];
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        a[kk] = p.js[(int64_t)(row0 + l15) * p.cp + (kk >> 2 ? qb : pb) * kJacB + 4 * (kk & 3) + lk];
#pragma unroll
        for (int h = 0; h < 2; ++h) b[h][kk] = jb[(4 * kk + lk) * kJacP + 16 * h + l15];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        d64x4_t o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) o = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], b[h][kk], o, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) p.js[(int64_t)(row0 + 4 * r + lk) * p.cp + (h ? qb : pb) * kJacB + l15] = o[r];
      }
      return;
    }
    w -= 2 * np * tiles;
    if (p.round == p.rounds || w >= 2 * np * np) return;
    const int h = w & 1, ta = (w >> 1) / np, tb = (w >> 1) - ta * np;
    int pa, qa, pb, qb;
    jac_blocks(p.nb, p.round - 1, ta, pa, qa);
    jac_blocks(p.nb, p.round - 1, tb, pb, qb);
    double t[2][8], b[8], a[2][8];
    d64x4_t s[2];
    jac_tile(p.g, p.cp, pa, qa, pb, qb, l15, lk, t);
    jac_cols(p.jlast + tb * kJacJ, h, l15, lk, b);
    jac_cols(p.jlast + ta * kJacJ, 0, l15, lk, a[0]);
    jac_cols(p.jlast + ta * kJacJ, 1, l15, lk, a[1]);
    jac_right(t, b, s);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const d64x4_t o = jac_left(a[u], s);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        p.gnext[(int64_t)((u ? qa : pa) * kJacB + 4 * r + lk) * p.cp + (h ? qb : pb) * kJacB + l15] = o[r];
    }
    return;
  }
  int bp, bq;
  jac_blocks(p.nb, p.round, blockIdx.x, bp, bq);
  if (wave < 3) {   // pp, qq, pq
    const int x = wave == 1 ? bq : bp, y = wave == 0 ? bp : bq;
    d64x4_t o;
    if (p.round == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = p.g[(int64_t)(x * kJacB + 4 * r + lk) * p.cp + y * kJacB + l15];
    } else {
      int ta, ha, tb, hb, pa, qa, pb, qb;
      jac_where(p.nb, p.round - 1, x, ta, ha);
      jac_where(p.nb, p.round - 1, y, tb, hb);
      jac_blocks(p.nb, p.round - 1, ta, pa, qa);
      jac_blocks(p.nb, p.round - 1, tb, pb, qb);
      double t[2][8], b[8], a[8];
      d64x4_t s[2];
      jac_tile(p.g, p.cp, pa, qa, pb, qb, l15, lk, t);
      jac_cols(p.jlast + tb * kJacJ, hb, l15, lk, b);
      jac_cols(p.jlast + ta * kJacJ, ha, l15, lk, a);
      if (gate == 0) return;
      jac_right(t, b, s);
      o = jac_left(a, s);
    }
    const int r0 = wave == 1 ? kJacB : 0, c0 = wave == 0 ? 0 : kJacB;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      A[0][r0 + 4 * r + lk][c0 + l15] = o[r];
      if (wave == 2) A[0][c0 + l15][r0 + 4 * r + lk] = o[r];
    }
  } else {
    for (int e = lane; e < kJacJ; e += 64) J[0][e / kJacP][e % kJacP] = e / kJacP == e % kJacP ? 1.0 : 0.0;
  }
  if (gate == 0) return;
  __syncthreads();
  // thread (i, j): the 2 x 2 block of row pair i and column pair j, and rows i
  // and 16 + i of J; one barrier a step, from one LDS copy into the other.
  // Each lane takes column pair j's angle and the row pair's from the lane
  // that has it: pair i = 4 wave + lk is the column pair of lane lk.
  const int i = 4 * wave + lk, j = (l15 + 4 * wave) & 15;
  const bool all = (p.round & 3) == 0;
  int pi = i, qi = kJacB + i, pj = j, qj = kJacB + j;   // the step's row and column pair
  if (all) {
    constexpr int m = kJacP - 1;
    pi = i ? i : m;
    qi = i ? m - i : 0;
    pj = j ? j : m;
    qj = j ? m - j : 0;
  }
  auto step = [&](auto from, auto whole) {
    constexpr int F = decltype(from)::value;
    const auto& a = A[F];
    const auto& v = J[F];
    const double app = a[pj][pj], aqq = a[qj][qj], apq = a[pj][qj];
    double a00 = a[pi][pj], a01 = a[pi][qj], a10 = a[qi][pj], a11 = a[qi][qj];
    double v00 = v[i][pj], v01 = v[i][qj], v10 = v[kJacB + i][pj], v11 = v[kJacB + i][qj];
    auto& an = A[1 - F];
    auto& vn = J[1 - F];
    double *w00 = &an[pi][pj], *w01 = &an[pi][qj], *w10 = &an[qi][pj], *w11 = &an[qi][qj];
    double *x0 = &vn[i][pj], *x1 = &vn[i][qj];
    if constexpr (decltype(whole)::value) {
      auto next = [](int x) { return x == kJacP - 2 ? 0 : x + 1; };
      pi = i ? next(pi) : pi;
      pj = j ? next(pj) : pj;
      qi = next(qi);
      qj = next(qj);
    } else {
      qi = kJacB + ((qi + 1) & (kJacB - 1));
      qj = kJacB + ((qj + 1) & (kJacB - 1));
    }
    double sj, uj;
    jac_angle(app, aqq, apq, p.tol2, sj, uj);
    const double si = jac_bcast(sj), ui = jac_bcast(uj);
    jac_rotate(a00, a01, sj, uj);
    jac_rotate(a10, a11, sj, uj);
    jac_rotate(a00, a10, si, ui);
    jac_rotate(a01, a11, si, ui);
    *w00 = a00;
    *w01 = a01;
    *w10 = a10;
    *w11 = a11;
    jac_rotate(v00, v01, sj, uj);
    jac_rotate(v10, v11, sj, uj);
    x0[0] = v00;
    x1[0] = v01;
    x0[kJacB * P] = v10;
    x1[kJacB * P] = v11;
    __syncthreads();
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  if (all) {   // 31 steps
    step(even, std::true_type{});
    for (int k = 1; k < kJacP - 1; k += 2) {
      step(odd, std::true_type{});
      step(even, std::true_type{});
    }
  } else {
    for (int k = 0; k < kJacB; k += 2) {
      step(even, std::false_type{});
      step(odd, std::false_type{});
    }
  }
  double* out = p.jthis + blockIdx.x * kJacJ;
  for (int e = tid; e < kJacJ; e += 256) out[e] = J[all][e / kJacP][e % kJacP];
}

struct JacGemm {
  const double* x;     // columns of X as rows: cp x rows
  const double* v;     // cp x cp
  const double* js;
  double* c;           // JAC_GRAM: G; JAC_APPLY: the new X
  double* c2;          // JAC_APPLY: the new V
  const double* sigma;
  const int* perm;
  int* ctl;            // JAC_GRAM: the count, JAC_APPLY: read
  double tol;
  int rows, cp, xtiles;
};
enum JacOp { JAC_GRAM, JAC_APPLY };

// 32 x 32 of the result a workgroup, K cut over eight waves, 16 k a wave and
// turn, operands straight from memory into the matrix cores' registers, four
// turns in flight: 512 columns are 136 and 512 tiles, latency and not the
// products, and a wave's whole share is under way at once (26 and 22 us at
// 512 columns; 32 x 64 tiles staged through LDS 27 and 23).
//   JAC_GRAM:  G(i, j) = x_perm(i) . x_perm(j) scaled below one, the upper
//              triangle's tiles, both halves written; pairs that are not orthogonal counted
//   JAC_APPLY: new x_j = sum_i Js(i, j) x_i, and the same of V
template <int OP>
__global__ void __launch_bounds__(512) jac_gemm_kernel(const JacGemm p) {
  __shared__ double red[8][16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, lk = lane >> 4;
  const bool second = OP == JAC_APPLY && (int)blockIdx.x >= p.xtiles;
  const int m0 = blockIdx.y * 32, n0 = ((int)blockIdx.x - (second ? p.xtiles : 0)) * 32;
  if (OP == JAC_GRAM && n0 < m0) return;
  if (OP == JAC_APPLY && *p.ctl == 0) return;
  const int K = OP == JAC_GRAM ? p.rows : p.cp;
  const int N = OP == JAC_GRAM || second ? p.cp : p.rows;   // columns of the result
  constexpr int D = 4;
  // a[d][t]: rows (JAC_APPLY: columns) m0 + 16 t + l15; b[d][t]: n0 + 16 t + l15
  double a[D][2][4], b[D][2][4];
  // raw buffers of 2^31 bytes (the host keeps matrices below that): an offset
  // past the end reads zero, so a guard is a select
  auto rsrc = [](const double* q) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(q), (short)0, (int)0x80000000, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t qa = rsrc(OP == JAC_GRAM ? p.x : p.js), qb = rsrc(second ? p.v : p.x);
  auto get = [](__amdgpu_buffer_rsrc_t rs, bool ok, int at) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, ok ? (uint32_t)at * 8u : 0x80000000u, 0, 0));
  };
  // two neighbours, zero past K (which may be inside the next row)
  auto get2 = [K](__amdgpu_buffer_rsrc_t rs, int k, int row, double& x, double& y) {
    typedef double d2_t __attribute__((ext_vector_type(2)));
    const d2_t v = __builtin_bit_cast(
        d2_t, __builtin_amdgcn_raw_buffer_load_b128(rs, k < K ? (uint32_t)(row + k) * 8u : 0x80000000u, 0, 0));
    x = v[0];
    y = k + 1 < K ? v[1] : 0.0;
  };
  int arow[2] = {}, brow[2] = {};
  if constexpr (OP == JAC_GRAM) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      arow[t] = p.perm[m0 + 16 * t + l15] * p.rows;
      brow[t] = p.perm[n0 + 16 * t + l15] * p.rows;
    }
  }
  auto load = [&](double (&xa)[2][4], double (&xb)[2][4], int turn) {
    const int k0 = (turn * 8 + wave) * 16;
    if constexpr (OP == JAC_GRAM) {   // a lane's four k are neighbours, the same in both operands
#pragma unroll
      for (int s = 0; s < 4; s += 2) {
        const int k = k0 + 4 * lk + s;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          get2(qa, k, arow[t], xa[t][s], xa[t][s + 1]);
          get2(qb, k, brow[t], xb[t][s], xb[t][s + 1]);
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = k0 + 4 * s + lk;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int n = n0 + 16 * t + l15;
          xa[t][s] = get(qa, k < K, k * p.cp + m0 + 16 * t + l15);
          xb[t][s] = get(qb, k < K && n < N, k * N + n);
        }
      }
    }
  };
  d64x4_t acc[2][2] = {};
  // turns past the last k read zeros
  const int turns = (K + 127) / 128;
#pragma unroll
  for (int d = 0; d < D; ++d) load(a[d], b[d], d);
  for (int turn = 0; turn < turns; turn += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][i][s], b[d][j][s], acc[i][j], 0, 0, 0);
      load(a[d], b[d], turn + d + D);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][8 * i + 4 * j + r][lane] = acc[i][j][r];
  __syncthreads();
  // wave w adds registers 2 w and 2 w + 1 over the waves
  // G by a power of two that brings the largest norm below one
  double scale = 1.0;
  if constexpr (OP == JAC_GRAM) scale = ldexp(1.0, -2 * max(-500, min(500, ilogb(p.sigma[p.perm[0]]))) - 2);
  bool over = false;
  double* c = second ? p.c2 : p.c;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int e = 2 * wave + h;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) v += red[w][e][lane];
    const int m = m0 + 16 * (e >> 3) + 4 * (e & 3) + lk, n = n0 + 16 * ((e >> 2) & 1) + l15;
    if (n >= N) continue;
    if constexpr (OP == JAC_GRAM) {
      c[(int64_t)m * N + n] = v * scale;
      if (n0 > m0) c[(int64_t)n * N + m] = v * scale;
      const double x = p.sigma[p.perm[m]], y = p.sigma[p.perm[n]];
      over = over || (n > m && fabs(v) > p.tol * (x * y));
    } else {
      c[(int64_t)m * N + n] = v;
    }
  }
  if (OP == JAC_GRAM && __any(over) && lane == 0) atomicAdd(p.ctl, 1);
}

}  // namespace

int32_t jac_gram(const double* x, int rows, int cp, const double* sigma, const int* perm, double tol, double* scratch,
                 int* ctl, hipStream_t st) {
  JacGemm g{};
  g.x = x;
  g.c = scratch;
  g.sigma = sigma;
  g.perm = perm;
  g.ctl = ctl;
  g.tol = tol;
  g.rows = rows;
  g.cp = cp;
  hipLaunchKernelGGL(jac_gemm_kernel<JAC_GRAM>, dim3(cp / 32, cp / 32), dim3(512), 0, st, g);
  return hip_check(hipGetLastError(), "jacobi gram");
}

int32_t jac_sweep(const double* x, const double* v, double* x2, double* v2, int rows, int cp, const int* perm,
                  double tol, double* scratch, const int* ctl, hipStream_t st) {
  const int64_t nn = (int64_t)cp * cp;
  const int np = cp / kJacP;
  double* g[2] = {scratch, scratch + nn};
  double* j[2] = {scratch + 3 * nn, scratch + 3 * nn + (int64_t)np * kJacJ};
  JacRound r{};
  r.js = scratch + 2 * nn;
  r.perm = perm;
  r.ctl = ctl;
  r.cp = cp;
  r.nb = 2 * np;
  r.rounds = r.nb - 1;
  r.tol2 = tol * tol;
  for (r.round = 0; r.round <= r.rounds; ++r.round) {
    // rounds 0 and 1 read the Gram matrix as formed
    const int from = r.round ? (r.round - 1) & 1 : 0;
    r.g = g[from];
    r.gnext = g[from ^ 1];
    r.jlast = j[(r.round + 1) & 1];
    r.jthis = j[r.round & 1];
    const int rot = r.round < r.rounds ? np : 0;
    const int waves = r.round == 0 ? cp : 2 * np * np + (r.round < r.rounds ? 2 * np * np : 0);
    hipLaunchKernelGGL(jac_round_kernel, dim3(rot + (waves + 3) / 4), dim3(256), 0, st, r);
  }
  JacGemm a{};
  a.x = x;
  a.v = v;
  a.js = r.js;
  a.c = x2;
  a.c2 = v2;
  a.ctl = const_cast<int*>(ctl);
  a.rows = rows;
  a.cp = cp;
  a.xtiles = (rows + 31) / 32;
  hipLaunchKernelGGL(jac_gemm_kernel<JAC_APPLY>, dim3(a.xtiles + cp / 32, cp / 32), dim3(512), 0, st, a);
  return hip_check(hipGetLastError(), "jacobi sweep");
}

}  // namespace tn
