// MPS classifier of section IV.A on the GPU: forward scores, softmax
// cross-entropy, and the gradient with respect to every site tensor.
//
// Scores f[b, l] = <W^l, Phi(x_b)> with Phi(p) = (cos(pi p/2), sin(pi p/2))
// per pixel and one MPS whose centre site carries the label leg.  The left
// chain absorbs sites 0..c-1 into v (v_{k+1} = (v_k (x) Phi_k) . A_k) and
// the right chain absorbs sites N-1..c+1 into u (u_k = Phi_k . (A_k . u_{k+1})).
//
// Chain kernel: one workgroup owns 16 samples and walks a run of sites with
// the samples' vectors resident in LDS in FP64; each site is a 16-row FP64
// matrix-core product against the site tensor (FP32 in HBM, widened
// exactly), followed by an exact power-of-two rescale per sample (exponents
// kept as integers).  Up to four independent runs share one launch.  The
// forward stores a vector every `ckpt_every` sites; the backward recomputes
// each segment from its checkpoint while carrying the adjoint through it
// with the mirrored step, then forms the segment's weight gradients (sums over
// the batch) of both sides in one launch.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "gemm_direct_kernel.h"
#include "internal.h"

namespace tn {

typedef float f32x4c_t __attribute__((ext_vector_type(4)));

constexpr int kRB = 16;        // samples per workgroup (rows of a 16x16 block)
constexpr int kMaxSeg = 64;    // sites per chain-kernel launch

struct ChainArgs {
  const float* w[kMaxSeg];  // site tensors of the run, in step order
  int first_site;         // site of step 0; step j is at first_site + dir * j
  int dir;
  int n_steps;
  int step_type;          // 0: v' = (v (x) Phi) . A   1: u' = Phi . (A . u)
  int n_sites;            // chain length (site 0 and n_sites-1 have a bond of 1)
  int chi;
  const float* pixels;    // [B, n_sites]
  int B;
  const float* v_in;      // vector block or NULL (unit vector, exponent 0)
  float* v_out;           // vector block (final vectors), may be NULL
  float* store;           // step inputs, may be NULL: step st's vectors at store + st * B * CHI,
  int64_t store_exp;      // its exponents at store + store_exp + st * B
  int lo;                 // v_in and v_out carry their low parts (see vblock_floats)
};

// A "vector block" holds B vectors of length CHI (zero beyond their bond
// dimension), then B exponents stored as floats, then the low parts of the
// B vectors: value = (hi + lo) * 2^e with hi = fl32(v), lo = fl32(v - hi).
// The running vectors handed from one chain launch to the next (and the
// checkpoints) keep the low parts, so the FP64 chain loses about 2^-48, not
// 2^-24, at every hand-off: random transfer matrices amplify a rounding of
// the running vector many times over by the end of the chain.  Blocks that
// only feed FP32 GEMM operands (adjoints, recomputed segment vectors) do
// not use the low parts.
__host__ __device__ inline int64_t vblock_floats(int B, int chi) { return 2 * (int64_t)B * chi + B; }
__host__ __device__ inline int64_t vblock_lo(int B, int chi) { return (int64_t)B * chi + B; }

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// One run of sites for one chain.  The running vectors and the products are
// FP64 (FP64 matrix cores, v_mfma_f64_16x16x4): a 784-site chain of FP32
// steps would round the vector at every site, and those errors compound.
// Site tensors and pixels are read as FP32 and widened exactly.
// ---------------------------------------------------------------------------
// Chain kernel.  A workgroup owns 16 samples and has one wave per 16-wide
// block of output columns (CHI / 16 waves).  Both step types have the form
//   out[r, n] = 2^-e(r) sum_s phi[r, s] sum_k x[r, k] W_s[k, n]
// with x the vector as the last site left it (not normalised), so a site
// starts its FP64 16x16x4 MFMAs right after the barrier: two products a
// value read from LDS, the features and the normaliser 2^-e (e the binary
// exponent of the row's largest entry, from an LDS maximum over the high
// words) applied to the 16 x 16 block at the end, when they have long been
// read.  The tensor of the next site is loaded into registers between the
// current site's MFMAs (two register sets, sites unrolled by two); CHI = 256
// loads its tensor in chunks within the site.
//
// Bound by the FP64 matrix cores of the compute units that have work (CHI =
// 128: 3.4 us a site).  Measured, 28 sites: CHI = 128, 1024 samples, four
// runs 241 -> 167 us; CHI = 64, 4096 samples, two runs 128 -> 95 us.
template <int CHI>
struct ChainSmem {
  static constexpr int NW = CHI / 16;
  double vec[2][kRB][CHI + 2];
  double phi[kMaxSeg][kRB][2];
  uint32_t pmax[3][kRB];      // high words of the rows' largest |entry|, sites in turn
};

__device__ __forceinline__ f32x4c_t chain_load4(const float* p) {
  typedef float f32x4cu_t __attribute__((ext_vector_type(4), aligned(4)));
  return *reinterpret_cast<const f32x4cu_t*>(p);
}

// Lane group g takes k = 16 j + 4 g + q (q < 4) of every sixteen: its x are 16-byte
// LDS reads, and a row of W read along k is covered in 64-byte runs by the
// four groups.  w[s][4 j + q]: W_s[16 j + 4 g + q, column] of one site.
template <int CHI>
struct ChainRegs {
  static constexpr bool PREFETCH = CHI <= 128;
  static constexpr int N = PREFETCH ? CHI / 4 : 4;   // k a set holds
  float w[2][N];
};

// Sixteen k of a site tensor with both bonds CHI into w[.][at .. at + 3]:
// TYPE 0 W[k, s, col], TYPE 1 W[col, s, k].  The lane's offset is a vector
// register, j's a scalar one.
template <int CHI, int TYPE>
__device__ __forceinline__ void chain_load16(ChainRegs<CHI>& R, int at, __amdgpu_buffer_rsrc_t rs, const float* W, int col,
                                             int g, int j) {
  if constexpr (TYPE == 0) {
    const uint32_t lane = (uint32_t)(8 * g * CHI + col) * 4u;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int s = 0; s < 2; ++s)
        R.w[s][at + q] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rs, lane, (2 * (16 * j + q) + s) * CHI * 4, 0));
  } else {
    const uint32_t lane = (uint32_t)(2 * col * CHI + 4 * g);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const f32x4c_t y = chain_load4(W + s * CHI + 16 * j + lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) R.w[s][at + q] = y[q];
    }
  }
}

// the same from a tensor of smaller bonds (the chain's ends, bonds below the
// padded CHI): zero beyond din in k; columns past dout repeat the last one
// and are cleared by the caller
template <int CHI, int TYPE>
__device__ __forceinline__ void chain_load16_part(ChainRegs<CHI>& R, int at, const float* W, int din, int dout, int col,
                                                  int g, int j) {
  const int c = min(col, dout - 1);
  const int64_t ks = TYPE == 0 ? 2 * (int64_t)dout : 1, ss = TYPE == 0 ? dout : din;
  const float* base = W + (TYPE == 0 ? (int64_t)c : 2 * (int64_t)c * din);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int s = 0; s < 2; ++s) R.w[s][at + q] = base[min(16 * j + 4 * g + q, din - 1) * ks + s * ss];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int s = 0; s < 2; ++s) R.w[s][at + q] = 16 * j + 4 * g + q < din ? R.w[s][at + q] : 0.f;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t chain_rsrc(const float* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, (int)0xffffffff, 0x00020000);
}

// binary exponent of a row from the high word of its largest entry (0 for a
// zero, denormal or overflowing row, which is left as it is)
__device__ __forceinline__ int chain_exp(uint32_t hi) {
  return hi >= 0x00100000u && hi < 0x7e37e43cu ? (int)(hi >> 20) - 1023 : 0;
}
__device__ __forceinline__ double chain_pow2(int e) { return __longlong_as_double((long long)(1023 + e) << 52); }

// maximum over the 16 lanes of a DPP row
template <int CTRL>
__device__ __forceinline__ uint32_t chain_dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t chain_rowmax(uint32_t x) {
  x = max(x, chain_dpp<0x128>(x));   // row_ror 8, 4, 2, 1
  x = max(x, chain_dpp<0x124>(x));
  x = max(x, chain_dpp<0x122>(x));
  return max(x, chain_dpp<0x121>(x));
}

// The products of one site.  LOAD: the next site's tensor (both bonds CHI)
// goes into `into` meanwhile, sixteen k with each sixteen k of products: all
// loads first would hold the matrix cores until they are issued.
template <int CHI, int TYPE, bool LOAD>
__device__ __forceinline__ void chain_products(const ChainRegs<CHI>& R, ChainRegs<CHI>& into, const float* Wn,
                                               const double* x, int col, int g, f64x4_t& acc0, f64x4_t& acc1) {
  constexpr int NJ = CHI / 16;
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  __amdgpu_buffer_rsrc_t rs;
  if constexpr (LOAD && TYPE == 0) rs = chain_rsrc(Wn);
  f64x2_t xr[3][2];   // two sixteens ahead
#pragma unroll
  for (int j = 0; j < 2 && j < NJ; ++j)
#pragma unroll
    for (int h = 0; h < 2; ++h) xr[j][h] = *reinterpret_cast<const f64x2_t*>(x + 16 * j + 2 * h);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j + 2 < NJ) {
#pragma unroll
      for (int h = 0; h < 2; ++h) xr[(j + 2) % 3][h] = *reinterpret_cast<const f64x2_t*>(x + 16 * (j + 2) + 2 * h);
    }
    if constexpr (LOAD) chain_load16<CHI, TYPE>(into, 4 * j, rs, Wn, col, g, j);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double xv = xr[j % 3][q >> 1][q & 1];
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, (double)R.w[0][4 * j + q], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, (double)R.w[1][4 * j + q], acc1, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// CHI = 256: the site's own tensor, sixteen k ahead of the products
template <int CHI, int TYPE>
__device__ __forceinline__ void chain_products_inline(ChainRegs<CHI> (&regs)[2], const float* W, int din, int dout,
                                                      const double* x, int col, int g, f64x4_t& acc0, f64x4_t& acc1) {
  constexpr int NJ = CHI / 16;
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  const bool full = din == CHI && dout == CHI;
  const __amdgpu_buffer_rsrc_t rs = chain_rsrc(W);
  auto load = [&](ChainRegs<CHI>& R, int j) {
    if (full) chain_load16<CHI, TYPE>(R, 0, rs, W, col, g, j);
    else chain_load16_part<CHI, TYPE>(R, 0, W, din, dout, col, g, j);
  };
  load(regs[0], 0);
#pragma unroll 1
  for (int j0 = 0; j0 < NJ; j0 += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = j0 + u;
      f64x2_t xr[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) xr[h] = *reinterpret_cast<const f64x2_t*>(x + 16 * j + 2 * h);
      if (j + 1 < NJ) load(regs[u ^ 1], j + 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double xv = xr[q >> 1][q & 1];
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, (double)regs[u].w[0][q], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, (double)regs[u].w[1][q], acc1, 0, 0, 0);
      }
    }
  }
}

// ex: exponents of the lane's rows 4 r + g
template <int CHI, int TYPE, int SET>
__device__ __forceinline__ void chain_step(const ChainArgs& a, ChainSmem<CHI>& sm, ChainRegs<CHI> (&regs)[2], int st,
                                           int (&ex)[4], int b0) {
  constexpr bool PRE = ChainRegs<CHI>::PREFETCH;
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 15, g = lane >> 4;
  const int col = wave * 16 + row;          // this lane's output column (type 0: z, type 1: a)
  // bonds: the chain's ends are 1
  auto site = [&](int j) { return a.first_site + a.dir * j; };
  auto left = [&](int j) { return site(j) == 0 ? 1 : a.chi; };
  auto right = [&](int j) { return site(j) == a.n_sites - 1 ? 1 : a.chi; };
  auto din_of = [&](int j) { return TYPE == 0 ? left(j) : right(j); };
  auto dout_of = [&](int j) { return TYPE == 0 ? right(j) : left(j); };
  const int dout = dout_of(st);
  const double* x = &sm.vec[st & 1][row][4 * g];
  // the input's exponents (site st - 1 left them) and the features of the output rows
  uint32_t hi[4];
  f64x2_t ph[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    hi[r] = sm.pmax[(st + 2) % 3][4 * r + g];
    ph[r] = *reinterpret_cast<const f64x2_t*>(&sm.phi[st][4 * r + g][0]);
  }
  if (tid < kRB) sm.pmax[(st + 1) % 3][tid] = 0;   // site st + 1's, last read by site st - 1
  f64x4_t acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0;
  if constexpr (PRE) {
    const bool more = st + 1 < a.n_steps;
    if (more && din_of(st + 1) == CHI && dout_of(st + 1) == CHI) {
      chain_products<CHI, TYPE, true>(regs[SET], regs[SET ^ 1], a.w[st + 1], x, col, g, acc0, acc1);
    } else {
      if (more)
#pragma unroll
        for (int j = 0; j < CHI / 16; ++j)
          chain_load16_part<CHI, TYPE>(regs[SET ^ 1], 4 * j, a.w[st + 1], din_of(st + 1), dout_of(st + 1), col, g, j);
      chain_products<CHI, TYPE, false>(regs[SET], regs[SET ^ 1], nullptr, x, col, g, acc0, acc1);
    }
  } else {
    chain_products_inline<CHI, TYPE>(regs, a.w[st], din_of(st), dout, x, col, g, acc0, acc1);
  }
  // FP64 16x16x4 result: lane (col + 16 g) register r holds row 4 r + g
  double outv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int e = chain_exp(hi[r]);
    double v = (ph[r][0] * acc0[r] + ph[r][1] * acc1[r]) * chain_pow2(-e);
    if (col >= dout) v = 0.0;
    ex[r] += e;
    outv[r] = v;
    sm.vec[(st + 1) & 1][4 * r + g][col] = v;
    const uint32_t m = chain_rowmax((uint32_t)(__double_as_longlong(v) >> 32) & 0x7fffffffu);
    if (row == 0) atomicMax(&sm.pmax[st % 3][4 * r + g], m);
  }
  __syncthreads();
  // a stored block holds this site's output (the next site's input), normalised
  float* dst = nullptr;     // vectors of the block to write
  float* dste = nullptr;    // its exponents
  float* dstl = nullptr;    // its low parts (running-vector hand-off only)
  if (a.store && st + 1 < a.n_steps) {
    dst = a.store + (int64_t)(st + 1) * a.B * CHI;
    dste = a.store + a.store_exp + (int64_t)(st + 1) * a.B;
  } else if (a.v_out && st + 1 == a.n_steps) {
    dst = a.v_out;
    dste = a.v_out + (int64_t)a.B * CHI;
    if (a.lo) dstl = a.v_out + vblock_lo(a.B, CHI);
  }
  if (dst) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = r * 4 + g, b = b0 + rr;
      const int e = chain_exp(sm.pmax[st % 3][rr]);
      if (b < a.B) {
        const double v = outv[r] * chain_pow2(-e);
        const float hi32 = (float)v;
        dst[(int64_t)b * CHI + col] = hi32;
        if (dstl) dstl[(int64_t)b * CHI + col] = (float)(v - (double)hi32);
        if (col == 0) dste[b] = (float)(ex[r] + e);
      }
    }
  }
}

template <int CHI, int TYPE>
__device__ __forceinline__ void chain_run(const ChainArgs& a, ChainSmem<CHI>& sm) {
  constexpr int NT = CHI / 16 * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 15, g = lane >> 4, col = wave * 16 + row;
  const int b0 = blockIdx.x * kRB;
  if (b0 >= a.B) return;
  // feature map of every site of the run
  for (int e = tid; e < a.n_steps * kRB; e += NT) {
    const int st = e / kRB, r = e % kRB, b = b0 + r;
    const int k = a.first_site + a.dir * st;
    const double p = b < a.B ? (double)a.pixels[(int64_t)b * a.n_sites + k] : 0.0;
    double sv, cv;
    sincospi(0.5 * p, &sv, &cv);
    sm.phi[st][r][0] = cv;
    sm.phi[st][r][1] = sv;
  }
  for (int e = tid; e < kRB * CHI; e += NT) {
    const int r = e / CHI, i = e % CHI, b = b0 + r;
    double x = 0.0;
    if (b < a.B) {
      if (a.v_in) {
        x = (double)a.v_in[(int64_t)b * CHI + i];
        if (a.lo) x += (double)a.v_in[vblock_lo(a.B, CHI) + (int64_t)b * CHI + i];
      } else {
        x = i == 0 ? 1.0 : 0.0;
      }
    }
    sm.vec[0][r][i] = x;
  }
  // the first site's input is taken as given: no normaliser
  if (tid < 3 * kRB) (&sm.pmax[0][0])[tid] = 0;
  int ex[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int b = b0 + 4 * r + g;
    ex[r] = (a.v_in && b < a.B) ? (int)a.v_in[(int64_t)a.B * CHI + b] : 0;
    // and stored so
    if (a.store && b < a.B) {
      const float x = a.v_in ? a.v_in[(int64_t)b * CHI + col] : (col == 0 ? 1.f : 0.f);
      a.store[(int64_t)b * CHI + col] = x;
      if (col == 0) a.store[a.store_exp + b] = (float)ex[r];
    }
  }
  ChainRegs<CHI> regs[2];
  __syncthreads();
  if constexpr (ChainRegs<CHI>::PREFETCH) {
    const int k = a.first_site, dl = k == 0 ? 1 : a.chi, dr = k == a.n_sites - 1 ? 1 : a.chi;
#pragma unroll
    for (int j = 0; j < CHI / 16; ++j)
      chain_load16_part<CHI, TYPE>(regs[0], 4 * j, a.w[0], TYPE == 0 ? dl : dr, TYPE == 0 ? dr : dl, col, g, j);
  }
  for (int st = 0; st < a.n_steps; st += 2) {
    chain_step<CHI, TYPE, 0>(a, sm, regs, st, ex, b0);
    if (st + 1 < a.n_steps) chain_step<CHI, TYPE, 1>(a, sm, regs, st + 1, ex, b0);
  }
  // a run of zero sites (never launched) would leave v_out unwritten
}

// blockIdx.y selects one of up to four independent runs (left and right
// chains, recomputation and adjoint) advancing in one launch
struct ChainRuns {
  ChainArgs a[4];
};
template <int CHI>
__global__ void __launch_bounds__(CHI / 16 * 64) chain_kernel(const ChainRuns runs) {
  __shared__ __attribute__((aligned(16))) ChainSmem<CHI> sm;
  const ChainArgs& a = runs.a[blockIdx.y];
  if (a.step_type == 0) chain_run<CHI, 0>(a, sm);
  else chain_run<CHI, 1>(a, sm);
}

// X[b, a, s] = v[b, a] * Phi_s(x_{b, site})
__global__ void expand_kernel(const float* vblk, const float* pixels, int n_pix, int site, int B, int chi, int d, float* x) {
  const int64_t total = (int64_t)B * d * 2;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int s = (int)(e & 1);
    const int64_t ba = e >> 1;
    const int b = (int)(ba / d), aa = (int)(ba % d);
    float sv, cv;
    sincospif(0.5f * pixels[(int64_t)b * n_pix + site], &sv, &cv);
    x[e] = vblk[(int64_t)b * chi + aa] * (s == 0 ? cv : sv);
  }
}

// Weight gradients of one segment per chain side.  A segment buffer holds E
// vector slots of B x pc floats followed by E x B exponents (at + eoff).
// Site k_j = k0 - j:
//   dA_{k_j}[a, s, z] = sum_b (V_j[b, a] Phi_s(x_{b, k_j}) 2^(e_V(b) + e_G(b))) G_j[b, z]
// with V_j in slot n - 1 - j of v and G_j in slot j of g.
//
// A workgroup owns 32 a (both s) by 64 z of one site and cuts the samples
// over its eight waves, each reading its samples' V and G rows straight into
// the operand registers (lanes along a and z) and forming the two features'
// products with V there: the expanded operand, twice V, never reaches memory,
// and the sums go straight into the caller's gradient tensors.  The features
// and exponents of a site are computed once a workgroup, kGradSamples at a
// time.  Bound by the FP32 matrix cores (chi = 128, 1024 samples, 56 sites:
// 3.8e9 flops, 24 us).  Measured, that launch: 49 us; the expanded operand, a
// batched GEMM and the scatter of its blocks took 164 us.
constexpr int kGradSamples = 1024;   // samples whose features are in LDS at a time

struct GradSide {
  const float* v;
  const float* g;
  int n, k0;
};
struct GradArgs {
  GradSide side[2];
  int first;                  // entry of this launch's first (entries: side 0's sites, then side 1's)
  float* dst[kMaxSeg];
  int64_t st[kMaxSeg][3];     // their strides
  int64_t eoff;
  const float* pixels;
  int n_pix, B, pc, chi, tiles_a;
};

template <int P>
__global__ void __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
    segment_grad_kernel(const GradArgs ga) {
  constexpr int CH = DirectInfo<P>::CH, NQ = DirectInfo<P>::NQ;
  constexpr int U = PrecInfo<P>::bf ? 2 : 4;   // chunks in flight
  constexpr int WAVES = kDirectWaves;
  __shared__ __attribute__((aligned(16))) float red[WAVES * 2 * 1024];
  __shared__ __attribute__((aligned(16))) float phi[2][kGradSamples];
  __shared__ __attribute__((aligned(16))) int exps[kGradSamples];
  const int entry = ga.first + blockIdx.y, sd = entry >= ga.side[0].n ? 1 : 0, j = sd ? entry - ga.side[0].n : entry;
  const GradSide& S = ga.side[sd];
  const int B = ga.B, pc = ga.pc, k = S.k0 - j;
  const float* V = S.v + (int64_t)(S.n - 1 - j) * B * pc;
  const float* G = S.g + (int64_t)j * B * pc;
  const float* ve = S.v + ga.eoff + (int64_t)(S.n - 1 - j) * B;
  const float* ge = S.g + ga.eoff + (int64_t)j * B;
  const int lane = threadIdx.x & 63, r = lane & 31, h4 = (lane >> 5) * 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tz = blockIdx.x / ga.tiles_a, ta = blockIdx.x - tz * ga.tiles_a;
  const int a0 = ta * 32, z0 = tz * 64;
  // columns past the padded bond repeat the last one and are not stored
  const int va = min(a0 + r, pc - 1), g0 = min(z0 + r, pc - 1), g1 = min(z0 + 32 + r, pc - 1);
  f32x16_t acc[2][2];   // [s][z block]
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[s][q] = f32x16_t{};

  struct Frag {
    f32x4_t v[NQ], g[2][NQ];
  };
  for (int base = 0; base < B; base += kGradSamples) {
    const int nb = min(kGradSamples, B - base);
    if (base) __syncthreads();   // the last samples' features are used up
    for (int i = threadIdx.x; i < kGradSamples; i += WAVES * 64) {
      float sv = 0.f, cv = 0.f;
      int e = 0;
      if (i < nb) {
        sincospif(0.5f * ga.pixels[(int64_t)(base + i) * ga.n_pix + k], &sv, &cv);
        e = (int)ve[base + i] + (int)ge[base + i];
      }
      phi[0][i] = cv;
      phi[1][i] = sv;
      exps[i] = e;
    }
    __syncthreads();
    const int nch = (nb + CH - 1) / CH;
    int c = wave * nch / WAVES;
    const int c1 = (wave + 1) * nch / WAVES;
    // the lane's column and half in a vector register, the sample in a scalar one
    const __amdgpu_buffer_rsrc_t rv = chain_rsrc(V + (int64_t)base * pc), rg = chain_rsrc(G + (int64_t)base * pc);
    auto at = [&](__amdgpu_buffer_rsrc_t rs, uint32_t voff, int soff) {
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
    };
    auto load = [&](Frag& f, int ch) {
      if ((ch + 1) * CH <= nb) {
        const uint32_t lv = (uint32_t)(h4 * pc + va) * 4u, l0 = (uint32_t)(h4 * pc + g0) * 4u,
                       l1 = (uint32_t)(h4 * pc + g1) * 4u;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int so = (ch * CH + 8 * q + i) * pc * 4;
            f.v[q][i] = at(rv, lv, so);
            f.g[0][q][i] = at(rg, l0, so);
            f.g[1][q][i] = at(rg, l1, so);
          }
      } else {
        // samples past the end repeat the last one (cleared below)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = min(ch * CH + 8 * q + h4 + i, nb - 1) * pc;
            f.v[q][i] = at(rv, (uint32_t)(row + va) * 4u, 0);
            f.g[0][q][i] = at(rg, (uint32_t)(row + g0) * 4u, 0);
            f.g[1][q][i] = at(rg, (uint32_t)(row + g1) * 4u, 0);
          }
      }
    };
    auto products = [&](Frag& f, int ch) {
      if ((ch + 1) * CH > nb) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (ch * CH + 8 * q + h4 + i >= nb) f.v[q][i] = f.g[0][q][i] = f.g[1][q][i] = 0.f;
      }
      f32x4_t x[2][NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int at = ch * CH + 8 * q + h4;
        const f32x4_t c0 = *reinterpret_cast<const f32x4_t*>(&phi[0][at]);
        const f32x4_t c1v = *reinterpret_cast<const f32x4_t*>(&phi[1][at]);
        const int4 e = *reinterpret_cast<const int4*>(&exps[at]);
        const int ee[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[0][q][i] = ldexpf(f.v[q][i] * c0[i], ee[i]);
          x[1][q][i] = ldexpf(f.v[q][i] * c1v[i], ee[i]);
        }
      }
      if constexpr (!PrecInfo<P>::bf) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q)
              acc[s][q] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[s][0][i], f.g[q][0][i], acc[s][q], 0, 0, 0);
      } else {
        constexpr int NPL = PrecInfo<P>::planes;
        bf16x8_t px[2][NPL], pg[2][NPL];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          direct_planes<P>(x[s], px[s]);
          direct_planes<P>(f.g[s], pg[s]);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            f32x16_t t = {};
#pragma unroll
            for (int m = 0; m < PrecInfo<P>::nprod; ++m)
              t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(px[s][prod_a(P, m)], pg[q][prod_b(P, m)], t, 0, 0, 0);
            acc[s][q] += t;
          }
      }
    };
    Frag f[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c1) load(f[u], c + u);
    for (; c < c1; c += U) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c + u < c1) {
          products(f[u], c + u);
          if (c + u + U < c1) load(f[u], c + u + U);
        }
    }
  }

  // the waves' sums, one s at a time: [wave][z block][register / 4][lane][register % 4]
  const int dl = k == 0 ? 1 : ga.chi, dr = k == ga.n_pix - 1 ? 1 : ga.chi;
  float* dst = ga.dst[blockIdx.y];
  const int64_t sa = ga.st[blockIdx.y][0], ss = ga.st[blockIdx.y][1], sz = ga.st[blockIdx.y][2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    if (s) __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const f32x4_t y = {acc[s][q][4 * e], acc[s][q][4 * e + 1], acc[s][q][4 * e + 2], acc[s][q][4 * e + 3]};
        *reinterpret_cast<f32x4_t*>(red + ((wave * 2 + q) * 4 + e) * 256 + lane * 4) = y;
      }
    __syncthreads();
    // a wave finishes four registers of one z block: rows 8 e + 4 (lane / 32) + i
    const int q = wave >> 2, e = wave & 3;
    f32x4_t t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) t += *reinterpret_cast<const f32x4_t*>(red + ((w * 2 + q) * 4 + e) * 256 + lane * 4);
    const int z = z0 + 32 * q + r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int aa = a0 + 8 * e + h4 + i;
      if (aa < dl && z < dr) dst[aa * sa + s * ss + z * sz] = t[i];
    }
  }
}

// logits[b, l] = 2^(e_v + e_u) sum_z T[b, l, z] u[b, z]
__global__ void logits_kernel(const float* t, const float* ublk, const float* vblk, int B, int L, int chi, int du,
                              float* logits, int64_t ls0, int64_t ls1) {
  const int64_t total = (int64_t)B * L;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / L), l = (int)(e % L);
    double acc = 0.0;
    for (int z = 0; z < du; ++z) acc += (double)t[((int64_t)b * L + l) * du + z] * (double)ublk[(int64_t)b * chi + z];
    const int ex = (int)vblk[(int64_t)B * chi + b] + (int)ublk[(int64_t)B * chi + b];
    logits[b * ls0 + l * ls1] = (float)ldexp(acc, ex);
  }
}

// gu[b, l, z] = g[b, l] * u[b, z] * 2^scale_exp(b)   (scale_exp from up to two exponent blocks)
__global__ void gu_kernel(const float* g, int64_t gs0, int64_t gs1, const float* ublk, const float* e1blk, int B, int L,
                          int chi, int du, float* gu) {
  const int64_t total = (int64_t)B * L * du;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int z = (int)(e % du);
    const int64_t bl = e / du;
    const int b = (int)(bl / L), l = (int)(bl % L);
    float v = g[b * gs0 + l * gs1] * ublk[(int64_t)b * chi + z];
    if (e1blk) v = ldexpf(v, (int)e1blk[(int64_t)B * chi + b] + (int)ublk[(int64_t)B * chi + b]);
    gu[e] = v;
  }
}

// abar[b, a] = sum_s Phi_s(x_c) Y[b, a, s]  into a vector block with exponent taken from `expblk`
__global__ void phi_contract_kernel(const float* y, const float* pixels, int n_pix, int site, int B, int d, int chi,
                                    const float* expblk, float* out) {
  const int64_t total = (int64_t)B * chi;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / chi), aa = (int)(e % chi);
    float v = 0.f;
    if (aa < d) {
      float sv, cv;
      sincospif(0.5f * pixels[(int64_t)b * n_pix + site], &sv, &cv);
      v = cv * y[((int64_t)b * d + aa) * 2 + 0] + sv * y[((int64_t)b * d + aa) * 2 + 1];
    }
    out[e] = v;
    if (aa == 0) out[(int64_t)B * chi + b] = expblk[(int64_t)B * chi + b];
  }
}

// ubar[b, z] = sum_l g[b, l] T[b, l, z]  into a vector block with exponent from `expblk`
__global__ void gt_kernel(const float* g, int64_t gs0, int64_t gs1, const float* t, int B, int L, int du, int chi,
                          const float* expblk, float* out) {
  const int64_t total = (int64_t)B * chi;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / chi), z = (int)(e % chi);
    float v = 0.f;
    if (z < du) {
      double acc = 0.0;
      for (int l = 0; l < L; ++l) acc += (double)g[b * gs0 + l * gs1] * (double)t[((int64_t)b * L + l) * du + z];
      v = (float)acc;
    }
    out[e] = v;
    if (z == 0) out[(int64_t)B * chi + b] = expblk[(int64_t)B * chi + b];
  }
}

__global__ void softmax_xent_kernel(const float* logits, int64_t ls0, int64_t ls1, const int64_t* labels, int B, int L,
                                    double* loss_part, float* dlogits, int64_t ds0, int64_t ds1) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  double m = -1e300;
  for (int l = 0; l < L; ++l) m = fmax(m, (double)logits[b * ls0 + l * ls1]);
  double z = 0.0;
  for (int l = 0; l < L; ++l) z += exp((double)logits[b * ls0 + l * ls1] - m);
  const int64_t yl = labels[b];
  if (yl < 0 || yl >= L) {  // a label outside 0..L-1 has no loss: NaN marks it
    loss_part[b] = __longlong_as_double(0x7ff8000000000000ll);
    for (int l = 0; l < L; ++l) dlogits[b * ds0 + l * ds1] = __int_as_float(0x7fc00000);
    return;
  }
  const int y = (int)yl;
  loss_part[b] = m + log(z) - (double)logits[b * ls0 + y * ls1];
  for (int l = 0; l < L; ++l) {
    const double p = exp((double)logits[b * ls0 + l * ls1] - m) / z;
    dlogits[b * ds0 + l * ds1] = (float)((p - (l == y ? 1.0 : 0.0)) / B);
  }
}

__global__ void mean_kernel(const double* part, int n, double* out) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += part[i];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = (red[0] + red[1] + red[2] + red[3]) / n;
}

static unsigned blocks_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 16384)); }

// ---------------------------------------------------------------------------
// host side

namespace {

struct Geometry {
  int N, c, L, B, chi, E;
  int pad_chi;                 // chain-kernel CHI (16, 32, 64, 128, 256)
  std::vector<int> left_b;     // left segment boundaries 0 = s_0 < ... < s_m = c
  std::vector<int> right_b;    // right boundaries N = t_0 > ... > t_m = c + 1
  int64_t vb;                  // floats per vector block
  size_t ckpt_floats;
};

int pad_of(int chi) {
  for (int p : {16, 32, 64, 128, 256})
    if (chi <= p) return p;
  return -1;
}

int32_t geometry(int32_t N, int32_t c, int32_t L, int32_t B, int32_t chi, int32_t E, Geometry& g) {
  if (N < 3 || c < 1 || c > N - 2) return fail(TN_ERR_INVALID_ARGUMENT, "need n_sites >= 3 and 1 <= label_site <= n_sites - 2");
  if (L < 1 || B < 1 || chi < 1) return fail(TN_ERR_INVALID_ARGUMENT, "n_labels, batch and chi must be >= 1");
  if (E < 1 || E > kMaxSeg) return fail(TN_ERR_INVALID_ARGUMENT, "ckpt_every must be in 1..%d", kMaxSeg);
  g.N = N;
  g.c = c;
  g.L = L;
  g.B = B;
  g.chi = chi;
  g.E = E;
  g.pad_chi = pad_of(chi);
  if (g.pad_chi < 0) return fail(TN_ERR_UNSUPPORTED, "bond dimension above 256");
  g.left_b.clear();
  for (int s = 0; s < c; s += E) g.left_b.push_back(s);
  g.left_b.push_back(c);
  g.right_b.clear();
  for (int t = N; t > c + 1; t -= E) g.right_b.push_back(t);
  g.right_b.push_back(c + 1);
  g.vb = vblock_floats(B, g.pad_chi);
  g.ckpt_floats = (size_t)(g.left_b.size() + g.right_b.size()) * g.vb;
  return TN_OK;
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

struct WsLayout {
  size_t vtmp0, vtmp1, xbuf, tbuf, ybuf, gubuf, seg_v[2], seg_g[2], part, total;
};

// per chain side (left, right): recomputed vectors and adjoints of one segment
WsLayout ws_layout(const Geometry& g) {
  WsLayout w;
  const size_t vb = (size_t)g.vb * 4;
  const size_t E = g.E;
  size_t o = 0;
  w.vtmp0 = o; o += al(vb);
  w.vtmp1 = o; o += al(vb);
  w.xbuf = o; o += al((size_t)g.B * g.chi * 2 * 4);
  w.tbuf = o; o += al((size_t)g.B * g.L * g.chi * 4);
  w.ybuf = o; o += al((size_t)g.B * g.chi * 2 * 4);
  w.gubuf = o; o += al((size_t)g.B * g.L * g.chi * 4);
  for (int side = 0; side < 2; ++side) {
    w.seg_v[side] = o; o += al(E * vb);
    w.seg_g[side] = o; o += al(E * vb);
  }
  w.part = o; o += al((size_t)g.B * 8);
  w.total = o;
  return w;
}

int32_t check_sites(const Geometry& g, const tn_tensor* sites, const char* name) {
  if (!sites) return fail(TN_ERR_INVALID_ARGUMENT, "%s is NULL", name);
  for (int k = 0; k < g.N; ++k) {
    char nm[48];
    snprintf(nm, sizeof(nm), "%s[%d]", name, k);
    TN_TRY(check_tensor(&sites[k], nm, TN_F32));
    const tn_tensor& t = sites[k];
    const int64_t dl = k == 0 ? 1 : g.chi, dr = k == g.N - 1 ? 1 : g.chi;
    if (k == g.c) {
      if (t.rank != 4 || t.shape[0] != dl || t.shape[1] != 2 || t.shape[2] != g.L || t.shape[3] != dr)
        return fail(TN_ERR_SHAPE_MISMATCH, "%s must be [%lld, 2, %d, %lld]", nm, (long long)dl, g.L, (long long)dr);
    } else if (t.rank != 3 || t.shape[0] != dl || t.shape[1] != 2 || t.shape[2] != dr) {
      return fail(TN_ERR_SHAPE_MISMATCH, "%s must be [%lld, 2, %lld]", nm, (long long)dl, (long long)dr);
    }
    int64_t st = 1;
    for (int q = t.rank - 1; q >= 0; --q) {
      if (t.stride[q] != st) return fail(TN_ERR_UNSUPPORTED, "%s must be contiguous", nm);
      st *= t.shape[q];
    }
  }
  return TN_OK;
}

ChainArgs chain_args(const Geometry& g, const tn_tensor* sites, const float* pixels, int step_type, int first_site,
                     int dir, int n_steps, const float* v_in, float* v_out, float* store, int lo) {
  ChainArgs a;
  std::memset(&a, 0, sizeof(a));
  a.first_site = first_site;
  a.dir = dir;
  a.n_steps = n_steps;
  a.step_type = step_type;
  a.n_sites = g.N;
  a.chi = g.chi;
  a.pixels = pixels;
  a.B = g.B;
  a.v_in = v_in;
  a.v_out = v_out;
  a.store = store;
  a.lo = lo;
  a.store_exp = (int64_t)g.E * g.B * g.pad_chi;   // segment buffers: E vector slots, then E x B exponents
  for (int j = 0; j < n_steps; ++j) a.w[j] = static_cast<const float*>(sites[first_site + dir * j].data);
  return a;
}

// up to four independent runs in one launch
int32_t launch_chains(const Geometry& g, const std::vector<ChainArgs>& runs, hipStream_t st) {
  ChainRuns r;
  int n = 0;
  for (const ChainArgs& a : runs)
    if (a.n_steps > 0) {
      if (n == 4) return fail(TN_ERR_INVALID_ARGUMENT, "at most four chain runs per launch");
      r.a[n++] = a;
    }
  if (n == 0) return TN_OK;
  const dim3 grid((unsigned)((g.B + kRB - 1) / kRB), (unsigned)n);
  for (int i = n; i < 4; ++i) r.a[i] = r.a[0];
  // one wave per 16 output columns
  switch (g.pad_chi) {
    case 16: hipLaunchKernelGGL(chain_kernel<16>, grid, dim3(64), 0, st, r); break;
    case 32: hipLaunchKernelGGL(chain_kernel<32>, grid, dim3(128), 0, st, r); break;
    case 64: hipLaunchKernelGGL(chain_kernel<64>, grid, dim3(256), 0, st, r); break;
    case 128: hipLaunchKernelGGL(chain_kernel<128>, grid, dim3(512), 0, st, r); break;
    default: hipLaunchKernelGGL(chain_kernel<256>, grid, dim3(1024), 0, st, r); break;
  }
  return hip_check(hipGetLastError(), "chain kernel");
}

int32_t launch_chain(const Geometry& g, const tn_tensor* sites, const float* pixels, int step_type, int first_site,
                     int dir, int n_steps, const float* v_in, float* v_out, float* store, int lo, hipStream_t st) {
  if (n_steps <= 0) return TN_OK;
  return launch_chains(g, {chain_args(g, sites, pixels, step_type, first_site, dir, n_steps, v_in, v_out, store, lo)},
                       st);
}

// Weight gradients of a segment on each side (n = 0: none): see segment_grad_kernel
int32_t segment_grads(const Geometry& g, const GradSide& s0, const GradSide& s1, const float* px, tn_tensor* dsites,
                      int32_t prec, hipStream_t st) {
  const int n = s0.n + s1.n;
  if (n <= 0) return TN_OK;
  GradArgs ga;
  std::memset(&ga, 0, sizeof(ga));
  ga.side[0] = s0;
  ga.side[1] = s1;
  ga.eoff = (int64_t)g.E * g.B * g.pad_chi;
  ga.pixels = px;
  ga.n_pix = g.N;
  ga.B = g.B;
  ga.pc = g.pad_chi;
  ga.chi = g.chi;
  ga.tiles_a = (g.chi + 31) / 32;
  auto f = prec == TN_PREC_SPLIT_BF16 ? segment_grad_kernel<P_X6> : segment_grad_kernel<P_FP32>;
  for (ga.first = 0; ga.first < n; ga.first += kMaxSeg) {
    const int cnt = std::min(kMaxSeg, n - ga.first);
    for (int i = 0; i < cnt; ++i) {
      const int e = ga.first + i;
      const tn_tensor& t = dsites[e < s0.n ? s0.k0 - e : s1.k0 - (e - s0.n)];
      ga.dst[i] = static_cast<float*>(t.data);
      for (int q = 0; q < 3; ++q) ga.st[i][q] = t.stride[q];
    }
    hipLaunchKernelGGL(f, dim3((unsigned)(ga.tiles_a * ((g.chi + 63) / 64)), (unsigned)cnt), dim3(kDirectWaves * 64), 0,
                       st, ga);
  }
  return hip_check(hipGetLastError(), "segment gradients");
}

// T[b, l, z] = sum_{a s} Xc[b, a, s] A_c[a, s, l, z]
int32_t label_t(const Geometry& g, const tn_tensor& ac, const float* x, float* t, int32_t prec, hipStream_t st) {
  tn_tensor xv = make_view(const_cast<float*>(x), TN_F32, {g.B, g.chi, 2});
  tn_tensor tv = make_view(t, TN_F32, {g.B, g.L, g.chi});
  const int32_t pa[2] = {1, 2}, pb[2] = {0, 1};
  return contract_between_impl(&xv, &ac, 2, pa, pb, &tv, nullptr, 0, prec, st);
}

// cumulative left/right forward: fills checkpoints, returns v_c and u_{c+1} blocks
int32_t forward_core(const Geometry& g, const tn_tensor* sites, const float* pixels, float* ckpt, hipStream_t st) {
  const size_t nl = g.left_b.size() - 1, nr = g.right_b.size() - 1, off = g.left_b.size();
  for (size_t j = 0; j < std::max(nl, nr); ++j) {
    std::vector<ChainArgs> runs;
    if (j < nl)  // slot 0 of each chain (the unit vector) is implicit
      runs.push_back(chain_args(g, sites, pixels, 0, g.left_b[j], 1, g.left_b[j + 1] - g.left_b[j],
                                j == 0 ? nullptr : ckpt + j * g.vb, ckpt + (j + 1) * g.vb, nullptr, 1));
    if (j < nr)
      runs.push_back(chain_args(g, sites, pixels, 1, g.right_b[j] - 1, -1, g.right_b[j] - g.right_b[j + 1],
                                j == 0 ? nullptr : ckpt + (off + j) * g.vb, ckpt + (off + j + 1) * g.vb, nullptr, 1));
    TN_TRY(launch_chains(g, runs, st));
  }
  return TN_OK;
}

}  // namespace

}  // namespace tn

using namespace tn;

extern "C" {

int32_t tn_mps_classifier_ckpt_shape(int32_t n_sites, int32_t label_site, int32_t batch, int32_t chi,
                                     int32_t ckpt_every, int64_t* n_floats) {
  if (!n_floats) return fail(TN_ERR_INVALID_ARGUMENT, "n_floats is NULL");
  Geometry g;
  TN_TRY(geometry(n_sites, label_site, 1, batch, chi, ckpt_every, g));
  *n_floats = (int64_t)g.ckpt_floats;
  return TN_OK;
}

int32_t tn_mps_classifier_workspace(int32_t n_sites, int32_t label_site, int32_t n_labels, int32_t batch, int32_t chi,
                                    int32_t ckpt_every, size_t* bytes) {
  if (!bytes) return fail(TN_ERR_INVALID_ARGUMENT, "bytes is NULL");
  Geometry g;
  TN_TRY(geometry(n_sites, label_site, n_labels, batch, chi, ckpt_every, g));
  *bytes = ws_layout(g).total;
  return TN_OK;
}

int32_t tn_mps_classifier_forward(int32_t n_sites, int32_t label_site, int32_t n_labels, const tn_tensor* sites,
                                  const tn_tensor* pixels, tn_tensor* logits, float* ckpt, int32_t ckpt_every,
                                  void* workspace, size_t ws_bytes, int32_t prec, void* stream) {
  TN_TRY(check_tensor(pixels, "pixels", TN_F32));
  TN_TRY(check_tensor(logits, "logits", TN_F32));
  if (pixels->rank != 2 || pixels->shape[1] != n_sites || pixels->stride[1] != 1 || pixels->stride[0] != n_sites)
    return fail(TN_ERR_SHAPE_MISMATCH, "pixels must be a contiguous [B, n_sites] tensor");
  const int B = (int)pixels->shape[0];
  if (n_sites < 3 || !sites) return fail(TN_ERR_INVALID_ARGUMENT, "need n_sites >= 3 and sites");
  const int chi = (int)sites[1].shape[0];
  Geometry g;
  TN_TRY(geometry(n_sites, label_site, n_labels, B, chi, ckpt_every > 0 ? ckpt_every : 28, g));
  TN_TRY(check_sites(g, sites, "sites"));
  if (logits->rank != 2 || logits->shape[0] != B || logits->shape[1] != n_labels)
    return fail(TN_ERR_SHAPE_MISMATCH, "logits must be [B, n_labels]");
  if (prec != TN_PREC_FP32 && prec != TN_PREC_SPLIT_BF16) return fail(TN_ERR_UNSUPPORTED, "classifier precision %d", prec);
  WsLayout w = ws_layout(g);
  if (!workspace || ws_bytes < w.total) return fail(TN_ERR_WORKSPACE_TOO_SMALL, "workspace needs %zu bytes", w.total);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  float* ck = ckpt;
  // without a checkpoint buffer the two slots per chain live in the workspace
  float* local[2] = {reinterpret_cast<float*>(ws + w.vtmp0), reinterpret_cast<float*>(ws + w.vtmp1)};
  const float* px = static_cast<const float*>(pixels->data);
  const float* vc;
  const float* uc;
  if (ck) {
    TN_TRY(forward_core(g, sites, px, ck, st));
    vc = ck + (g.left_b.size() - 1) * g.vb;
    uc = ck + (g.left_b.size() + g.right_b.size() - 1) * g.vb;
  } else {
    // whole chains in runs of at most kMaxSeg sites, ping-ponging between two blocks
    const float* prev = nullptr;
    int k = 0, slot = 0;
    while (k < g.c) {
      const int n = std::min(kMaxSeg, g.c - k);
      TN_TRY(launch_chain(g, sites, px, 0, k, 1, n, prev, local[slot], nullptr, 1, st));
      prev = local[slot];
      slot ^= 1;
      k += n;
    }
    vc = prev;
    float* uloc[2] = {reinterpret_cast<float*>(ws + w.seg_v[0]), reinterpret_cast<float*>(ws + w.seg_g[0])};
    prev = nullptr;
    int t = g.N;
    slot = 0;
    while (t > g.c + 1) {
      const int n = std::min(kMaxSeg, t - (g.c + 1));
      TN_TRY(launch_chain(g, sites, px, 1, t - 1, -1, n, prev, uloc[slot], nullptr, 1, st));
      prev = uloc[slot];
      slot ^= 1;
      t -= n;
    }
    uc = prev;
  }
  // label site
  float* xbuf = reinterpret_cast<float*>(ws + w.xbuf);
  float* tbuf = reinterpret_cast<float*>(ws + w.tbuf);
  hipLaunchKernelGGL(expand_kernel, dim3(blocks_of((int64_t)B * chi * 2)), dim3(256), 0, st, vc, px, n_sites, label_site,
                     B, g.pad_chi, chi, xbuf);
  TN_TRY(hip_check(hipGetLastError(), "expand"));
  TN_TRY(label_t(g, sites[label_site], xbuf, tbuf, prec, st));
  hipLaunchKernelGGL(logits_kernel, dim3(blocks_of((int64_t)B * n_labels)), dim3(256), 0, st, tbuf, uc, vc, B, n_labels,
                     g.pad_chi, chi, static_cast<float*>(logits->data), logits->stride[0], logits->stride[1]);
  return hip_check(hipGetLastError(), "logits");
}

int32_t tn_mps_classifier_backward(int32_t n_sites, int32_t label_site, int32_t n_labels, const tn_tensor* sites,
                                   const tn_tensor* pixels, const float* ckpt, int32_t ckpt_every,
                                   const tn_tensor* dlogits, tn_tensor* dsites, void* workspace, size_t ws_bytes,
                                   int32_t prec, void* stream) {
  TN_TRY(check_tensor(pixels, "pixels", TN_F32));
  TN_TRY(check_tensor(dlogits, "dlogits", TN_F32));
  if (!ckpt) return fail(TN_ERR_INVALID_ARGUMENT, "the backward needs the forward's checkpoints");
  if (pixels->rank != 2 || pixels->shape[1] != n_sites || pixels->stride[1] != 1 || pixels->stride[0] != n_sites)
    return fail(TN_ERR_SHAPE_MISMATCH, "pixels must be a contiguous [B, n_sites] tensor");
  const int B = (int)pixels->shape[0];
  if (n_sites < 3 || !sites || !dsites) return fail(TN_ERR_INVALID_ARGUMENT, "need n_sites >= 3, sites and dsites");
  const int chi = (int)sites[1].shape[0];
  Geometry g;
  TN_TRY(geometry(n_sites, label_site, n_labels, B, chi, ckpt_every, g));
  TN_TRY(check_sites(g, sites, "sites"));
  for (int k = 0; k < n_sites; ++k) {
    char nm[32];
    snprintf(nm, sizeof(nm), "dsites[%d]", k);
    TN_TRY(check_tensor(&dsites[k], nm, TN_F32));
    if (dsites[k].rank != sites[k].rank) return fail(TN_ERR_SHAPE_MISMATCH, "%s has the wrong rank", nm);
    for (int q = 0; q < sites[k].rank; ++q)
      if (dsites[k].shape[q] != sites[k].shape[q]) return fail(TN_ERR_SHAPE_MISMATCH, "%s has the wrong shape", nm);
  }
  if (dlogits->rank != 2 || dlogits->shape[0] != B || dlogits->shape[1] != n_labels)
    return fail(TN_ERR_SHAPE_MISMATCH, "dlogits must be [B, n_labels]");
  if (prec != TN_PREC_FP32 && prec != TN_PREC_SPLIT_BF16) return fail(TN_ERR_UNSUPPORTED, "classifier precision %d", prec);
  WsLayout w = ws_layout(g);
  if (!workspace || ws_bytes < w.total) return fail(TN_ERR_WORKSPACE_TOO_SMALL, "workspace needs %zu bytes", w.total);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  const float* px = static_cast<const float*>(pixels->data);
  const float* gl = static_cast<const float*>(dlogits->data);
  const int64_t gs0 = dlogits->stride[0], gs1 = dlogits->stride[1];
  const int64_t vb = g.vb;
  const int pc = g.pad_chi;
  const float* vc = ckpt + (g.left_b.size() - 1) * vb;
  const float* uc = ckpt + (g.left_b.size() + g.right_b.size() - 1) * vb;
  float* xbuf = reinterpret_cast<float*>(ws + w.xbuf);
  float* tbuf = reinterpret_cast<float*>(ws + w.tbuf);
  float* ybuf = reinterpret_cast<float*>(ws + w.ybuf);
  float* gubuf = reinterpret_cast<float*>(ws + w.gubuf);
  float* abar = reinterpret_cast<float*>(ws + w.vtmp0);   // adjoint of the left vector
  float* ubar = reinterpret_cast<float*>(ws + w.vtmp1);   // adjoint of the right vector
  float* segv[2] = {reinterpret_cast<float*>(ws + w.seg_v[0]), reinterpret_cast<float*>(ws + w.seg_v[1])};
  float* segg[2] = {reinterpret_cast<float*>(ws + w.seg_g[0]), reinterpret_cast<float*>(ws + w.seg_g[1])};
  const tn_tensor& ac = sites[label_site];

  // ---- label site
  hipLaunchKernelGGL(expand_kernel, dim3(blocks_of((int64_t)B * chi * 2)), dim3(256), 0, st, vc, px, n_sites, label_site,
                     B, pc, chi, xbuf);
  TN_TRY(label_t(g, ac, xbuf, tbuf, prec, st));
  // dA_c[a, s, l, z] = sum_b Xc[b, a, s] (g[b, l] u[b, z] 2^(e_v + e_u))
  hipLaunchKernelGGL(gu_kernel, dim3(blocks_of((int64_t)B * n_labels * chi)), dim3(256), 0, st, gl, gs0, gs1, uc, vc, B,
                     n_labels, pc, chi, gubuf);
  {
    tn_tensor xv = make_view(xbuf, TN_F32, {B, chi, 2});
    tn_tensor gv = make_view(gubuf, TN_F32, {B, n_labels, chi});
    const int32_t pa[1] = {0}, pb[1] = {0};
    TN_TRY(contract_between_impl(&xv, &gv, 1, pa, pb, &dsites[label_site], nullptr, 0, prec, st));
  }
  // abar_c[b, a] = sum_s Phi_s sum_{l z} A_c[a, s, l, z] g[b, l] u[b, z]   (exponent e_u)
  hipLaunchKernelGGL(gu_kernel, dim3(blocks_of((int64_t)B * n_labels * chi)), dim3(256), 0, st, gl, gs0, gs1, uc,
                     (const float*)nullptr, B, n_labels, pc, chi, gubuf);
  {
    tn_tensor gv = make_view(gubuf, TN_F32, {B, n_labels, chi});
    tn_tensor yv = make_view(ybuf, TN_F32, {B, chi, 2});
    const int32_t pa[2] = {1, 2}, pb[2] = {2, 3};
    TN_TRY(contract_between_impl(&gv, &ac, 2, pa, pb, &yv, nullptr, 0, prec, st));
  }
  hipLaunchKernelGGL(phi_contract_kernel, dim3(blocks_of((int64_t)B * pc)), dim3(256), 0, st, ybuf, px, n_sites,
                     label_site, B, chi, pc, uc, abar);
  // ubar_{c+1}[b, z] = sum_l g[b, l] T[b, l, z]   (exponent e_v)
  hipLaunchKernelGGL(gt_kernel, dim3(blocks_of((int64_t)B * pc)), dim3(256), 0, st, gl, gs0, gs1, tbuf, B, n_labels,
                     chi, pc, vc, ubar);
  TN_TRY(hip_check(hipGetLastError(), "label site"));

  // ---- chains, segment by segment from the label site outwards; round r
  // takes left segment nl-1-r and right segment nr-1-r.  Per side: one
  // launch recomputes the segment's vectors from its checkpoint and carries
  // the adjoint through it (the two are independent), then the segment's
  // weight gradients.
  const int nl = (int)g.left_b.size() - 1, nr = (int)g.right_b.size() - 1;
  const size_t off = g.left_b.size();
  for (int r = 0; r < std::max(nl, nr); ++r) {
    std::vector<ChainArgs> runs;
    int jl = nl - 1 - r, jr = nr - 1 - r;
    if (jl >= 0) {
      const int s0 = g.left_b[jl], s1 = g.left_b[jl + 1], n = s1 - s0;
      const float* ck = jl == 0 ? nullptr : ckpt + jl * vb;
      // v_{s0} .. v_{s1-1}: step i stores the input of site s0 + i
      runs.push_back(chain_args(g, sites, px, 0, s0, 1, n, ck, nullptr, segv[0], 1));
      // abar_{s1} -> abar_{s0}: step i at site s1-1-i stores abar_{s1-i}
      runs.push_back(chain_args(g, sites, px, 1, s1 - 1, -1, n, abar, abar, segg[0], 0));
    }
    if (jr >= 0) {
      const int t0 = g.right_b[jr], t1 = g.right_b[jr + 1], n = t0 - t1;   // sites t1 .. t0-1
      const float* ck = jr == 0 ? nullptr : ckpt + (off + jr) * vb;
      // u_{t0} .. u_{t1+1}: step i at site t0-1-i stores u_{t0-i}
      runs.push_back(chain_args(g, sites, px, 1, t0 - 1, -1, n, ck, nullptr, segv[1], 1));
      // ubar_{t1} -> ubar_{t0}: step i at site t1+i stores ubar_{t1+i}
      runs.push_back(chain_args(g, sites, px, 0, t1, 1, n, ubar, ubar, segg[1], 0));
    }
    TN_TRY(launch_chains(g, runs, st));
    GradSide sl{}, sr{};
    // site k = s1-1-j: from v_k (segv slot n-1-j) and abar_{k+1} (segg slot j)
    if (jl >= 0) sl = {segv[0], segg[0], g.left_b[jl + 1] - g.left_b[jl], g.left_b[jl + 1] - 1};
    // site k = t0-1-j: from ubar_k (segg slot n-1-j) and u_{k+1} (segv slot j)
    if (jr >= 0) sr = {segg[1], segv[1], g.right_b[jr] - g.right_b[jr + 1], g.right_b[jr] - 1};
    TN_TRY(segment_grads(g, sl, sr, px, dsites, prec, st));
  }
  return TN_OK;
}

int32_t tn_softmax_xent(const tn_tensor* logits, const int64_t* labels, int32_t batch, double* loss, tn_tensor* dlogits,
                        void* workspace, size_t ws_bytes, void* stream) {
  TN_TRY(check_tensor(logits, "logits", TN_F32));
  TN_TRY(check_tensor(dlogits, "dlogits", TN_F32));
  if (!labels || !loss) return fail(TN_ERR_INVALID_ARGUMENT, "labels and loss must be given");
  if (logits->rank != 2 || logits->shape[0] != batch || dlogits->rank != 2 || dlogits->shape[0] != batch ||
      dlogits->shape[1] != logits->shape[1])
    return fail(TN_ERR_SHAPE_MISMATCH, "logits and dlogits must be [batch, n_labels]");
  if (!workspace || ws_bytes < (size_t)batch * 8) return fail(TN_ERR_WORKSPACE_TOO_SMALL, "workspace needs %d bytes", batch * 8);
  hipStream_t st = static_cast<hipStream_t>(stream);
  double* part = static_cast<double*>(workspace);
  hipLaunchKernelGGL(softmax_xent_kernel, dim3((batch + 255) / 256), dim3(256), 0, st,
                     static_cast<const float*>(logits->data), logits->stride[0], logits->stride[1], labels, batch,
                     (int)logits->shape[1], part, static_cast<float*>(dlogits->data), dlogits->stride[0],
                     dlogits->stride[1]);
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, st, part, batch, loss);
  return hip_check(hipGetLastError(), "softmax xent");
}

}  // extern "C"
