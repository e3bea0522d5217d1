// Contraction GEMM for problems with few output tiles (a site of a chain at
// a bond of a few hundred, a step of a small network), where a call lasts as
// long as one tile's own chain of loads and products.
//
// A workgroup of eight waves owns one 32 x 32 tile and cuts K over its
// waves.  Every wave reads its own k of the tile's rows and columns, so there
// is no barrier before the sums, a wave's loads are in flight together, and
// the code is a few KB (it starts cold on every compute unit).  The waves'
// partial sums meet in LDS once, each wave adding and storing its share of
// the tile.
//
// The k of a matrix-core product may be taken in any order as long as both
// operands use the same one: lane half h holds k = 8 g + 4 h + (0..3) of
// each group of eight.
//
// Bound by launch and one round of loads below about 256 tiles, by the loads
// and products of a compute unit's tiles, one after the other, above.
// Measured against the staged 32 x 32 kernel of one wave (graph replay): 100
// x 200 x 100 split-BF16 9.4 -> 3.4 us, 256 x 512 x 256 FP32 11.6 -> 4.4 us,
// 512 x 512 x 1024 split-BF16 32.8 -> 8.8 us.  64 x 64 tiles, and two, four
// or sixteen waves a tile, were no faster at any number of tiles.
#pragma once

#include "gemm_kernel.h"
#include "internal.h"

namespace tn {

// A row index (M or N) of up to three axes, innermost last: operand strides
// in elements (the host checks that offsets stay below 2^31 bytes) and
// output strides
struct DirectRows {
  int32_t one;   // a single axis (the last): no digits to form
  uint32_t d1, m1, h1, d2, m2, h2;
  int32_t sx[3];
  int64_t sc[3];
};

struct DirectDesc {
  const float* a;
  const float* b;
  float* c;
  int32_t M, N, K, tiles_m;
  int64_t a_bs, b_bs, c_bs;
  const uint32_t* a_scale_bits;
  uint32_t* c_absmax;
  DirectRows gm, gn;
  // K: up to two axes, k = q dk + r
  uint32_t dk, mk, hk;
  int32_t ska[2], skb[2];
};

__device__ __forceinline__ void direct_digits(const DirectRows& g, uint32_t idx, uint32_t& r0, uint32_t& r1, uint32_t& r2) {
  const uint32_t q = fast_div(idx, g.m2, g.h2);
  r2 = idx - q * g.d2;
  r0 = fast_div(q, g.m1, g.h1);
  r1 = q - r0 * g.d1;
}
__device__ __forceinline__ int32_t direct_in(const DirectRows& g, uint32_t idx) {
  if (g.one) return (int32_t)idx * g.sx[2];
  uint32_t r0, r1, r2;
  direct_digits(g, idx, r0, r1, r2);
  return (int32_t)r0 * g.sx[0] + (int32_t)r1 * g.sx[1] + (int32_t)r2 * g.sx[2];
}
__device__ __forceinline__ int64_t direct_out(const DirectRows& g, uint32_t idx) {
  if (g.one) return (int64_t)idx * g.sc[2];
  uint32_t r0, r1, r2;
  direct_digits(g, idx, r0, r1, r2);
  return (int64_t)r0 * g.sc[0] + (int64_t)r1 * g.sc[1] + (int64_t)r2 * g.sc[2];
}

template <int P>
struct DirectInfo {
  static constexpr int CH = PrecInfo<P>::bf ? 16 : 8;   // k per chunk (one bf16 product, four fp32 products)
  static constexpr int NQ = CH / 8;                     // groups of eight k a chunk
  static constexpr int NC = 32 / CH;                    // chunks a block of 32 k
};

template <int P>
__device__ __forceinline__ void direct_planes(const f32x4_t (&x)[DirectInfo<P>::NQ], bf16x8_t (&pl)[PrecInfo<P>::planes]) {
  constexpr int NPL = PrecInfo<P>::planes;
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  u32x4_t w[NPL];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      uint32_t t[3];
      split_pair<NPL>(x[q][2 * e], x[q][2 * e + 1], t);
#pragma unroll
      for (int p = 0; p < NPL; ++p) w[p][2 * q + e] = t[p];
    }
#pragma unroll
  for (int p = 0; p < NPL; ++p) pl[p] = __builtin_bit_cast(bf16x8_t, w[p]);
}

// how an operand is read (DirectOperand)
enum DirectMode : int { D_ANY = 0, D_ROW = 1, D_STAGED = 2 };

constexpr int kDirectWaves = 8;         // waves that share a tile's K
constexpr int kDirectStage = 32 * 32;   // floats of a wave's block of one operand, and of a wave's sums
// LDS floats: per wave a block of each operand that is read along k (the
// first one's place takes the wave's sums in the end), the |C| maxima
constexpr int direct_lds(int am, int bm) {
  return (am == D_STAGED && bm == D_STAGED ? 2 : 1) * kDirectWaves * kDirectStage + kDirectWaves;
}

// orders a wave's LDS stores before its later loads (its LDS accesses are
// served in order; the compiler must keep them so)
__device__ __forceinline__ void direct_wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One wave's reads of one operand: 32 rows, k in blocks of 32.
//   D_ANY: four 4-byte loads a group of eight k, lanes along the rows, the
//     row's offset in a vector register and k's in a scalar one.
// With unit stride along k (with two contracted axes runs of whole fours):
//   D_ROW: each lane reads its own row in 16-byte pieces, straight into the
//     operand registers: the shortest way for one tile a compute unit and a
//     short K, but an instruction touches 64 lines.
//   D_STAGED: a row of a block is one 128-byte line, so eight lanes read a
//     row, and the block passes through the wave's own LDS, its pieces
//     XOR-swizzled by row so that neither side conflicts.  With many tiles
//     the lines touched bound the loads: 1536 x 1024 x 512 FP32, both
//     operands along k, 34.9 us by rows, 21.6 staged; at 100 x 200 x 100 the
//     detour costs 0.3 of 3.5 us.
template <int P, int MODE, int MK>
struct DirectOperand {
  static constexpr int NQ = DirectInfo<P>::NQ;
  static constexpr bool KV = MODE != D_ANY, STAGED = MODE == D_STAGED;
  struct Set {
    f32x4_t x[4];   // staged: pieces of rows 8 i + lane / 8; else groups of eight k
  };
  const float* base;
  __amdgpu_buffer_rsrc_t rs;   // raw buffer (stride 0) over the whole 32-bit offset range
  float* lds;
  int32_t sk[2];
  int32_t roff[STAGED ? 4 : 1];
  uint32_t dk, mk, hk;

  // row(i): element offset of row i (0..31) of the tile, a real row
  template <class F>
  __device__ __forceinline__ void init(const float* p, float* stage, const int32_t (&sk_)[2], uint32_t dk_,
                                       uint32_t mk_, uint32_t hk_, F&& row) {
    const int lane = threadIdx.x & 63;
    base = p;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, (int)0xffffffff, 0x00020000);
    lds = stage;
    sk[0] = sk_[0];
    sk[1] = sk_[1];
    dk = dk_;
    mk = mk_;
    hk = hk_;
    if constexpr (STAGED) {
#pragma unroll
      for (int i = 0; i < 4; ++i) roff[i] = row(8 * i + (lane >> 3));
    } else {
      roff[0] = row(lane & 31);
    }
  }

  // element offset of contracted index k
  __device__ __forceinline__ int32_t koff(int k) const {
    if constexpr (MK == 1) return KV ? k : k * sk[1];
    const uint32_t q = fast_div((uint32_t)k, mk, hk), r = (uint32_t)k - q * dk;
    return (int32_t)q * sk[0] + (int32_t)r * sk[1];
  }

  // one contracted axis: byte offset of (this lane's row, first k of its half)
  // and the element j further k0 on, whose offset is a scalar
  __device__ __forceinline__ uint32_t voff() const {
    const int h4 = (threadIdx.x & 32) >> 3;
    return (uint32_t)(roff[0] + (KV ? h4 : h4 * sk[1])) * 4u;
  }
  __device__ __forceinline__ float at(uint32_t vo, int k0, int j) const {
    const int step = sk[1] * 4;
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, k0 * step + j * step, 0));
  }

  // the block of k0 .. min(k0 + 32, kend) - 1; kend - k0 is a multiple of eight
  __device__ __forceinline__ void load(Set& s, int k0, int kend) const {
    const int lane = threadIdx.x & 63;
    if constexpr (STAGED) {
      const int k = k0 + (lane & 7) * 4;
      if (k < kend) {
        const int32_t ko = koff(k);
#pragma unroll
        for (int i = 0; i < 4; ++i) s.x[i] = load4u(base + (uint32_t)(roff[i] + ko));
      }
    } else {
      const int h4 = (lane >> 5) * 4;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int kg = k0 + 8 * g;
        if (kg < kend) {
          if constexpr (KV) {
            if constexpr (MK == 1)
              s.x[g] = load4u(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base + kg) + voff()));
            else
              s.x[g] = load4u(base + (uint32_t)(roff[0] + koff(kg + h4)));
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if constexpr (MK == 1) s.x[g][j] = at(voff(), kg, j);
              else s.x[g][j] = base[(uint32_t)(roff[0] + koff(kg + h4 + j))];
            }
          }
        }
      }
    }
  }

  // the block into the wave's LDS
  __device__ __forceinline__ void put(const Set& s) const {
    if constexpr (STAGED) {
      const int lane = threadIdx.x & 63;
      direct_wave_order();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 8 * i + (lane >> 3);
        *reinterpret_cast<f32x4_t*>(lds + (row * 8 + ((lane & 7) ^ ((row >> 1) & 7))) * 4) = s.x[i];
      }
      direct_wave_order();
    }
  }

  // chunk q of the block (after put)
  __device__ __forceinline__ void chunk(const Set& s, int q, f32x4_t (&f)[NQ]) const {
    const int lane = threadIdx.x & 63, r = lane & 31;
#pragma unroll
    for (int g = 0; g < NQ; ++g) {
      if constexpr (STAGED)
        f[g] = *reinterpret_cast<const f32x4_t*>(lds + (r * 8 + ((2 * (q * NQ + g) + (lane >> 5)) ^ ((r >> 1) & 7))) * 4);
      else
        f[g] = s.x[q * NQ + g];
    }
  }

  // the partial last chunk, k0 .. K - 1, element by element; the rest reads
  // k = K - 1 and becomes zero (no branch, so the loads are in flight together)
  template <class F>
  __device__ __forceinline__ void tail(int k0, int K, f32x4_t (&f)[NQ], F&& row) const {
    const int kl = k0 + ((threadIdx.x & 32) >> 3);
    const int32_t off = STAGED ? row(threadIdx.x & 31) : roff[0];
#pragma unroll
    for (int g = 0; g < NQ; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        f[g][j] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rs, (uint32_t)(off + koff(min(kl + 8 * g + j, K - 1))) * 4u, 0, 0));
#pragma unroll
    for (int g = 0; g < NQ; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) f[g][j] = kl + 8 * g + j < K ? f[g][j] : 0.f;
  }
};

// The waves' partial sums of one tile into red (direct_lds floats), ordered
// by a barrier.  arow(i), brow(i): element offsets of row i of A's share and
// column i of B's (0..31, clamped to the problem: the products of a repeated
// row are never stored).  D: a descriptor with K, the contracted strides ska,
// skb and, for MK = 2, the inner axis dk, mk, hk.
template <int P, int AM, int BM, int MK, class D, class FA, class FB>
__device__ __forceinline__ void direct_sums(const D& d, const float* A, const float* B, FA&& arow, FB&& brow,
                                            float* red) {
  constexpr int WK = kDirectWaves;
  constexpr int CH = DirectInfo<P>::CH, NQ = DirectInfo<P>::NQ, NC = DirectInfo<P>::NC;
  // Blocks in flight.  One where the bf16 terms need the registers, or the
  // offsets of two contracted axes do (FP32, 333 x 333, K = 2 x 600 17.4 -> 13.1
  // us; 512 x 1024, K = 2 x 256 14.5 -> 11.5; 216 shapes 1.08 in the mean, none
  // slower), or where A is read in 4-byte loads, 16 a block: the shorter code
  // starts sooner than a second block helps (both operands so, 333 x 1000 x 666
  // 11.5 -> 10.0 us, 100 x 200 x 100 4.3 -> 3.9; 140 shapes 1.05 in the mean, the
  // worst 2 % slower).  A along k alone gains 2 % in the mean and loses up to 4.
  constexpr int NS = PrecInfo<P>::bf || MK == 2 || AM == D_ANY ? 1 : 2;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* stage = red + wave * kDirectStage;
  DirectOperand<P, AM, MK> oa;
  DirectOperand<P, BM, MK> ob;
  oa.init(A, stage, d.ska, d.dk, d.mk, d.hk, arow);
  ob.init(B, stage + (AM == D_STAGED && BM == D_STAGED ? WK * kDirectStage : 0), d.skb, d.dk, d.mk, d.hk, brow);

  f32x16_t acc = {};
  // One chunk's products.  The split precisions form them in a chain from
  // zero and add it to the sum in one rounding (the matrix cores' own
  // accumulation onto a large sum is biased, see gemm_kernel.h).
  auto products = [&](const f32x4_t (&fa)[NQ], const f32x4_t (&fb)[NQ]) {
    if constexpr (!PrecInfo<P>::bf) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[0][e], fb[0][e], acc, 0, 0, 0);
    } else {
      constexpr int NPL = PrecInfo<P>::planes;
      bf16x8_t pa[NPL], pb[NPL];
      direct_planes<P>(fa, pa);
      direct_planes<P>(fb, pb);
      f32x16_t t = NPL > 1 ? f32x16_t{} : acc;
#pragma unroll
      for (int q = 0; q < PrecInfo<P>::nprod; ++q)
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[prod_a(P, q)], pb[prod_b(P, q)], t, 0, 0, 0);
      if constexpr (NPL > 1) acc += t;
      else acc = t;
    }
  };

  const int nfull = d.K / CH, nch = (d.K + CH - 1) / CH;
  const int c0 = (int)((uint32_t)(wave * nch) / WK), c1 = (int)((uint32_t)((wave + 1) * nch) / WK);
  const bool tail = wave == WK - 1 && nch != nfull;   // a partial last chunk
  const int kbeg = c0 * CH, kend = (c1 - (tail ? 1 : 0)) * CH;
  typename DirectOperand<P, AM, MK>::Set sa[NS];
  typename DirectOperand<P, BM, MK>::Set sb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (kbeg + 32 * s < kend) {
      oa.load(sa[s], kbeg + 32 * s, kend);
      ob.load(sb[s], kbeg + 32 * s, kend);
    }
  if (tail) {
    f32x4_t fa[NQ], fb[NQ];
    oa.tail(nfull * CH, d.K, fa, arow);
    ob.tail(nfull * CH, d.K, fb, brow);
    products(fa, fb);
  }
  for (int k0 = kbeg; k0 < kend; k0 += 32 * NS) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int k = k0 + 32 * s, next = k + 32 * NS;
      if (s > 0 && k >= kend) continue;
      oa.put(sa[s]);
      ob.put(sb[s]);
      // an operand that went to LDS is refilled at once, one that is used
      // from its registers after the products
      if (AM == D_STAGED && next < kend) oa.load(sa[s], next, kend);
      if (BM == D_STAGED && next < kend) ob.load(sb[s], next, kend);
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (q == 0 || k + q * CH < kend) {
          f32x4_t fa[NQ], fb[NQ];
          oa.chunk(sa[s], q, fa);
          ob.chunk(sb[s], q, fb);
          products(fa, fb);
        }
      if (AM != D_STAGED && next < kend) oa.load(sa[s], next, kend);
      if (BM != D_STAGED && next < kend) ob.load(sb[s], next, kend);
    }
  }

  // the wave's sums over its first block: [wave][register / 4][lane][register % 4]
  direct_wave_order();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4_t v = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    *reinterpret_cast<f32x4_t*>(stage + q * 256 + lane * 4) = v;
  }
  __syncthreads();
}

// Registers e = 2 wave and 2 wave + 1 of the tile, summed over the waves:
// lane l holds rows 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
__device__ __forceinline__ f32x2_t direct_total(const float* red, int wave) {
  static_assert(kDirectWaves == 8, "eight waves finish a tile of 16 registers, two each");
  f32x2_t v = {0.f, 0.f};
  const float* p = red + (wave >> 1) * 256 + (threadIdx.x & 63) * 4 + (wave & 1) * 2;
#pragma unroll
  for (int w = 0; w < kDirectWaves; ++w) {
    const f32x2_t y = *reinterpret_cast<const f32x2_t*>(p + w * kDirectStage);
    v[0] += y[0];
    v[1] += y[1];
  }
  return v;
}

template <int P, int AM, int BM, int MK>
__device__ __forceinline__ void direct_tile(const DirectDesc& d, int bid, int bz, float* red, float* mx) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tn = bid / d.tiles_m, tm = bid - tn * d.tiles_m;
  const int m0 = tm * 32, n0 = tn * 32;
  direct_sums<P, AM, BM, MK>(
      d, d.a + bz * d.a_bs, d.b + bz * d.b_bs, [&](int i) { return direct_in(d.gm, (uint32_t)min(m0 + i, d.M - 1)); },
      [&](int i) { return direct_in(d.gn, (uint32_t)min(n0 + i, d.N - 1)); }, red);
  float scale = 1.0f;
  if (d.a_scale_bits) scale = pow2_inverse_scale(d.a_scale_bits[bz]);
  float* C = d.c + bz * d.c_bs;
  const int n = n0 + (lane & 31);
  const int64_t on = direct_out(d.gn, (uint32_t)min(n, d.N - 1));
  const f32x2_t total = direct_total(red, wave);
  float amax = 0.f;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int e = 2 * wave + x;
    const float v = total[x] * scale;
    const int m = m0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (m < d.M && n < d.N) {
      C[direct_out(d.gm, (uint32_t)m) + on] = v;
      amax = fmaxf(amax, fabsf(v));
    }
  }
  if (d.c_absmax) {   // one atomic per workgroup
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
    if (lane == 0) mx[wave] = amax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int w = 1; w < kDirectWaves; ++w) amax = fmaxf(amax, mx[w]);
      atomicMax(d.c_absmax + bz, __float_as_uint(amax));
    }
  }
}

// four waves a SIMD: two workgroups a compute unit, so that one's loads run
// under the other's products
template <int P, int AM, int BM, int MK>
__global__ void __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
    gemm_direct_kernel(const DirectDesc d) {
  __shared__ __attribute__((aligned(16))) float red[direct_lds(AM, BM)];
  direct_tile<P, AM, BM, MK>(d, blockIdx.x, blockIdx.z, red, red + direct_lds(AM, BM) - kDirectWaves);
}

// Tiles of many 2-D problems in one launch (the halves of an uneven batch of
// chains), each problem a range of workgroups; D_STAGED where every problem's
// operand has unit stride along k
template <int P, int AM, int BM>
__global__ void __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
    gemm_direct_grouped_kernel(const Gemm2D* probs, const int32_t* tile_start, int32_t n_probs) {
  __shared__ __attribute__((aligned(16))) float red[direct_lds(AM, BM)];
  const int prob = grouped_find(tile_start, n_probs, blockIdx.x);
  const Gemm2D& p = probs[prob];
  DirectDesc d;
  d.a = p.a;
  d.b = p.b;
  d.c = p.c;
  d.M = p.M;
  d.N = p.N;
  d.K = p.K;
  d.tiles_m = (p.M + 31) / 32;
  d.a_bs = d.b_bs = d.c_bs = 0;
  d.a_scale_bits = p.a_scale_bits;
  d.c_absmax = p.c_absmax;
  d.gm.one = d.gn.one = 1;
  d.gm.sx[2] = (int32_t)p.sam;
  d.gm.sc[2] = p.scm;
  d.gn.sx[2] = (int32_t)p.sbn;
  d.gn.sc[2] = p.scn;
  d.ska[1] = (int32_t)p.sak;
  d.skb[1] = (int32_t)p.sbk;
  const int tile = (int)blockIdx.x - tile_start[prob];
  if (tile >= d.tiles_m * ((p.N + 31) / 32)) return;
  direct_tile<P, AM, BM, 1>(d, tile, 0, red, red + direct_lds(AM, BM) - kDirectWaves);
}

// Two independent problems in one launch (the same step of a chain's two
// ends or directions): workgroups below tiles0 take the first, the rest the
// second.  Where a mode is D_ANY the operand may have any layout.
struct DirectPair {
  DirectDesc d0, d1;
  int32_t tiles0;
};

template <int P, int A0, int B0, int A1, int B1>
__global__ void __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
    gemm_direct_pair_kernel(const DirectPair p) {
  constexpr int LDS = direct_lds(A0, B0) > direct_lds(A1, B1) ? direct_lds(A0, B0) : direct_lds(A1, B1);
  __shared__ __attribute__((aligned(16))) float red[LDS];
  float* mx = red + LDS - kDirectWaves;
  const int bid = blockIdx.x;
  if (bid < p.tiles0) direct_tile<P, A0, B0, 1>(p.d0, bid, 0, red, mx);
  else direct_tile<P, A1, B1, 1>(p.d1, bid - p.tiles0, 0, red, mx);
}

// The first contraction of a site of the operator sweeps with the operator
// step in its epilogue, physical dimension 2:
//   left:  T2[a', t, v, b]  = sum_{u, s} W[u, v, t, s] sum_a  L[a', u, a] A[a, s, b]
//   right: T2'[u, a, t, b'] = sum_{s, v} W[u, v, t, s] sum_b'' A[a, s, b''] R[b', v, b'']
// The operator mixes the inner index of the rows with that of the columns,
// so a tile holds all of both for a few outer ones: left 32 / wl a' times u
// by s times 16 b, right 16 a times s by 32 / wr b' times v.  The tile of
// the product (FP32, as it would be stored) goes through LDS and the step
// sums in FP64 as the separate step does, a thread all the results of one
// pair of outer indices; the intermediate never reaches memory.
struct DirectWstep {
  const float* x;   // rows (outer, inner), unit stride along k
  const float* y;   // columns
  const float* w;
  float* out;
  int32_t K, no_x, no_y, ni_x, ni_y;   // k, outer and inner extents of rows and columns
  int32_t per_x, per_y, tiles_x;       // outer indices a tile; tiles along x
  int32_t xo, xi, yo, yi;              // element strides
  int32_t ska[2], skb[2];
  uint32_t dk, mk, hk;                 // unused (one contracted axis)
  int32_t w0, w1, w2, w3, wl, wr;
};
constexpr int kDirectMaxW = 8;   // operator bond

// W: the operator bond on both sides, or 0 for any (at most kDirectMaxW)
template <int P, bool LEFT, int KM, int W>
__device__ __forceinline__ void direct_wstep_tile(const DirectWstep& d, int bid, float* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ty = bid / d.tiles_x, tx = bid - ty * d.tiles_x;
  const int x0 = tx * d.per_x, y0 = ty * d.per_y;
  const int wl = W ? W : d.wl, wr = W ? W : d.wr;
  // the operator's entries, sw[((v * 2 + t) * wl + u) * 2 + s] (left) or
  // [((u * 2 + t) * 2 + s) * wr + v] (right): the sum's index runs fastest.
  // One a thread (at most 256), read before the products.
  const int nw = wl * wr * 4;
  float wv = 0.f;
  if ((int)threadIdx.x < nw) {
    const uint32_t i = threadIdx.x;
    uint32_t u, v, t, s;
    if constexpr (LEFT) {
      s = i & 1;
      const uint32_t q = (i >> 1) / (uint32_t)wl;
      u = (i >> 1) - q * wl;
      t = q & 1;
      v = q >> 1;
    } else {
      const uint32_t q = i / (uint32_t)wr;
      v = i - q * wr;
      s = q & 1;
      t = (q >> 1) & 1;
      u = q >> 2;
    }
    wv = d.w[(int)u * d.w0 + (int)v * d.w1 + (int)t * d.w2 + (int)s * d.w3];
  }
  // left: columns (s, b) as s 16 + b; right: columns (b', v), rows (a, s)
  direct_sums<P, KM, LEFT ? (int)D_ANY : KM, 1>(
      d, d.x, d.y,
      [&](int i) {
        const int o = LEFT ? (int)((uint32_t)i / (uint32_t)wl) : i >> 1, in = LEFT ? i - o * wl : i & 1;
        return min(x0 + o, d.no_x - 1) * d.xo + in * d.xi;
      },
      [&](int i) {
        const int o = LEFT ? i & 15 : (int)((uint32_t)i / (uint32_t)wr), in = LEFT ? i >> 4 : i - o * wr;
        return min(y0 + o, d.no_y - 1) * d.yo + in * d.yi;
      },
      red);
  // the tile's sums, then (over the partial sums, which are read by then) its rows
  const f32x2_t sum = direct_total(red, wave);
  __syncthreads();
  float* t1 = red;                                            // [32][33]
  double* sw = reinterpret_cast<double*>(red + 32 * 34);
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int e = 2 * wave + x;
    t1[(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 33 + (lane & 31)] = sum[x];
  }
  if ((int)threadIdx.x < nw) sw[threadIdx.x] = (double)wv;
  __syncthreads();
  const int da = d.no_x, db = d.no_y;
  if constexpr (LEFT) {
    // a thread: one (a', t, b), all v
    for (int i = threadIdx.x; i < d.per_x * 32; i += kDirectWaves * 64) {
      const int b = i & 15, t = (i >> 4) & 1, al = i >> 5;
      if (x0 + al >= da || y0 + b >= db) continue;
      const float* x = t1 + al * wl * 33 + b;
      float* out = d.out + ((int64_t)(x0 + al) * 2 + t) * wr * db + y0 + b;
      if constexpr (W > 0) {
        double xs[W][2];
#pragma unroll
        for (int u = 0; u < W; ++u) {
          xs[u][0] = (double)x[u * 33];
          xs[u][1] = (double)x[u * 33 + 16];
        }
#pragma unroll
        for (int v = 0; v < W; ++v) {
          const double* c = sw + (v * 2 + t) * W * 2;
          double acc = 0.0;
#pragma unroll
          for (int u = 0; u < W; ++u) {
            acc += c[2 * u] * xs[u][0];
            acc += c[2 * u + 1] * xs[u][1];
          }
          out[(int64_t)v * db] = (float)acc;
        }
      } else {
        for (int v = 0; v < wr; ++v) {
          const double* c = sw + (v * 2 + t) * wl * 2;
          double acc = 0.0;
          for (int u = 0; u < wl; ++u) {
            acc += c[2 * u] * (double)x[u * 33];
            acc += c[2 * u + 1] * (double)x[u * 33 + 16];
          }
          out[(int64_t)v * db] = (float)acc;
        }
      }
    }
  } else {
    // a thread: one (a, t, b'), all u
    const int nb = W ? 32 / (W ? W : 1) : d.per_y;
    for (int i = threadIdx.x; i < 32 * nb; i += kDirectWaves * 64) {
      const int q = (int)((uint32_t)i / (uint32_t)nb), b = i - q * nb, t = q & 1, al = q >> 1;
      if (x0 + al >= da || y0 + b >= db) continue;
      const float* x = t1 + al * 66 + b * wr;
      float* out = d.out + ((int64_t)(x0 + al) * 2 + t) * db + y0 + b;
      const int64_t us = (int64_t)da * 2 * db;
      if constexpr (W > 0) {
        double xs[2][W];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int v = 0; v < W; ++v) xs[s][v] = (double)x[s * 33 + v];
#pragma unroll
        for (int u = 0; u < W; ++u) {
          const double* c = sw + (u * 2 + t) * 2 * W;
          double acc = 0.0;
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int v = 0; v < W; ++v) acc += c[s * W + v] * xs[s][v];
          out[u * us] = (float)acc;
        }
      } else {
        for (int u = 0; u < wl; ++u) {
          const double* c = sw + (u * 2 + t) * 2 * wr;
          double acc = 0.0;
          for (int s = 0; s < 2; ++s)
            for (int v = 0; v < wr; ++v) acc += c[s * wr + v] * (double)x[s * 33 + v];
          out[u * us] = (float)acc;
        }
      }
    }
  }
}

struct DirectWstepPair {
  DirectWstep l, r;
  int32_t tiles_l;   // workgroups below it take the left problem
};

// KM: D_ROW or D_STAGED for the operands along k; W: every operator bond, or 0
template <int P, int KM, int W>
__global__ void __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
    direct_wstep_kernel(const DirectWstepPair p) {
  __shared__ __attribute__((aligned(16))) float red[direct_lds(KM, KM)];
  const int bid = blockIdx.x;
  if (bid < p.tiles_l) direct_wstep_tile<P, true, KM, W>(p.l, bid, red);
  else direct_wstep_tile<P, false, KM, W>(p.r, bid - p.tiles_l, red);
}

}  // namespace tn
