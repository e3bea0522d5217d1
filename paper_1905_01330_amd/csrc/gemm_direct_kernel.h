// Contraction GEMM for problems with few output tiles (a site of a chain at
// a bond of a few hundred, a step of a small network), where a call lasts as
// long as one tile's own chain of loads and products.
//
// A workgroup of eight waves owns one 32 x 32 tile and cuts K over its
// waves.  Every wave reads its own k of the tile's rows and columns straight
// from memory into the matrix-core operand registers: nothing is staged
// through LDS, so there is no barrier before the sums, all of a wave's loads
// are in flight at once, and the code is a few KB (it starts cold on every
// compute unit).  The waves' partial sums meet in LDS once, each wave adding
// and storing its share of the tile.
//
// The k of a matrix-core product may be taken in any order as long as both
// operands use the same one: lane half h holds k = 8 g + 4 h + (0..3) of
// each group of eight, so a k-contiguous operand is read in 16-byte loads
// and any other in four 4-byte loads whose lanes run along the rows.
//
// Bound by launch and one round of loads below about 256 tiles, by the
// matrix cores (FP32) above.  Measured against the staged 32 x 32 kernel of
// one wave (graph replay): 100 x 200 x 100 split-BF16 9.4 -> 3.4 us, 256 x
// 512 x 256 FP32 11.6 -> 4.3 us, 512 x 512 x 1024 split-BF16 32.8 -> 8.8 us.
// 64 x 64 tiles (four or eight waves) were slower up to 1500 tiles of 32 x
// 32, and sixteen waves a tile slower everywhere.
#pragma once

#include "gemm_kernel.h"

namespace tn {

// A row index (M or N) of up to three axes, innermost last: operand strides
// in elements (the host checks that offsets stay below 2^31 bytes) and
// output strides
struct DirectRows {
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
  uint32_t r0, r1, r2;
  direct_digits(g, idx, r0, r1, r2);
  return (int32_t)r0 * g.sx[0] + (int32_t)r1 * g.sx[1] + (int32_t)r2 * g.sx[2];
}
__device__ __forceinline__ int64_t direct_out(const DirectRows& g, uint32_t idx) {
  uint32_t r0, r1, r2;
  direct_digits(g, idx, r0, r1, r2);
  return (int64_t)r0 * g.sc[0] + (int64_t)r1 * g.sc[1] + (int64_t)r2 * g.sc[2];
}

template <int P>
struct DirectInfo {
  static constexpr int CH = PrecInfo<P>::bf ? 16 : 8;   // k per chunk (one bf16 product, four fp32 products)
  static constexpr int NQ = CH / 8;                     // groups of eight k
};

// One operand's four k (kb + h4 + 0..3; kb is the same in the whole wave, h4
// the lane's half) of one row.  KV: unit stride along k.  MK: contracted axes
// (1 or 2; the inner one's extent is a multiple of four where KV).  LIMIT:
// k >= K reads 0.  row: the row's element offset; lane: with one contracted
// axis, the byte offset of (row, h4), so that a load is a uniform base plus a
// 32-bit lane offset.
template <bool KV, int MK, bool LIMIT>
__device__ __forceinline__ f32x4_t direct_load4(const float* base, int32_t row, uint32_t lane, int kb, int h4,
                                                const DirectDesc& d, const int32_t (&sk)[2]) {
  f32x4_t x = {0.f, 0.f, 0.f, 0.f};
  if constexpr (MK == 1) {
    if constexpr (KV && !LIMIT) {
      x = load4u(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base + kb) + lane));
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (LIMIT && kb + h4 + j >= d.K) continue;
        const float* p = base + (KV ? (int64_t)(kb + j) : (int64_t)(kb + j) * sk[1]);
        x[j] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + lane);
      }
    }
  } else {
    const int kg = kb + h4;
#pragma unroll
    for (int j = 0; j < (KV && !LIMIT ? 1 : 4); ++j) {
      if (LIMIT && kg + j >= d.K) continue;
      const uint32_t q = fast_div((uint32_t)(kg + j), d.mk, d.hk), r = (uint32_t)(kg + j) - q * d.dk;
      const float* p = base + (uint32_t)(row + (int32_t)q * sk[0] + (int32_t)r * sk[1]);
      if constexpr (KV && !LIMIT) x = load4u(p);
      else x[j] = *p;
    }
  }
  return x;
}

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

constexpr int kDirectWaves = 8;   // waves that share a tile's K
constexpr int kDirectLds = kDirectWaves * 16 * 64 + kDirectWaves;   // floats: the waves' sums, their |C| maxima

template <int P, bool AKV, bool BKV, int MK>
__device__ __forceinline__ void direct_tile(const DirectDesc& d, int bid, int bz, float* red) {
  constexpr int WK = kDirectWaves;
  constexpr int CH = DirectInfo<P>::CH, NQ = DirectInfo<P>::NQ;
  constexpr int U = PrecInfo<P>::bf ? 3 : 8;   // chunks in flight (48 or 64 k)
  const int lane = threadIdx.x & 63, r = lane & 31, h4 = (lane >> 5) * 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tn = bid / d.tiles_m, tm = bid - tn * d.tiles_m;
  const int m0 = tm * 32, n0 = tn * 32;
  const float* A = d.a + bz * d.a_bs;
  const float* B = d.b + bz * d.b_bs;
  // rows past the end read the last one: their products are never stored
  const int32_t ao = direct_in(d.gm, (uint32_t)min(m0 + r, d.M - 1));
  const int32_t bo = direct_in(d.gn, (uint32_t)min(n0 + r, d.N - 1));
  const uint32_t al = (uint32_t)(ao + (AKV ? h4 : h4 * d.ska[1])) * 4u;
  const uint32_t bl = (uint32_t)(bo + (BKV ? h4 : h4 * d.skb[1])) * 4u;

  f32x16_t acc = {};
  const int nfull = d.K / CH, nch = (d.K + CH - 1) / CH;
  int c = (int)((uint32_t)(wave * nch) / WK);
  int c1 = (int)((uint32_t)((wave + 1) * nch) / WK);
  const bool tail = wave == WK - 1 && nch != nfull;   // a partial last chunk, read element by element
  c1 -= tail ? 1 : 0;

  struct Frag {
    f32x4_t a[NQ], b[NQ];
  };
  auto load = [&](Frag& f, int ch) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      f.a[q] = direct_load4<AKV, MK, false>(A, ao, al, ch * CH + 8 * q, h4, d, d.ska);
      f.b[q] = direct_load4<BKV, MK, false>(B, bo, bl, ch * CH + 8 * q, h4, d, d.skb);
    }
  };
  // One chunk's products; `refill` issues the loads that take its registers
  // over as soon as they are free.  The split precisions form a chunk's
  // products in a chain from zero and add it to the sum in one rounding (the
  // matrix cores' own accumulation onto a large sum is biased, see
  // gemm_kernel.h).
  auto products = [&](const Frag& f, auto&& refill) {
    if constexpr (!PrecInfo<P>::bf) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[0][e], f.b[0][e], acc, 0, 0, 0);
      refill();
    } else {
      constexpr int NPL = PrecInfo<P>::planes;
      bf16x8_t pa[NPL], pb[NPL];
      direct_planes<P>(f.a, pa);
      direct_planes<P>(f.b, pb);
      refill();
      f32x16_t t = NPL > 1 ? f32x16_t{} : acc;
#pragma unroll
      for (int q = 0; q < PrecInfo<P>::nprod; ++q)
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[prod_a(P, q)], pb[prod_b(P, q)], t, 0, 0, 0);
      if constexpr (NPL > 1) acc += t;
      else acc = t;
    }
  };

  Frag f[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (c + u < c1) load(f[u], c + u);
  if (tail) {
    Frag g;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      g.a[q] = direct_load4<AKV, MK, true>(A, ao, al, nfull * CH + 8 * q, h4, d, d.ska);
      g.b[q] = direct_load4<BKV, MK, true>(B, bo, bl, nfull * CH + 8 * q, h4, d, d.skb);
    }
    products(g, [] {});
  }
  // steady state: every chunk refilled with the one U on
  for (; c + 2 * U <= c1; c += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) products(f[u], [&] { load(f[u], c + u + U); });
  }
  for (; c < c1; c += U) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c1)
        products(f[u], [&] {
          if (c + u + U < c1) load(f[u], c + u + U);
        });
  }

#pragma unroll
  for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 64 + lane] = acc[e];
  float scale = 1.0f;
  if (d.a_scale_bits) scale = pow2_inverse_scale(d.a_scale_bits[bz]);
  float* C = d.c + bz * d.c_bs;
  const int n = n0 + r;
  const int64_t on = direct_out(d.gn, (uint32_t)min(n, d.N - 1));
  __syncthreads();
  constexpr int RPW = 16 / WK;   // accumulator registers that a wave finishes
  float amax = 0.f;
#pragma unroll
  for (int x = 0; x < RPW; ++x) {
    // register e holds row 8 (e / 4) + 4 (lane / 32) + e % 4 of the tile
    const int e = wave * RPW + x;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < WK; ++w) v += red[(w * 16 + e) * 64 + lane];
    v *= scale;
    const int m = m0 + 8 * (e >> 2) + h4 + (e & 3);
    if (m < d.M && n < d.N) {
      C[direct_out(d.gm, (uint32_t)m) + on] = v;
      amax = fmaxf(amax, fabsf(v));
    }
  }
  if (d.c_absmax) {   // one atomic per workgroup
    float* mx = red + WK * 16 * 64;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
    if (lane == 0) mx[wave] = amax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int w = 1; w < WK; ++w) amax = fmaxf(amax, mx[w]);
      atomicMax(d.c_absmax + bz, __float_as_uint(amax));
    }
  }
}

// four waves a SIMD: two workgroups a compute unit, so that one's loads run
// under the other's products
template <int P, bool AKV, bool BKV, int MK>
__global__ void __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
    gemm_direct_kernel(const DirectDesc d) {
  __shared__ float red[kDirectLds];
  direct_tile<P, AKV, BKV, MK>(d, blockIdx.x, blockIdx.z, red);
}

}  // namespace tn
