// Direct contraction kernels (gemm_direct_kernel.h): instantiations, the
// problems they take, and the launch.
#include <algorithm>
#include <type_traits>

#include "gemm_direct_kernel.h"
#include "gemm_inst_decl.h"

namespace tn {

typedef void (*DirectFn)(const DirectDesc);

// calls f with the kernel precision as a constant
template <class F>
static void with_prec(int32_t prec, F&& f) {
  if (prec == TN_PREC_FP32) f(std::integral_constant<int, P_FP32>());
  else if (prec == TN_PREC_BF16) f(std::integral_constant<int, P_BF16>());
  else if (prec == TN_PREC_SPLIT_BF16) f(std::integral_constant<int, P_X6>());
  else f(std::integral_constant<int, P_X3>());
}

template <int P, int KM, int MK>
static DirectFn direct_layout(bool akv, bool bkv) {
  return akv ? (bkv ? gemm_direct_kernel<P, KM, KM, MK> : gemm_direct_kernel<P, KM, D_ANY, MK>)
             : (bkv ? gemm_direct_kernel<P, D_ANY, KM, MK> : gemm_direct_kernel<P, D_ANY, D_ANY, MK>);
}

template <int P>
static DirectFn direct_fn(bool akv, bool bkv, int mk, bool staged) {
  if (mk == 2) return direct_layout<P, D_STAGED, 2>(akv, bkv);
  return staged ? direct_layout<P, D_STAGED, 1>(akv, bkv) : direct_layout<P, D_ROW, 1>(akv, bkv);
}

// Operands along k by their own rows while a compute unit has about one tile
// and a wave a few chunks; else through LDS (the figures are at DirectMode's
// reader: at up to 256 tiles they cross near K = 512)
static bool direct_staged(int64_t tiles, int64_t K) { return tiles > 256 || K >= 512; }

static bool direct_rows(const Group& g, DirectRows& r) {
  if (g.n > 3) return false;
  r.one = g.n <= 1;
  Group t;
  t.n = 3;
  for (int i = 0; i < 3; ++i) {
    const int src = i - (3 - g.n);
    t.dim[i] = src >= 0 ? g.dim[src] : 1u;
    r.sx[i] = src >= 0 ? (int32_t)g.s[0][src] : 0;
    r.sc[i] = src >= 0 ? g.s[1][src] : 0;
  }
  set_fast_div(t);
  r.d1 = t.dim[1];
  r.m1 = t.mul[1];
  r.h1 = t.shr[1];
  r.d2 = t.dim[2];
  r.m2 = t.mul[2];
  r.h2 = t.shr[2];
  return true;
}

// Up to three axes a free index, two contracted ones, and every element of
// an operand within 2^31 bytes of its view's base (32-bit offsets).
bool direct_ok(const GemmDesc& d) {
  if (d.gm.n > 3 || d.gn.n > 3 || d.gk.n > 2) return false;
  auto extent = [](const Group& g, int t) {
    int64_t e = 0;
    for (int i = 0; i < g.n; ++i) {
      if (g.s[t][i] < 0) return (int64_t)1 << 40;
      e += (int64_t)(g.dim[i] - 1) * g.s[t][i];
    }
    return e;
  };
  const int64_t lim = (1ll << 29) - 8;
  return extent(d.gm, 0) + extent(d.gk, 0) < lim && extent(d.gn, 0) + extent(d.gk, 1) < lim;
}

static int32_t direct_desc(const GemmDesc& d, DirectDesc& x, int64_t& tiles) {
  x.a = d.a;
  x.b = d.b;
  x.c = d.c;
  x.M = d.M;
  x.N = d.N;
  x.K = d.K;
  x.a_bs = d.a_bs;
  x.b_bs = d.b_bs;
  x.c_bs = d.c_bs;
  x.a_scale_bits = d.a_scale_bits;
  x.c_absmax = d.c_absmax;
  if (!direct_ok(d) || !direct_rows(d.gm, x.gm) || !direct_rows(d.gn, x.gn))
    return fail(TN_ERR_UNSUPPORTED, "problem does not fit the direct kernels");
  // K = 1 has no axis left: stride 0
  const int nk = d.gk.n, last = nk - 1;
  x.dk = nk > 0 ? d.gk.dim[last] : 1;
  x.mk = nk > 0 ? d.gk.mul[last] : 1;
  x.hk = nk > 0 ? d.gk.shr[last] : 0;
  for (int i = 0; i < 2; ++i) {
    const int src = i - (2 - nk);
    x.ska[i] = src >= 0 ? (int32_t)d.gk.s[0][src] : 0;
    x.skb[i] = src >= 0 ? (int32_t)d.gk.s[1][src] : 0;
  }
  x.tiles_m = (d.M + 31) / 32;
  tiles = (int64_t)x.tiles_m * ((d.N + 31) / 32);
  if (tiles >= (1ll << 31) || d.batch > 65535) return fail(TN_ERR_UNSUPPORTED, "grid too large");
  return TN_OK;
}

int32_t launch_gemm_direct(const GemmDesc& d, int32_t prec, hipStream_t st) {
  DirectDesc x;
  int64_t tiles = 0;
  TN_TRY(direct_desc(d, x, tiles));
  const bool akv = d.a_mode == LOAD_KVEC, bkv = d.b_mode == LOAD_KVEC;
  const int mk = d.gk.n == 2 ? 2 : 1;
  const bool staged = direct_staged(tiles * d.batch, d.K);
  DirectFn f = nullptr;
  with_prec(prec, [&](auto p) { f = direct_fn<p.value>(akv, bkv, mk, staged); });
  hipLaunchKernelGGL(f, dim3((unsigned)tiles, 1, (unsigned)d.batch), dim3(kDirectWaves * 64), 0, st, x);
  return hip_check(hipGetLastError(), "direct gemm launch");
}

// ---- tiles of many problems a launch ------------------------------------------

// offsets as in direct_ok
bool direct_grouped_ok(const Gemm2D& p) {
  const int64_t lim = (1ll << 29) - 8;
  auto fits = [&](int64_t rows, int64_t sr, int64_t sk) {
    return sr >= 0 && sk >= 0 && (rows - 1) * sr < lim && (p.K - 1) * sk < lim && (rows - 1) * sr + (p.K - 1) * sk < lim;
  };
  return fits(p.M, p.sam, p.sak) && fits(p.N, p.sbn, p.sbk);
}

int32_t launch_direct_grouped(const Gemm2D* dev_probs, const int32_t* dev_tile_start, int32_t n_probs,
                              int32_t total_tiles, int32_t prec, int variant, hipStream_t st) {
  const bool akv = variant == 1 || variant == 2, bkv = variant == 1 || variant == 3;
  void (*f)(const Gemm2D*, const int32_t*, int32_t) = nullptr;
  with_prec(prec, [&](auto pr) {
    constexpr int P = pr.value;
    f = akv ? (bkv ? gemm_direct_grouped_kernel<P, D_STAGED, D_STAGED> : gemm_direct_grouped_kernel<P, D_STAGED, D_ANY>)
            : (bkv ? gemm_direct_grouped_kernel<P, D_ANY, D_STAGED> : gemm_direct_grouped_kernel<P, D_ANY, D_ANY>);
  });
  hipLaunchKernelGGL(f, dim3((unsigned)total_tiles), dim3(kDirectWaves * 64), 0, st, dev_probs, dev_tile_start, n_probs);
  return hip_check(hipGetLastError(), "direct grouped launch");
}

// ---- two problems a launch ---------------------------------------------------

typedef void (*PairFn)(const DirectPair);

// the layouts that the chains' steps have: both ends (k, any), or the left
// one (any, any) with the right one (k, k)
template <int P, int KM>
static PairFn pair_layout(bool both_ka) {
  return both_ka ? gemm_direct_pair_kernel<P, KM, D_ANY, KM, D_ANY> : gemm_direct_pair_kernel<P, D_ANY, D_ANY, KM, KM>;
}
template <int P>
static PairFn pair_fn(bool both_ka, bool staged) {
  return staged ? pair_layout<P, D_STAGED>(both_ka) : pair_layout<P, D_ROW>(both_ka);
}

// whether an operand can be read in 16-byte loads along k by the kernels of one contracted axis
static bool along_k(int32_t mode, const GemmDesc& d) { return mode == LOAD_KVEC || d.K == 1; }

// 1: both ends (k, any); 2: (any, any) and (k, k); 0: no paired kernel.  The
// first problem may be absent (l = nullptr), as may the second.
static int pair_kind(const GemmDesc* l, const GemmDesc* r) {
  for (const GemmDesc* d : {l, r})
    if (d && (d->batch != 1 || d->gk.n > 1 || !direct_ok(*d))) return 0;
  if ((!l || along_k(l->a_mode, *l)) && (!r || along_k(r->a_mode, *r))) {
    // both kinds fit where the right problem reads both along k: the second
    // kind then loads 16 bytes
    if (!r || !along_k(r->b_mode, *r) || r->K == 1) return 1;
  }
  if (!r || (along_k(r->a_mode, *r) && along_k(r->b_mode, *r))) return 2;
  return 0;
}

bool direct_pair_ok(const GemmDesc* l, const GemmDesc* r) { return pair_kind(l, r) != 0; }

int32_t launch_direct_pair(const GemmDesc* l, const GemmDesc* r, int32_t prec, hipStream_t st) {
  const int kind = pair_kind(l, r);
  if (!kind || (!l && !r)) return fail(TN_ERR_UNSUPPORTED, "no paired kernel for these layouts");
  DirectPair p;
  int64_t t0 = 0, t1 = 0;
  if (l) TN_TRY(direct_desc(*l, p.d0, t0));
  if (r) TN_TRY(direct_desc(*r, p.d1, t1));
  note_direct(l, r, prec);
  if (!l) p.d0 = p.d1;
  if (!r) p.d1 = p.d0;
  if (t0 + t1 >= (1ll << 31)) return fail(TN_ERR_UNSUPPORTED, "grid too large");
  p.tiles0 = (int32_t)t0;
  const bool ka = kind == 1, staged = direct_staged(t0 + t1, (r ? r : l)->K);
  PairFn f = nullptr;
  with_prec(prec, [&](auto pr) { f = pair_fn<pr.value>(ka, staged); });
  hipLaunchKernelGGL(f, dim3((unsigned)(t0 + t1)), dim3(kDirectWaves * 64), 0, st, p);
  return hip_check(hipGetLastError(), "direct pair launch");
}

// ---- first contraction and operator step of a sweep's site --------------------

// every offset below 2^29 elements, no negative stride, unit stride along k
// (left: of the environment; right: of both)
static bool wstep_prob(const WstepSite& s, bool left, DirectWstep& d) {
  const tn_tensor &e = *s.env, &a = *s.site, &w = *s.mpo;
  const int64_t da = a.shape[0], db = a.shape[2], wl = w.shape[0], wr = w.shape[1];
  if (a.shape[1] != 2 || wl > kDirectMaxW || wr > kDirectMaxW) return false;
  for (const tn_tensor* t : {&e, &a, &w}) {
    int64_t ext = 0;
    for (int i = 0; i < t->rank; ++i) {
      if (t->stride[i] < 0) return false;
      ext += (t->shape[i] - 1) * t->stride[i];
    }
    if (ext >= (1ll << 29) - 8) return false;
  }
  const int64_t K = left ? da : db;
  auto unit = [&](int64_t stride) { return stride == 1 || K == 1; };
  if (!unit(e.stride[2]) || (!left && !unit(a.stride[2]))) return false;
  if (da * db * 2 * std::max(wl, wr) >= (1ll << 31)) return false;
  d.w = static_cast<const float*>(w.data);
  d.out = s.out;
  d.K = (int32_t)K;
  d.no_x = (int32_t)da;
  d.no_y = (int32_t)db;
  d.wl = (int32_t)wl;
  d.wr = (int32_t)wr;
  d.w0 = (int32_t)w.stride[0];
  d.w1 = (int32_t)w.stride[1];
  d.w2 = (int32_t)w.stride[2];
  d.w3 = (int32_t)w.stride[3];
  d.ska[0] = d.skb[0] = 0;
  d.dk = d.mk = 1;
  d.hk = 0;
  if (left) {
    d.x = static_cast<const float*>(e.data);
    d.xo = (int32_t)e.stride[0];
    d.xi = (int32_t)e.stride[1];
    d.ska[1] = 1;
    d.ni_x = (int32_t)wl;
    d.y = static_cast<const float*>(a.data);
    d.yo = (int32_t)a.stride[2];
    d.yi = (int32_t)a.stride[1];
    d.skb[1] = (int32_t)a.stride[0];
    d.ni_y = 2;
  } else {
    d.x = static_cast<const float*>(a.data);
    d.xo = (int32_t)a.stride[0];
    d.xi = (int32_t)a.stride[1];
    d.ska[1] = 1;
    d.ni_x = 2;
    d.y = static_cast<const float*>(e.data);
    d.yo = (int32_t)e.stride[0];
    d.yi = (int32_t)e.stride[1];
    d.skb[1] = 1;
    d.ni_y = (int32_t)wr;
  }
  d.per_x = 32 / d.ni_x;
  d.per_y = 32 / d.ni_y;
  d.tiles_x = (d.no_x + d.per_x - 1) / d.per_x;
  return true;
}

typedef void (*WstepFn)(const DirectWstepPair);

// bond: the operator bond if all four are the same (the bulk of the chain;
// the bonds of the Ising and Heisenberg operators have their own kernels)
template <int P>
static WstepFn wstep_fn(bool staged, int bond) {
  if (bond == 3) return staged ? direct_wstep_kernel<P, D_STAGED, 3> : direct_wstep_kernel<P, D_ROW, 3>;
  if (bond == 5) return staged ? direct_wstep_kernel<P, D_STAGED, 5> : direct_wstep_kernel<P, D_ROW, 5>;
  return staged ? direct_wstep_kernel<P, D_STAGED, 0> : direct_wstep_kernel<P, D_ROW, 0>;
}

bool direct_wstep_ok(const WstepSite* l, const WstepSite* r) {
  DirectWstep d;
  return (!l || wstep_prob(*l, true, d)) && (!r || wstep_prob(*r, false, d));
}

int32_t launch_direct_wstep(const WstepSite* l, const WstepSite* r, int32_t prec, hipStream_t st) {
  DirectWstepPair p;
  if ((!l && !r) || (l && !wstep_prob(*l, true, p.l)) || (r && !wstep_prob(*r, false, p.r)))
    return fail(TN_ERR_UNSUPPORTED, "sites do not fit the fused operator step");
  if (!l) p.l = p.r;
  if (!r) p.r = p.l;
  auto tiles = [](const DirectWstep& d) { return (int64_t)d.tiles_x * ((d.no_y + d.per_y - 1) / d.per_y); };
  const int64_t tl = l ? tiles(p.l) : 0, tr = r ? tiles(p.r) : 0;
  if (tl + tr >= (1ll << 31)) return fail(TN_ERR_UNSUPPORTED, "grid too large");
  p.tiles_l = (int32_t)tl;
  const bool staged = direct_staged(tl + tr, (r ? p.r : p.l).K);
  const int wl = p.l.wl, bond = wl == p.l.wr && wl == p.r.wl && wl == p.r.wr ? wl : 0;
  WstepFn f = nullptr;
  with_prec(prec, [&](auto pr) { f = wstep_fn<pr.value>(staged, bond); });
  hipLaunchKernelGGL(f, dim3((unsigned)(tl + tr)), dim3(kDirectWaves * 64), 0, st, p);
  return hip_check(hipGetLastError(), "fused operator step launch");
}

}  // namespace tn
