// Direct contraction kernels (gemm_direct_kernel.h): instantiations, the
// problems they take, and the launch.
#include "gemm_direct_kernel.h"
#include "gemm_inst_decl.h"

namespace tn {

typedef void (*DirectFn)(const DirectDesc);

template <int P>
static DirectFn direct_fn(bool akv, bool bkv, int mk) {
  if (mk == 2)
    return akv ? (bkv ? gemm_direct_kernel<P, true, true, 2> : gemm_direct_kernel<P, true, false, 2>)
               : (bkv ? gemm_direct_kernel<P, false, true, 2> : gemm_direct_kernel<P, false, false, 2>);
  return akv ? (bkv ? gemm_direct_kernel<P, true, true, 1> : gemm_direct_kernel<P, true, false, 1>)
             : (bkv ? gemm_direct_kernel<P, false, true, 1> : gemm_direct_kernel<P, false, false, 1>);
}

static bool direct_rows(const Group& g, DirectRows& r) {
  if (g.n > 3) return false;
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

int32_t launch_gemm_direct(const GemmDesc& d, int32_t prec, hipStream_t st) {
  DirectDesc x;
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
  const int64_t tiles = (int64_t)x.tiles_m * ((d.N + 31) / 32);
  if (tiles >= (1ll << 31) || d.batch > 65535) return fail(TN_ERR_UNSUPPORTED, "grid too large");
  const bool akv = d.a_mode == LOAD_KVEC, bkv = d.b_mode == LOAD_KVEC;
  const int mk = nk == 2 ? 2 : 1;
  DirectFn f = prec == TN_PREC_FP32         ? direct_fn<P_FP32>(akv, bkv, mk)
             : prec == TN_PREC_BF16         ? direct_fn<P_BF16>(akv, bkv, mk)
             : prec == TN_PREC_SPLIT_BF16   ? direct_fn<P_X6>(akv, bkv, mk)
                                            : direct_fn<P_X3>(akv, bkv, mk);
  hipLaunchKernelGGL(f, dim3((unsigned)tiles, 1, (unsigned)d.batch), dim3(kDirectWaves * 64), 0, st, x);
  return hip_check(hipGetLastError(), "direct gemm launch");
}

}  // namespace tn
