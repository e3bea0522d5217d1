// Host-side internal interfaces of the library.
#pragma once

#include <vector>

#include "common.h"

namespace tn {

// ---- tensors -------------------------------------------------------------
int32_t check_tensor(const tn_tensor* t, const char* name, int32_t dtype);
int64_t numel(const tn_tensor& t);
// [lo, hi) byte range touched by a view (hi = lo for an empty view)
void byte_extent(const tn_tensor& t, uintptr_t& lo, uintptr_t& hi);
bool overlaps(const tn_tensor& a, const tn_tensor& b);
bool has_internal_overlap(const tn_tensor& t);
tn_tensor make_view(void* data, int32_t dtype, std::initializer_list<int64_t> shape);
tn_tensor contiguous_view(void* data, int32_t dtype, int32_t rank, const int64_t* shape);

// ---- GEMM plan (contraction of strided views) ------------------------------
// Builds the GEMM view of a tensordot: M = free axes of a (ascending),
// N = free axes of b (ascending), K = pairs in the given order.  Axes of
// extent 1 are dropped and axes contiguous in every tensor of their group
// are merged; each group is ordered so its most contiguous axis is inner.
int32_t plan_gemm(const tn_tensor& a, const tn_tensor& b, int32_t n_pairs, const int32_t* axes_a,
                  const int32_t* axes_b, const tn_tensor& out, GemmDesc& d);
// (re)select the operand load and store modes after a descriptor's pointers
// or batch strides change
void choose_modes(GemmDesc& d);

// reductions: out[r] = sum_k x * y (y may be null)
struct AxisSpec {
  int64_t dim;
  int64_t s[3];
};
void build_group(std::vector<AxisSpec> axes, int primary, int n_strides, Group& g);
// scratch: nullable device buffer of scratch_bytes (TN_REDUCE_WORKSPACE_BYTES
// enables the split reduction of few long sums)
constexpr size_t kReduceScratchBytes = TN_REDUCE_WORKSPACE_BYTES;
int32_t launch_reduce(ReduceDesc& d, void* scratch, size_t scratch_bytes, hipStream_t st);
int32_t reduce_from_axes(const float* x, const float* y, float* out, const std::vector<AxisSpec>& r_axes,
                         const std::vector<AxisSpec>& k_axes, bool bf16_round, void* scratch, size_t scratch_bytes,
                         hipStream_t st);

// ---- GEMM launch -----------------------------------------------------------
int32_t launch_gemm(GemmDesc& d, int32_t prec, hipStream_t st);
// While one of these lives on a thread, launch_gemm on that thread never
// times tile candidates (the cached or heuristic tile is used): timing
// creates HIP events, which the allocation-free entry points avoid.
struct NoTimingScope {
  NoTimingScope();
  ~NoTimingScope();
  bool prev;
};
// While one of these lives on a thread, launch_gemm on that thread serves
// GEMMs that share the chip with a concurrent stream (the two halves of a
// two-directional sweep or inner product): tiles are estimated for half the
// compute units, timed as two copies running at once, and cached apart
// from the same GEMM issued alone.
struct SharedChipScope {
  explicit SharedChipScope(bool on = true);
  ~SharedChipScope();
  bool prev;
};
// While one of these lives on a thread, launch_gemm on that thread may cut
// a GEMM that fills few compute units into k-slices: the slices run as one
// batched launch into dense partial results in `scratch` (device, at least
// `floats` floats; the caller's, not shared with concurrent work) and a
// second kernel adds them in slice order into C.  The tuner times the slice
// counts beside the tiles; the choice is cached with the tile (the cache
// value is tile + 100 log2(slices)).
struct SplitKScope {
  // at most 2^max_lg slices a GEMM (capped at 64)
  SplitKScope(float* scratch, size_t floats, int max_lg = 2);
  ~SplitKScope();
  float* prev_p;
  size_t prev_n;
  int prev_lg;
};
// Householder QR of a column-major m x n FP64 matrix (m >= n, m <= 2048 when
// householder_qr_fits): factorised in place, with the panels' triangular
// factors in tf (householder_tf_doubles(n) doubles) and tau (n doubles);
// householder_apply_q replaces y (m x ncols, column-major) by Q y.
bool householder_qr_fits(int64_t m);
size_t householder_tf_doubles(int64_t n);
int32_t householder_qr(double* xc, int m, int n, double* tau, double* tf, hipStream_t st);
int32_t householder_apply_q(const double* xc, int m, int n, const double* tf, double* y, int ncols, hipStream_t st);
// K <= 32 with N or M <= 16 (and no batch, scale or max-abs): the HBM-bound path
bool gemm_small_fits(const GemmDesc& d);
int32_t launch_gemm_small(const GemmDesc& d, int32_t prec, hipStream_t st);
// direct kernels (gemm_direct.hip): 32 x 32 tiles, eight waves cutting K
bool direct_ok(const GemmDesc& d);
int32_t launch_gemm_direct(const GemmDesc& d, int32_t prec, hipStream_t st);
// whether a GEMM issued now beside another of its size runs whole on the
// direct kernel: few tiles, not a problem of the small-extent path, no tile
// forced, no tuning and no tile cache file that could say otherwise
bool direct_chosen(const GemmDesc& d, int32_t prec);
// the products of such a launch (either may be null): their lines in the log
// and the thread's last choice, as launch_gemm has them
void note_direct(const GemmDesc* l, const GemmDesc* r, int32_t prec);
// two independent GEMMs (either may be null) in one launch of the direct
// kernel, where direct_pair_ok
bool direct_pair_ok(const GemmDesc* l, const GemmDesc* r);
int32_t launch_direct_pair(const GemmDesc* l, const GemmDesc* r, int32_t prec, hipStream_t st);
// a site of the operator sweeps: its environment (L_k or R_k+1), tensors and
// the intermediate it leaves for the second contraction (dense T2[a', t, v, b]
// on the left, T2'[u, a, t, b'] on the right)
struct WstepSite {
  const tn_tensor* env;
  const tn_tensor* site;
  const tn_tensor* mpo;
  float* out;
};
// the first contraction and the operator step of a left and a right site
// (either may be null) in one launch, where direct_wstep_ok
bool direct_wstep_ok(const WstepSite* l, const WstepSite* r);
int32_t launch_direct_wstep(const WstepSite* l, const WstepSite* r, int32_t prec, hipStream_t st);
int32_t launch_gemm_cfg(GemmDesc& d, int32_t prec, int cfg, hipStream_t st);
int gemm_num_cfgs();

// grouped GEMM over compact 2-D problems (uneven batches)
struct Gemm2D {
  const float* a;
  const float* b;
  float* c;
  int32_t M, N, K;
  int64_t sam, sak, sbk, sbn, scm, scn;
  const uint32_t* a_scale_bits;
  uint32_t* c_absmax;
};
// The problem of a grouped launch that holds workgroup bid: the last whose
// first tile is not past it, every wave looking at 64 entries at a time (a
// search by one thread is a chain of loads from a cold cache)
__device__ __forceinline__ int grouped_find(const int32_t* tile_start, int n_probs, int bid) {
  const int lane = threadIdx.x & 63;
  int n = 0;
  for (int i = 0; i < n_probs; i += 64) n += __popcll(__ballot(i + lane < n_probs && tile_start[i + lane] <= bid));
  return __builtin_amdgcn_readfirstlane(n - 1);
}
// variant: 0 run-time gathers; 1..4 fast gathers, for launches whose every
// problem passes grouped_variant with that value
int grouped_variant(const Gemm2D& p);
// cfg 2 (32 x 32 tiles) is the direct kernel, for launches whose every problem
// passes direct_grouped_ok
bool direct_grouped_ok(const Gemm2D& p);
int32_t launch_direct_grouped(const Gemm2D* dev_probs, const int32_t* dev_tile_start, int32_t n_probs,
                              int32_t total_tiles, int32_t prec, int variant, hipStream_t st);
int32_t launch_gemm_grouped(const Gemm2D* dev_probs, const int32_t* dev_tile_start, int32_t n_probs,
                            int32_t total_tiles, int32_t prec, int cfg, int variant, hipStream_t st);
int grouped_tile_m(int cfg);
// the library's side stream for the caller's stream s on the current device
// (s in, side stream out): one of a pool of four per device (created on first
// use, default priority, never destroyed), assigned to caller streams in
// turn and kept, so calls on up to four different streams do not queue
// behind each other's side work.  Work is forked from and joined back into
// the caller's stream by events.
int32_t side_stream(hipStream_t& s);

// A place in one or two streams' work that another stream waits for.  It has
// an event for each stream that it is set on: a capture keeps the events
// recorded on each of its streams until it ends, and destroying an event takes
// it from the stream it was last recorded on alone, so one event for both
// would be looked at by the capture's end after it is gone.
class StreamMark {
 public:
  StreamMark() = default;
  StreamMark(const StreamMark&) = delete;
  StreamMark& operator=(const StreamMark&) = delete;
  ~StreamMark() {
    for (int i = 0; i < n_; ++i) (void)hipEventDestroy(ev_[i]);
  }
  int32_t set(hipStream_t s) {
    int i = 0;
    while (i < n_ && on_[i] != s) ++i;
    if (i == 2) return fail(TN_ERR_DEVICE, "a mark is set on two streams at most");
    if (i == n_) {
      TN_TRY(hip_check(hipEventCreateWithFlags(&ev_[i], hipEventDisableTiming), "create event"));
      on_[i] = s;
      ++n_;
    }
    last_ = i;
    return hip_check(hipEventRecord(ev_[i], s), "record event");
  }
  // s's later work waits for where the mark was last set, if it was
  int32_t wait(hipStream_t s) const {
    return last_ < 0 ? TN_OK : hip_check(hipStreamWaitEvent(s, ev_[last_], 0), "wait event");
  }

 private:
  hipStream_t on_[2] = {};
  hipEvent_t ev_[2] = {};
  int n_ = 0, last_ = -1;
};
// grouped tile configuration pinned by tn_tune_force_grouped_config, or -1
int forced_grouped_cfg();
// the tuning level when timing is allowed on st now (not disabled on this
// thread, stream not capturing), else 0
int tune_timing_level(hipStream_t st);
// tuned grouped tile of a step (signature, precision), or -1; record a choice
// (timed choices are appended to the tile cache file)
int grouped_tune_get(uint64_t sig, int prec);
void grouped_tune_put(uint64_t sig, int prec, int cfg, bool timed);
int grouped_tile_n(int cfg);

// ---- complex contraction on the real path (complex.hip) -----------------------
size_t c64_workspace_bytes(const tn_tensor& b);
int32_t contract_c64_impl(const tn_tensor* a, const tn_tensor* b, int32_t n_pairs, const int32_t* axes_a,
                          const int32_t* axes_b, int conj_a, int conj_b, tn_tensor* out, void* workspace,
                          size_t ws_bytes, int32_t prec, hipStream_t st);

// ---- contraction entry used by the network driver -----------------------------
int32_t contract_between_impl(const tn_tensor* a, const tn_tensor* b, int32_t n_pairs, const int32_t* axes_a,
                              const int32_t* axes_b, tn_tensor* out, void* scratch, size_t scratch_bytes,
                              int32_t prec, hipStream_t st);

}  // namespace tn
