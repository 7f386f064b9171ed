// runtime.cpp -- host side of the library: contexts, validation, planning of
// the inter-sequence tasks, and the alignment pipeline
//   forward fill -> 32-bit re-run of saturated pairs -> reversed pass (begin)
//   -> banded traceback (CIGAR) -> masked max array (score2) -> records,
// following the order of the paper's method section.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <tuple>
#include <mutex>
#include <numeric>
#include <string>
#include <thread>
#include <vector>

#include "../../include/swx.h"
#include "runtime_internal.h"
#include "swx_internal.h"
#include "swx_kernels.h"

namespace swx {

static thread_local std::string g_last_error;

static int fail(int code, const std::string &msg) {
  g_last_error = msg;
  return code;
}

#define HIP_TRY(expr)                                                                \
  do {                                                                               \
    hipError_t _e = (expr);                                                          \
    if (_e != hipSuccess)                                                            \
      return fail(SWX_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(_e));   \
  } while (0)

// ---- device memory pool ---------------------------------------------------
// Bump allocation from large blocks that are kept across calls; reset() makes
// the whole pool reusable.  Calls on one context are serialised, so a reset at
// the start of a call cannot free memory that a running call still uses.
// In fixed mode (use_fixed) every allocation comes from one given block and
// nothing is ever allocated from the device: a request past its end fails.
class DevArena {
 public:
  ~DevArena() { release(); }
  void reset() {
    cur_ = 0;
    off_ = 0;
    fixed_off_ = 0;
  }
  void use_fixed(void *p, size_t bytes) {
    fixed_ = p;
    fixed_size_ = bytes;
    fixed_off_ = 0;
    fixed_short_ = false;
  }
  void use_pool() { fixed_ = nullptr; }
  bool fixed() const { return fixed_ != nullptr; }
  bool fixed_exhausted() const { return fixed_short_; }
  void release() {
    for (auto &b : blocks_) (void)hipFree(b.ptr);
    blocks_.clear();
    cur_ = 0;
    off_ = 0;
  }
  // returns nullptr on failure
  void *alloc(size_t bytes) {
    bytes = (bytes + 255) & ~size_t(255);
    if (bytes == 0) bytes = 256;
    if (fixed_) {
      if (bytes > fixed_size_ - fixed_off_) {
        fixed_short_ = true;
        return nullptr;
      }
      void *p = (char *)fixed_ + fixed_off_;
      fixed_off_ += bytes;
      return p;
    }
    const size_t cur0 = cur_, off0 = off_;
    while (cur_ < blocks_.size()) {
      Block &b = blocks_[cur_];
      if (off_ + bytes <= b.size) {
        void *p = (char *)b.ptr + off_;
        off_ += bytes;
        return p;
      }
      ++cur_;
      off_ = 0;
    }
    size_t sz = std::max(bytes, size_t(64) << 20);
    void *p = nullptr;
    if (hipMalloc(&p, sz) != hipSuccess) {
      (void)hipGetLastError();   // (a caller with a smaller way to go on launches kernels next)
      cur_ = cur0;
      off_ = off0;
      return nullptr;
    }
    blocks_.push_back({p, sz});
    cur_ = blocks_.size() - 1;
    off_ = bytes;
    return p;
  }
  template <class T>
  T *get(int64_t count) {
    return (T *)alloc(sizeof(T) * (size_t)std::max<int64_t>(count, 1));
  }
  // Everything taken since a mark is given back (no kernel may use it any more).
  struct Mark {
    size_t cur, off, fixed_off;
  };
  Mark mark() const { return {cur_, off_, fixed_off_}; }
  void rewind(const Mark &m) {
    cur_ = m.cur;
    off_ = m.off;
    fixed_off_ = m.fixed_off;
    fixed_short_ = false;
  }

 private:
  struct Block {
    void *ptr;
    size_t size;
  };
  std::vector<Block> blocks_;
  size_t cur_ = 0, off_ = 0;
  void *fixed_ = nullptr;
  size_t fixed_size_ = 0, fixed_off_ = 0;
  bool fixed_short_ = false;
};

// ---- static scratch of the entry point that allocates nothing ---------------
// One array per GPU (each device holds its own copy of a __device__ variable),
// kept until the process ends.  Host code never uses its name as an address:
// the device address comes from hipGetSymbolAddress, taken once per device
// with that device current (at the first context made on it).
static __device__ __align__(256) uint8_t scratch[SWX_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_use[kMaxDevices];   // one call at a time per device

// the device address of `scratch` on `device` (current), or nullptr
static void *scratch_address(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[device] = ptr;
  }
  return g_scratch_ptr[device];
}

}  // namespace swx

struct swx_ctx {
  int device = 0;
  hipStream_t stream = nullptr;   // the stream of the running call (own, or the caller's)
  hipStream_t own = nullptr;      // the context's own stream
  swx::DevArena arena;
  std::mutex mu;
  hipEvent_t ev[8] = {};
  double stage_ms[8] = {};
  int nstages = 0;
  int64_t fill_cells = 0;   // cells of the last forward fill launch
  // of the running batch: longest query and reference, the mean query
  // weighted by reference length, and the mean reference
  int64_t max_q = 0, max_r = 0, mean_q = 0, mean_r = 0;
  // > 0: batches stand for one of this many pairs (the autotuner's samples), and
  // take the routes that depend on the number of pairs as it would
  int64_t route_pairs = 0;
  // routing of long pairs to the intra-sequence path and its launch shape
  int64_t long_cells = -1;                 // qlen * rlen above this (-1: from the batch) ...
  int64_t long_rlen = int64_t(1) << 16;    // ... or a reference longer than this
  int64_t intra_jobs = 2048;               // target column chunks over all long pairs
  int32_t fill_rows = 32;                  // strip height of the batched fill
  int32_t fill_sched = 1;                  // task order of the batched fill (InterArgs::sched)
  int32_t fill_coop = 0;                   // cooperative tasks: 0 automatic, 1 never, 2 always
  int32_t intra_bits = 0;                  // long pairs' lanes: 0 automatic, 16 where scores fit, 32
  int32_t cus = 0;                         // compute units of the device
  unsigned long long *queue = nullptr;     // work-queue counter of the batched fill
  // side streams (default priority) for independent kernels of one stage
  static constexpr int kAux = 3;   // side streams, created on first use
  bool side_streams = true;
  hipStream_t aux[kAux] = {};
  hipEvent_t fork_ev = nullptr;
  hipEvent_t join_ev[kAux] = {};
  // one-pair calls (swx_align): pinned host memory the kernels read the inputs
  // from and write the result to, made on first use
  int8_t *pair_in = nullptr;
  swx::PairOut *pair_out = nullptr;
  // pinned landing area of the small device-to-host reads between stages
  static constexpr int64_t kPinned = 512;   // int64 values
  int64_t *pinned = nullptr;
  uint64_t *pinned_flag = nullptr;          // behind it: the number of the last read (k_publish)
  uint64_t reads = 0, pairs = 0;            // numbers given out (k_publish, k_pair_rest)
  // small host-memory inputs and outputs go through pinned memory that kernels
  // read and write, made on first use
  static constexpr int64_t kStage = int64_t(4) << 20;
  int8_t *stage_in = nullptr, *stage_out = nullptr;
  bool stage_busy = false;                  // stage_in may still be read, on ...
  hipStream_t stage_stream = nullptr;
  int64_t out_used = 0;                     // bytes of stage_out taken by the running call ...
  struct OutCopy { void *dst; const void *src; size_t bytes; };
  std::vector<OutCopy> out_copies;          // ... and what to copy from it when it has finished
  void *scratch = nullptr;   // this device's static scratch (swx_align_batch_noalloc)
};

struct swx_profile {
  swx_ctx *ctx = nullptr;
  std::vector<int8_t> query;
  std::vector<int8_t> matrix;
  int32_t n = 0, o = 0, e = 0;
  // alphabets above 4 symbols: the query profile on the device, built once
  // (forward strips of 32 and of 16 rows, and the reversed table)
  uint8_t *dev = nullptr;
  uint8_t *fwd32 = nullptr, *fwd16 = nullptr, *rev = nullptr;
  int32_t qp32 = 0, qp16 = 0;
  int64_t rev_row = 0;
};

namespace swx {

// Runs a call on the caller's stream: while it lives, ctx->stream names
// `user` (when not null) instead of the context's own stream.  Every stage of
// a call issues its work on ctx->stream, so the call is ordered after the
// work the caller queued on that stream before it; side streams fork from it
// and join back into it.  Callers hold ctx->mu.
struct StreamScope {
  swx_ctx *c;
  hipStream_t saved;
  StreamScope(swx_ctx *c_, void *user) : c(c_), saved(c_->stream) {
    if (user) c->stream = (hipStream_t)user;
  }
  ~StreamScope() { c->stream = saved; }
  StreamScope(const StreamScope &) = delete;
  StreamScope &operator=(const StreamScope &) = delete;
};

struct Scoring {
  int32_t n, o, e, bias, smax;
  const int8_t *dmat;       // device copy
  uint32_t lut[8];
  bool qsel;
};

static int make_scoring(const int8_t *mat, int32_t n, int32_t o, int32_t e, Scoring *sc) {
  if (!mat) return fail(SWX_EINVAL, "matrix is null");
  if (n < 1 || n > 32) return fail(SWX_EINVAL, "alphabet size n must be in [1, 32]");
  if (e < 0 || o < e) return fail(SWX_EINVAL, "gaps must satisfy gap_open >= gap_extend >= 0");
  if (o > 32767) return fail(SWX_EINVAL, "gap_open must be <= 32767");
  int mn = 127, mx = -128;
  for (int k = 0; k < n * n; ++k) {
    mn = std::min<int>(mn, mat[k]);
    mx = std::max<int>(mx, mat[k]);
  }
  sc->n = n;
  sc->o = o;
  sc->e = e;
  // the fills' bias: at least -min S, so that every biased score S + bias is
  // a byte >= 0; the gap open penalty where that qualifies, since the fill's
  // saturating H = hb - bias is then also its H - o (one instruction fewer
  // per cell)
  sc->bias = mn < 0 ? -mn : 0;
  if (o >= sc->bias && o + mx <= 255) sc->bias = o;
  sc->smax = mx;
  sc->qsel = (n <= 4);
  // QSEL column LUTs: lut[r] holds, for query symbols a = 0..3, the biased
  // score S(a, r) + bias in byte a; lut[pad] = 0 (pad scores -bias <= 0).
  for (int r = 0; r < 8; ++r) sc->lut[r] = 0;
  if (sc->qsel) {
    for (int r = 0; r < n; ++r) {
      uint32_t w = 0;
      for (int a = 0; a < n; ++a) w |= (uint32_t)(uint8_t)(mat[a * n + r] + sc->bias) << (8 * a);
      sc->lut[r] = w;
    }
  }
  return SWX_OK;
}

// The query profile of a batch whose pairs all use one query (k_build_qprof):
// forward strips of R rows, and the reversed table of 16 shifted copies.
struct SharedProf {
  const uint8_t *fwd = nullptr, *rev = nullptr;
  int64_t fwd_row = 0, rev_row = 0;
  int32_t qlen = 0, R = 0;
};

// ---- device-side planning of one fill pass ---------------------------------
struct Plan {
  int64_t n = 0, ntasks = 0;
  int lane_bits = 16, R = 32;
  InterTask *d_tasks = nullptr;
  int64_t *d_sorted = nullptr;   // slot -> pair id
  uint32_t *d_bnd = nullptr;
  uint2 *d_rsym = nullptr;       // packed reference symbols
  uint8_t *d_prof = nullptr;
};

static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Waves per task of a batched fill pass: a pass with fewer tasks than the
// device holds waves (two per SIMD) leaves SIMDs idle and makes its largest
// task the critical path, so its tasks run on a workgroup's four waves each.
static int coop_waves(int32_t policy, int64_t ntasks, int32_t cus) {
  if (policy == 1) return 1;
  if (policy == 2) return kCoopWaves;
  return ntasks < (int64_t)cus * 4 * 2 ? kCoopWaves : 1;
}


// Wait for a stream by polling it.  A blocking wait sleeps until an interrupt
// wakes the thread, tens of microseconds after the stream has drained, and
// every host read between the stages of a call paid that with an idle device.
static hipError_t wait_stream(hipStream_t st) {
  for (;;) {
    const hipError_t e = hipStreamQuery(st);
    if (e != hipErrorNotReady) return e;
    std::this_thread::yield();
  }
}

// Waits until a kernel of the stream has written `want` to a word of pinned
// memory: that shows on the host a few microseconds before the end of the
// kernel does.  The stream is asked now and then, so that an error ends the wait.
static hipError_t wait_word(hipStream_t st, const uint64_t *word, uint64_t want) {
  for (uint32_t spins = 1;; ++spins) {
    if (__atomic_load_n(word, __ATOMIC_ACQUIRE) == want) return hipSuccess;
    if (spins % 256 == 0) {
      const hipError_t e = hipStreamQuery(st);
      if (e == hipSuccess)
        return __atomic_load_n(word, __ATOMIC_ACQUIRE) == want ? hipSuccess : hipErrorUnknown;
      if (e != hipErrorNotReady) return e;
      std::this_thread::yield();
    } else {
      __builtin_ia32_pause();
    }
  }
}

template <class T>
static T *alloc_or_null(DevArena &A, int64_t n) { return A.get<T>(n); }

// Sort the pass's pairs by (band, padded query height, reference length) on
// the device, cut them into tasks, derive buffer offsets and allocate.
static int read_two(swx_ctx *ctx, const int64_t *a, int64_t na, const int64_t *b, int64_t nb, int64_t *h);
static int plan_pass(swx_ctx *ctx, const Scoring &sc, const int64_t *ids, int64_t n,
                     const int32_t *qlen, const int64_t *rlen, const int32_t *band,
                     const int32_t *band_q, int lane_bits, int R, Plan &pl,
                     const SharedProf *sp = nullptr) {
  DevArena &A = ctx->arena;
  hipStream_t st = ctx->stream;
  pl = Plan{};
  pl.n = n;
  pl.lane_bits = lane_bits;
  pl.R = R;
  if (n == 0) return SWX_OK;
  const int slots = lane_bits == 16 ? kSlots16 : kSlots32;
  const int halves = lane_bits == 16 ? 2 : 1;
  pl.ntasks = (n + slots - 1) / slots;
  uint64_t *k0 = A.get<uint64_t>(n), *k1 = A.get<uint64_t>(n);
  int64_t *v0 = A.get<int64_t>(n), *v1 = A.get<int64_t>(n);
  pl.d_tasks = A.get<InterTask>(pl.ntasks);
  int64_t *bsz = A.get<int64_t>(pl.ntasks + 1), *qsz = A.get<int64_t>(pl.ntasks + 1);
  int64_t *boff = A.get<int64_t>(pl.ntasks + 1), *qoff = A.get<int64_t>(pl.ntasks + 1);
  if (!k0 || !k1 || !v0 || !v1 || !pl.d_tasks || !bsz || !qsz || !boff || !qoff)
    return fail(SWX_ENOMEM, "device pool exhausted (plan)");
  size_t tmp_bytes = 0;
  HIP_TRY(plan_sort(n, nullptr, ids, qlen, rlen, band, R, ctx->max_q, ctx->max_r, k0, k1, v0, v1, nullptr, &tmp_bytes, nullptr, st));
  void *tmp = A.alloc(tmp_bytes);
  if (!tmp) return fail(SWX_ENOMEM, "device pool exhausted (sort)");
  HIP_TRY(plan_sort(n, nullptr, ids, qlen, rlen, band, R, ctx->max_q, ctx->max_r, k0, k1, v0, v1, tmp, &tmp_bytes, &pl.d_sorted, st));
  // profile bytes per padded row and task; -1: a profile shared by every task
  const int64_t per_row = sc.qsel ? 0 : (sp ? -1 : (int64_t)(sc.n + 1) * halves * 64);
  HIP_TRY(plan_tasks_dev(   // also clears bsz[ntasks], qsz[ntasks]
                         n, nullptr, pl.ntasks, slots, R, per_row, pl.d_sorted, qlen, rlen, band,
                         band_q, pl.d_tasks, bsz, qsz, st));
  size_t t1 = 0, t2 = 0;
  HIP_TRY(launch_exclusive_scan(bsz, boff, pl.ntasks + 1, nullptr, &t1, st));
  void *s1 = A.alloc(t1);
  if (!s1) return fail(SWX_ENOMEM, "device pool exhausted (scan)");
  HIP_TRY(launch_exclusive_scan(bsz, boff, pl.ntasks + 1, s1, &t1, st));
  HIP_TRY(launch_exclusive_scan(qsz, qoff, pl.ntasks + 1, nullptr, &t2, st));
  void *s2 = A.alloc(t2);
  if (!s2) return fail(SWX_ENOMEM, "device pool exhausted (scan)");
  HIP_TRY(launch_exclusive_scan(qsz, qoff, pl.ntasks + 1, s2, &t2, st));
  HIP_TRY(plan_offsets_dev(pl.ntasks, pl.d_tasks, boff, qoff, st));
  int64_t tot[2];
  int rc;
  if ((rc = read_two(ctx, boff + pl.ntasks, 1, qoff + pl.ntasks, 1, tot))) return rc;
  pl.d_bnd = A.get<uint32_t>(tot[0]);
  pl.d_rsym = A.get<uint2>(rsym_offset(tot[0]));
  if (!pl.d_bnd || !pl.d_rsym) return fail(SWX_ENOMEM, "device pool exhausted (boundary planes)");
  if (per_row > 0) {
    pl.d_prof = A.get<uint8_t>(tot[1]);
    if (!pl.d_prof) return fail(SWX_ENOMEM, "device pool exhausted (profiles)");
  }
  return SWX_OK;
}

// Runs independent launches side by side: each goes to a side stream that
// first waits for everything queued on the main stream, and the main stream
// then waits for all of them.  Launches come with a cost estimate (an
// estimated run time alone on the device) and are placed longest first on the
// least loaded of three side streams (the device gives a process four
// hardware queues: with the main stream, one each; measured: the benchmark's
// traceback stage 4.46 -> 4.28 ms against two).  A `lead` launch (one whose few,
// long waves leave most of the device to others) goes first, alone, and its
// stream is charged only kLeadShare of its cost: the launches beside it run
// mostly in its shadow.
struct SideLaunch {
  double cost;
  std::function<hipError_t(hipStream_t)> fn;
  bool lead = false;
};
constexpr double kLeadShare = 0.2;

// Side streams are made on first use, so a context that never needs them
// (short pairs only) holds a single stream and a single hardware queue.
// False when side streams are off or could not be made.
static bool have_side_streams(swx_ctx *ctx) {
  if (!ctx->side_streams) return false;
  bool have = true;
  for (int k = 0; k < swx_ctx::kAux; ++k)
    if (!ctx->aux[k] && hipStreamCreate(&ctx->aux[k]) != hipSuccess) {
      ctx->aux[k] = nullptr;
      have = false;
    }
  return have;
}

static int run_side_by_side(swx_ctx *ctx, std::vector<SideLaunch> &ls) {
  if (ls.empty()) return SWX_OK;
  if (ls.size() == 1 || !ctx->side_streams) {
    for (auto &l : ls) HIP_TRY(l.fn(ctx->stream));
    return SWX_OK;
  }
  constexpr int na = swx_ctx::kAux;
  if (!have_side_streams(ctx)) {   // no side streams: one after the other on the main stream
    for (auto &l : ls) HIP_TRY(l.fn(ctx->stream));
    return SWX_OK;
  }
  std::stable_sort(ls.begin(), ls.end(), [](const SideLaunch &x, const SideLaunch &y) {
    return x.lead != y.lead ? x.lead : x.cost > y.cost;
  });
  HIP_TRY(hipEventRecord(ctx->fork_ev, ctx->stream));
  for (int k = 0; k < na; ++k) HIP_TRY(hipStreamWaitEvent(ctx->aux[k], ctx->fork_ev, 0));
  // place every launch first, then submit stream by stream: the lead's
  // stream is filled before the other one starts (measured: interleaved
  // submission lets the other stream's first kernel take the device first)
  double load[na] = {};
  std::vector<int> where(ls.size());
  for (size_t x = 0; x < ls.size(); ++x) {
    int k = 0;
    for (int y = 1; y < na; ++y)
      if (load[y] < load[k]) k = y;
    load[k] += ls[x].lead ? kLeadShare * ls[x].cost : ls[x].cost;
    where[x] = k;
  }
  for (int k = 0; k < na; ++k)
    for (size_t x = 0; x < ls.size(); ++x)
      if (where[x] == k) HIP_TRY(ls[x].fn(ctx->aux[k]));
  for (int k = 0; k < na; ++k) {
    HIP_TRY(hipEventRecord(ctx->join_ev[k], ctx->aux[k]));
    HIP_TRY(hipStreamWaitEvent(ctx->stream, ctx->join_ev[k], 0));
  }
  return SWX_OK;
}

// profile (general alphabets) + fill for one plan; when mark_fill >= 0,
// events mark_fill and mark_fill + 1 bracket the fill kernel alone
static int run_fill(swx_ctx *ctx, Plan &pl, const Scoring &sc, const PairView &view, bool rev,
                    const int32_t *d_target, FillOut out, int64_t score_bound,
                    int mark_fill = -1, uint32_t anchor = 0, int lastcol = 0,
                    const SharedProf *sp = nullptr) {
  hipStream_t st = ctx->stream;
  if (pl.ntasks == 0) {
    if (mark_fill >= 0) {
      HIP_TRY(hipEventRecord(ctx->ev[mark_fill], st));
      HIP_TRY(hipEventRecord(ctx->ev[mark_fill + 1], st));
    }
    return SWX_OK;
  }
  PackArgs pk{};
  pk.tasks = pl.d_tasks;
  pk.ntasks = pl.ntasks;
  pk.slot_pair = pl.d_sorted;
  pk.view = view;
  pk.prof = pl.d_prof;
  pk.rsym = pl.d_rsym;
  pk.matrix = sc.dmat;
  pk.n = sc.n;
  pk.bias = sc.bias;
  pk.halves = pl.lane_bits == 16 ? 2 : 1;
  pk.strip_rows = pl.R;
  pk.rev = rev ? 1 : 0;
  HIP_TRY(inter_pack_ref(pk, st));
  if (!sc.qsel && !sp) HIP_TRY(inter_pack(pk, st));
  InterArgs a{};
  a.tasks = pl.d_tasks;
  a.ntasks = pl.ntasks;
  a.slot_pair = pl.d_sorted;
  a.view = view;
  a.prof = (sc.qsel || sp) ? nullptr : pl.d_prof;
  if (sp && !sc.qsel) {
    a.qprof = rev ? sp->rev : sp->fwd;
    a.qprof_row = rev ? sp->rev_row : sp->fwd_row;
    a.qprof_copy = (int64_t)(sc.n + 1) * sp->rev_row;
    a.qprof_qlen = sp->qlen;
  }
  a.bnd = pl.d_bnd;
  a.rsym = pl.d_rsym;
  for (int k = 0; k < 8; ++k) a.lut[k] = sc.lut[k];
  a.n = sc.n;
  a.o = sc.o;
  a.e = sc.e;
  a.bias = sc.bias;
  a.rev = rev ? 1 : 0;
  // without a possible score above the 16-bit value field the row code needs
  // no saturation (scores are at most smax * min(qlen, rlen))
  a.clamp = score_bound > kInter16Limit - 1 ? 1 : 0;
  a.pair3 = score_bound <= kInter16PairLimit ? 1 : 0;
  a.code_top = pl.R - 1;
  a.dummy = sc.dmat;   // any readable device bytes
  a.target = d_target;
  a.out = out;
  a.sched = ctx->fill_sched;
  a.cus = ctx->cus;
  a.queue = ctx->queue;
  a.anchor = anchor;
  a.lastcol = lastcol;
  a.coop = coop_waves(ctx->fill_coop, pl.ntasks, ctx->cus);
  // A forward pass with somewhat more tasks than the device holds waves (eight
  // per compute unit: 2048) runs a second round of them, nearly empty at first:
  // cooperative tasks still end sooner, up to a number of tasks per compute
  // unit that was measured for each number of strips (how well they fill four
  // waves is not all of it: five do better than six).  Profiles read per task
  // keep a lone wave waiting, so that four gain more.  Fill on one wave / four
  // waves per task, queries of equal height, references of 300 to 500: four
  // strips 2200 tasks 3.14 / 2.63 ms, 2500 3.22 / 2.92, 2700 3.28 / 3.22; five
  // 2200 3.89 / 3.41, 2500 4.04 / 3.75, 3000 4.14 / 4.49; six 2200 4.70 / 4.88;
  // seven 2200 5.45 / 5.00, 2500 (references of 150 to 500) 3.81 / 3.99; eight
  // 2500 6.39 / 5.58; ten 2200 7.93 / 7.22, 2500 (150 to 500) 5.43 / 5.78; three
  // 2100 3.16 / 3.31.  Profiles per task: four strips 3300 2.59 / 2.55, six 2500
  // 3.31 / 2.70, ten 2500 4.69 / 3.82.
  if (!rev && a.coop == 1 && ctx->fill_coop == 0 && pl.lane_bits == 16 && ctx->mean_q > 0) {
    const int64_t strips = (ctx->mean_q + pl.R - 1) / pl.R;
    int most = 20;   // tasks per two compute units
    if (strips < 4 || (strips == 6 && !a.prof)) most = 16;
    else if (a.prof) most = strips <= 5 ? 26 : 20;
    else if (strips == 5 || strips == 7 || strips == 10) most = 19;
    if (2 * pl.ntasks < most * (int64_t)ctx->cus) a.coop = kCoopWaves;
  }
  // Cooperative tasks of a reversed pass whose queries fill eight strips run on
  // eight waves while the device holds them all so (one per compute unit): 2,000
  // reads of 300 against 1,500, reversed stage on four / eight waves 1.81 / 1.62 ms,
  // proteins 9.59 / 8.01, of 1,000 against 400 7.80 / 7.36.  With more tasks they
  // hold it with their strips' waits where four leave room for other tasks
  // (200,000 reads of 260 against windows of their own 1.86 / 2.65), except in a
  // search of one query among references of very unequal length, whose launch ends
  // on a few large tasks, up to 3.5 tasks per compute unit: lengths log-normal
  // around 300 (sigma 0.6), a query of 300 against 60,000 targets 1.87 / 1.72,
  // 100,000 2.49 / 2.21, of 420 1.93 / 1.82 and 2.46 / 2.57, of 600 2.04 / 2.04 and
  // 2.88 / 2.83; but 200,000 of 420 3.73 / 3.92 (sigma 0.3: 2.27 / 2.96), and 100,000
  // of equal length 1.45 / 1.71.
  if (a.coop > 1 && rev && ctx->mean_q >= kCoopMaxWaves * pl.R &&
      (pl.ntasks <= ctx->cus ||
       (sp && ctx->max_r >= 3 * ctx->mean_r && 2 * pl.ntasks <= 7 * (int64_t)ctx->cus)))
    a.coop = kCoopMaxWaves;
  // A pass runs its tasks by area (padded rows x swept columns, its cost),
  // largest first: the plan's order (by band, height, then width) leaves
  // mid-sized tasks of short, wide pairs for the end of the launch.  Passes
  // whose tasks all start at once (at most two per compute unit) keep the
  // plan's order and save the sort's launches.
  if (pl.ntasks > 2 * (int64_t)std::max(ctx->cus, 1)) {
    DevArena &A = ctx->arena;
    const int64_t nt = pl.ntasks;
    uint64_t *k0 = A.get<uint64_t>(nt), *k1 = A.get<uint64_t>(nt);
    int64_t *v0 = A.get<int64_t>(nt), *v1 = A.get<int64_t>(nt);
    if (!k0 || !k1 || !v0 || !v1) return fail(SWX_ENOMEM, "device pool exhausted (task order)");
    HIP_TRY(inter_area_keys(pl.d_tasks, nt, pl.R, k0, v0, st));
    size_t tb = 0;
    int64_t *order = nullptr;
    HIP_TRY(sort_keys(nt, k0, k1, v0, v1, nullptr, &tb, &order, st, 24));
    void *tmp = A.alloc(tb);
    if (!tmp) return fail(SWX_ENOMEM, "device pool exhausted (task order)");
    HIP_TRY(sort_keys(nt, k0, k1, v0, v1, tmp, &tb, &order, st, 24));
    a.order = order;
  }
  // A reversed pass over many tasks: its largest tasks (full rectangles of
  // weak alignments, no early exit) each take the four waves of a workgroup,
  // launched first beside the rest.  On one wave each they start first and
  // end last: on the benchmark workload the ~50 largest of 7,800 tasks ran
  // 2.0-3.1 ms against 2.1 ms of work per wave slot (the stage went 3.5 ->
  // 3.3 ms with the split).
  const int64_t nsplit = (rev && a.coop == 1 && ctx->fill_coop == 0 && ctx->side_streams &&
                          pl.ntasks >= (int64_t)ctx->cus * 8)
                             ? std::min<int64_t>(pl.ntasks / 16, ctx->cus / 2)
                             : 0;
  if (nsplit > 0 && mark_fill < 0) {
    InterArgs big = a, rest = a;
    big.order = a.order + (pl.ntasks - nsplit);   // the order lists the largest last
    big.ntasks = nsplit;
    big.coop = kCoopWaves;
    big.sched = 1;   // a grid of its own, all resident: no device queue
    rest.ntasks = pl.ntasks - nsplit;
    const int lb = pl.lane_bits, R = pl.R;
    std::vector<SideLaunch> ls;
    ls.push_back({2.0, [=](hipStream_t s_) { return inter_fill(big, lb, R, s_); }, true});
    ls.push_back({1.0, [=](hipStream_t s_) { return inter_fill(rest, lb, R, s_); }});
    return run_side_by_side(ctx, ls);
  }
  if (mark_fill >= 0) HIP_TRY(hipEventRecord(ctx->ev[mark_fill], st));
  HIP_TRY(inter_fill(a, pl.lane_bits, pl.R, st));
  if (mark_fill >= 0) HIP_TRY(hipEventRecord(ctx->ev[mark_fill + 1], st));
  return SWX_OK;
}

static int scan(swx_ctx *ctx, const int64_t *in, int64_t *out, int64_t n) {
  if (n == 0) return SWX_OK;
  size_t tmp = 0;
  HIP_TRY(launch_exclusive_scan(in, out, n, nullptr, &tmp, ctx->stream));
  void *t = ctx->arena.alloc(tmp);
  if (!t) return fail(SWX_ENOMEM, "device pool exhausted (scan)");
  HIP_TRY(launch_exclusive_scan(in, out, n, t, &tmp, ctx->stream));
  return SWX_OK;
}

// n values from the device; small reads land in pinned memory (a direct copy,
// no staging through the runtime's own buffers).  Callers hold ctx->mu.
static int read_two(swx_ctx *ctx, const int64_t *a, int64_t na, const int64_t *b, int64_t nb, int64_t *h) {
  const uint64_t seq = ++ctx->reads;
  HIP_TRY(publish(a, na, b, nb, ctx->pinned, ctx->pinned_flag, seq, ctx->stream));
  HIP_TRY(wait_word(ctx->stream, ctx->pinned_flag, seq));
  memcpy(h, ctx->pinned, 8 * (size_t)(na + nb));
  if (ctx->stream == ctx->stage_stream) ctx->stage_busy = false;
  return SWX_OK;
}

static int read_i64(swx_ctx *ctx, const int64_t *d, int64_t *h, int64_t n = 1) {
  if (n <= swx_ctx::kPinned) return read_two(ctx, d, n, nullptr, 0, h);
  HIP_TRY(hipMemcpyAsync(h, d, 8 * n, hipMemcpyDeviceToHost, ctx->stream));
  HIP_TRY(wait_stream(ctx->stream));
  return SWX_OK;
}

// Host arrays to device buffers (16-byte aligned).  Small ones in one kernel,
// through pinned memory.
struct HostIn { void *dst; const void *src; int64_t bytes; };
static int upload(swx_ctx *ctx, const HostIn *in, int count) {
  int64_t total = 0;
  for (int k = 0; k < count; ++k) total += round_up(in[k].bytes, 16);
  bool pin = !ctx->arena.fixed() && total <= swx_ctx::kStage && count <= kCopySetMax;
  if (pin && !ctx->stage_in &&
      hipHostMalloc(&ctx->stage_in, swx_ctx::kStage, hipHostMallocDefault) != hipSuccess) {
    ctx->stage_in = nullptr;
    pin = false;
  }
  if (!pin) {
    for (int k = 0; k < count; ++k)
      if (in[k].bytes)
        HIP_TRY(hipMemcpyAsync(in[k].dst, in[k].src, in[k].bytes, hipMemcpyHostToDevice, ctx->stream));
    return SWX_OK;
  }
  if (ctx->stage_busy) HIP_TRY(hipStreamSynchronize(ctx->stage_stream));
  CopySet c{};
  int64_t at = 0;
  for (int k = 0; k < count; ++k) {
    if (in[k].bytes == 0) continue;
    memcpy(ctx->stage_in + at, in[k].src, (size_t)in[k].bytes);
    c.add(ctx->stage_in + at, in[k].dst, in[k].bytes);
    at += round_up(in[k].bytes, 16);
  }
  ctx->stage_busy = true;
  ctx->stage_stream = ctx->stream;
  HIP_TRY(copy_set(c, ctx->stream));
  return SWX_OK;
}

// Where kernels write an output of `bytes` bytes for the caller's host memory:
// pinned memory, copied when the call's work has finished (finish_outputs).
// Null: no room there, the caller copies from a device buffer.
static void *host_place(swx_ctx *ctx, int64_t bytes) {
  if (ctx->arena.fixed() || ctx->out_used + round_up(bytes, 256) > swx_ctx::kStage) return nullptr;
  if (!ctx->stage_out &&
      hipHostMalloc(&ctx->stage_out, swx_ctx::kStage, hipHostMallocDefault) != hipSuccess) {
    ctx->stage_out = nullptr;
    return nullptr;
  }
  void *at = ctx->stage_out + ctx->out_used;
  ctx->out_used += round_up(bytes, 256);
  return at;
}
static void *host_out(swx_ctx *ctx, void *dst, int64_t bytes) {
  void *at = host_place(ctx, bytes);
  if (at) ctx->out_copies.push_back({dst, at, (size_t)bytes});
  return at;
}
static void finish_outputs(swx_ctx *ctx) {
  for (const auto &o : ctx->out_copies) memcpy(o.dst, o.src, o.bytes);
  ctx->out_copies.clear();
}

// ids of the pairs whose flag is set (device list) and their count (device)
static int select_flagged_dev(swx_ctx *ctx, const uint8_t *flag, int64_t np, int64_t **ids,
                              const int64_t **count_dev) {
  DevArena &A = ctx->arena;
  int64_t *f64 = A.get<int64_t>(np + 1), *pos = A.get<int64_t>(np + 1);
  *ids = A.get<int64_t>(np);
  if (!f64 || !pos || !*ids) return fail(SWX_ENOMEM, "device pool exhausted (select)");
  HIP_TRY(flags_to_i64(np, flag, f64, ctx->stream));   // also clears f64[np]
  int rc = scan(ctx, f64, pos, np + 1);
  if (rc) return rc;
  HIP_TRY(compact_flags(np, flag, pos, *ids, ctx->stream));
  *count_dev = pos + np;
  return SWX_OK;
}

// the same with the count read back to the host
static int select_flagged(swx_ctx *ctx, const uint8_t *flag, int64_t np, int64_t **ids,
                          int64_t *count) {
  const int64_t *cd = nullptr;
  int rc = select_flagged_dev(ctx, flag, np, ids, &cd);
  if (rc) return rc;
  return read_i64(ctx, cd, count);
}

// ---- banded traceback: classify by band width, one register kernel per
// width class, a general kernel for bands wider than 64 diagonals ------------
struct DeviceBatch {
  const int8_t *qcat, *rcat;
  const int64_t *qoff, *roff, *pair_q, *pair_r;
  int64_t qcat_len, rcat_len, nq, nr, npairs;
};

static int gather_info(swx_ctx *ctx, int64_t n, const int64_t *d_ids, const int32_t *qlen,
                       const int64_t *rlen, const int32_t *score, const int32_t *qend,
                       const int64_t *rend, const int32_t *band, std::vector<int64_t> &info);

// Long pairs take the fastest shapes whose scratch can be had: 0 any, 1 none of
// two rows per lane and no planned chunks (more strips, so more hand-over rows),
// kLean the least scratch.  The call that allocates nothing has 64 MiB for
// everything: 1,000 x 5,000,000 takes 150 MiB of hand-over rows in the planned
// four strips and none in one.
constexpr int kLean = 2;

// Shape of a wave traceback over m rows, w columns and a band of bw diagonals
// when `jobs` such pairs share the device (rl 0: too tall for every choice).
// Strip s starts SH + 110 (spread) or SH + 128 steps after strip s - 1 and sweeps a window of
// SH + bw columns; the waves of a pair's workgroups run its strips in turn,
// and a step costs about 16 instructions per row of a lane plus 30: the
// cheapest of the longer of those two paths.  With fewer pairs than compute
// units a pair's strips spread over up to four waves in each of `segs`
// workgroups (at most one per compute unit, 32 per XCD), as in the
// intra-sequence fill.
// rl_lo, rl_hi: rows per lane to choose from.
struct TbShape {
  int rl, waves, segs;
  bool operator<(const TbShape &x) const {
    return rl != x.rl ? rl < x.rl : waves != x.waves ? waves < x.waves : segs < x.segs;
  }
  bool operator==(const TbShape &x) const { return rl == x.rl && waves == x.waves && segs == x.segs; }
};

static TbShape tb_wave_shape(int64_t m, int64_t w, int64_t bw, int n, int64_t jobs, int32_t cus,
                             int rl_lo, int rl_hi) {
  jobs = std::max<int64_t>(jobs, 1);
  const int64_t segs_max =
      (cus <= 0 || jobs >= cus)
          ? 1
          : std::max<int64_t>(1, std::min<int64_t>(cus / jobs, 32 / ((jobs + 7) / 8)));
  TbShape best{0, 0, 0};
  double best_cost = 0;
  for (int RL : {2, 4, 8, 16}) {
    const int64_t SH = 64 * RL, nstrips = (m + SH - 1) / SH;
    if (RL < rl_lo || RL > rl_hi || nstrips > tb_wave_max_strips()) continue;
    int64_t waves = tb_wave_waves(m, n, RL), g = 1;
    if (segs_max > 1) {
      const int64_t w4 = std::min<int64_t>(4, waves);
      g = std::min<int64_t>(segs_max, (nstrips + w4 - 1) / w4);
      if (g > 1) waves = w4;
    }
    if (RL == 2 && g == 1) continue;   // (spread pairs only)
    const int64_t win = std::min<int64_t>(SH + bw, w + 1) + 63;
    const int64_t chain = (nstrips - 1) * (SH + (g > 1 ? 110 : 128)) + win;
    const int64_t turns = (nstrips + waves * g - 1) / (waves * g) * win;
    const double cost = (double)std::max(chain, turns) * (16 * RL + 30) * (waves > 4 ? 1.5 : 1.0);
    if (best.rl == 0 || cost < best_cost) {
      best = TbShape{RL, (int)waves, (int)g};
      best_cost = cost;
    }
  }
  return best;
}

// Code bytes and hand-over words of a pair on the wave traceback.
static void tb_wave_scratch(const TbWaveJob &jb, int RL, int64_t *dir_bytes, int64_t *bnd_words) {
  const int64_t SH = 64 * RL, nstrips = (jb.m + SH - 1) / SH;
  *dir_bytes = 0;
  for (int64_t s = 0; s < nstrips; ++s) {
    int64_t clo, chi;
    tbw_window(s, SH, jb.dlo, jb.bw, jb.w, &clo, &chi);
    *dir_bytes += ((chi - clo) + 63) * 64 * tb_code_bytes(RL);
  }
  *dir_bytes = round_up(*dir_bytes, 256);
  *bnd_words = 2 * (jb.w + 1) * (nstrips + 1);
}

// The shape with the least scratch (the hand-over words grow with the strips,
// the codes with their height).
static TbShape tb_wave_least(const TbWaveJob &jb, int n, int64_t jobs, int32_t cus) {
  TbShape best{0, 0, 0};
  int64_t least = 0;
  for (int RL : {4, 8, 16}) {
    const TbShape sh = tb_wave_shape(jb.m, jb.w, jb.bw, n, jobs, cus, RL, RL);
    if (sh.rl == 0) continue;
    int64_t d, b;
    tb_wave_scratch(jb, RL, &d, &b);
    if (best.rl == 0 || d + 4 * b < least) {
      best = sh;
      least = d + 4 * b;
    }
  }
  return best;
}

// Traceback a workgroup per pair (k_tb_pairs), by its scratch, which counts
// the waves' steps (128 bytes each): a whole batch up to kTbPairsBytes, else
// its wide bands up to kTbWideBytes.  Measured on reads (traceback stage with
// the per-lane kernels / all by pairs / only wide bands by pairs): 10,000
// reads (0.2 GB) 1.51 / 0.56 / 1.16 ms, 20,000 (0.4 GB) 1.57 / 0.86 / 1.22,
// 50,000 (1 GB, 0.15 wide) 1.52 / 1.66 / 1.35, 100,000 (0.3 wide) 1.77 / 2.94
// / 1.60, 200,000 (0.6 wide) 1.83 / 5.53 / 2.16.  Batches of at most
// kTbPairsAll pairs are not sorted either, unless the sizes turn out larger
// than kTbPairsBytes (then after the read that tells).  The call that allocates nothing keeps
// the per-lane kernels, whose scratch is a few times smaller.
static constexpr int64_t kTbPairsAll = 32768, kTbPairsMax = int64_t(1) << 18;
static constexpr int64_t kTbPairsBytes = int64_t(600) << 20, kTbWideBytes = int64_t(384) << 20;
// Queries of more than 256 rows keep a lane busy for longer: batches of them (on
// average) go by pairs up to twice the size (per-lane kernels / by pairs, a
// protein of 300 against 20,000 targets, 0.8 GB, 3.21 / 1.65 ms, 30,000, 1.2 GB,
// 3.28 / 2.35; of 550 against 20,000, 0.9 GB, 5.00 / 3.57; of 100 against
// 50,000, 0.8 GB, 0.84 / 1.18; 45,000 reads of 100 to 250, 0.9 GB, 1.27 / 1.41).
static constexpr int64_t kTbTallRows = 256, kTbTallBytes = int64_t(1300) << 20;
static constexpr int64_t kTbGraphPairs = 4096, kTbGraphBytes = int64_t(1) << 30;   // of a graph (fixed, worst case)

// A batch traced a workgroup per pair without a class pass: scratch and CIGAR
// words at fixed strides for the longest query and reference, up to
// kTbGraphBytes, so that nothing has to be read back before the kernel.  With
// `defer` the CIGARs' total is not read either: the compaction and the records
// compare it with the capacity on the device, and finish_cigars reads it with
// the call's last read.  101 host reads: 0.39 -> 0.33 ms for the whole call with
// what AloneRest saves (nine launches and two waits less in all).
struct TbDirect {
  int64_t max_q, max_r, stride;
  bool defer;
  // set by run_traceback when it deferred: the total's place, and for host
  // memory the words' place in pinned memory and its room
  const int64_t *total;
  uint32_t *pin;
  int64_t room;
  uint32_t *cscr;
};

static int place_cigars(swx_ctx *ctx, int64_t np, const TbArgs &ta, const int64_t *coff,
                        const uint8_t *cls, const int64_t *cig_off_final, TbDirect *direct,
                        swx_batch_out *out, uint32_t *flags, int *rc_range);

// max_rows: most rows of a pair (the shape of the launch, no limit)
static int run_traceback(swx_ctx *ctx, const Scoring &sc, const DeviceBatch &b, int64_t np,
                         int64_t max_rows, TbDirect *by_stride,
                         const int32_t *score, const int32_t *qbeg, const int32_t *qend,
                         const int64_t *rbeg, const int64_t *rend, const int64_t *qstart,
                         const int64_t *rstart, const int32_t *qlen, const int64_t *rlen,
                         int32_t *cig_len, int64_t *cig_off_final, uint8_t *err,
                         swx_batch_out *out, uint32_t *flags, int *rc_range) {
  DevArena &A = ctx->arena;
  hipStream_t st = ctx->stream;
  int rc;
  TbArgs ta{};
  ta.score = score; ta.qbeg = qbeg; ta.qend = qend; ta.rbeg = rbeg; ta.rend = rend;
  ta.qstart = qstart; ta.rstart = rstart; ta.qlen = qlen; ta.rlen = rlen;
  ta.qcat = b.qcat; ta.rcat = b.rcat; ta.matrix = sc.dmat;
  ta.n = sc.n; ta.o = sc.o; ta.e = sc.e; ta.smax = sc.smax;
  ta.cig_len = cig_len; ta.err = err;
  ta.wave_cells = np <= kTbFewPairs ? kWaveTbCellsFew : kWaveTbCells;
  if (by_stride) {
    ta.cig_stride = by_stride->max_q + by_stride->max_r + 2;
    ta.cig = A.get<uint32_t>(np * ta.cig_stride);
    TbPairs tp{};
    tp.stride = by_stride->stride;
    tp.scratch = A.get<uint8_t>(np * tp.stride);
    if (ta.cig && tp.scratch) {
      HIP_TRY(tb_pairs(ta, tp, np, max_rows, st));
      HIP_TRY(scan_lens(np, cig_len, cig_off_final, st));
      return place_cigars(ctx, np, ta, nullptr, nullptr, cig_off_final, by_stride, out, flags, rc_range);
    }
    // (device memory is short: the classes below take what the pairs need)
  }
  uint8_t *cls = A.get<uint8_t>(np);
  uint64_t *k0 = A.get<uint64_t>(np), *k1 = A.get<uint64_t>(np);
  int64_t *v0 = A.get<int64_t>(np), *v1 = A.get<int64_t>(np);
  int64_t *coff = A.get<int64_t>(np);
  // pairs per class, the CIGAR scratch's words, then the wave kernel's scratch
  // bytes per class and its cursor
  int64_t *counts = A.get<int64_t>(18);
  if (!cls || !k0 || !k1 || !v0 || !v1 || !coff || !counts)
    return fail(SWX_ENOMEM, "device pool exhausted (traceback)");
  HIP_TRY(hipMemsetAsync(counts, 0, 18 * 8, st));
  // a small batch is traced pair by pair, in pair order (k_tb_pairs): it
  // needs no sort unless some of its pairs are long
  const int64_t rp = std::max(np, ctx->route_pairs);
  const bool pairs_ok = !A.fixed() && rp <= kTbPairsMax;
  const bool few = pairs_ok && rp <= kTbPairsAll;
  HIP_TRY(tb_classify(ta, np, cls, k0, v0, coff, counts, counts + 8, pairs_ok ? counts + 9 : nullptr, st));
  int64_t *sorted = nullptr;
  auto sort = [&]() -> int {
    size_t tmp_bytes = 0;
    HIP_TRY(sort_keys(np, k0, k1, v0, v1, nullptr, &tmp_bytes, &sorted, st, kTbKeyBits));
    void *tmp = A.alloc(tmp_bytes);
    if (!tmp) return fail(SWX_ENOMEM, "device pool exhausted (sort)");
    HIP_TRY(sort_keys(np, k0, k1, v0, v1, tmp, &tmp_bytes, &sorted, st, kTbKeyBits));
    return SWX_OK;
  };
  if (!few && (rc = sort())) return rc;
  // the class counts and the scratch sizes in one read
  int64_t hc[17];
  if ((rc = read_i64(ctx, counts, hc, 17))) return rc;
  const int64_t capw = hc[8];
  uint32_t *cscr = A.get<uint32_t>(capw);
  if (!cscr) return fail(SWX_ENOMEM, "device pool exhausted (CIGAR scratch)");
  ta.cig = cscr;
  ta.cig_off = coff;
  // plan every class first, read all their buffer sizes back in one go, then
  // launch the classes' kernels side by side: the small classes would not
  // fill the GPU alone.  totals: [c - 1] code words of band class c, [3] and
  // [4] code and boundary words of the strip class.
  int64_t *totals = A.get<int64_t>(8);
  if (!totals) return fail(SWX_ENOMEM, "device pool exhausted (traceback sizes)");
  struct BandPlan { TbTask *tasks; int64_t nt; int32_t bw; };
  BandPlan bands[3];
  int nbands = 0;
  TbwTask *wtasks = nullptr;
  int64_t wnt = 0;
  // classes traced a workgroup per pair (few: all of them)
  TbPairs tp{};
  int64_t pblocks = 0;
  std::vector<SideLaunch> launches;
  const int64_t pair_bytes = hc[10] + hc[11] + hc[12] + hc[14];
  const double whole = (double)rp / (double)np;   // (of what the batch stands for)
  bool all = pairs_ok && whole * (double)pair_bytes <=
                             (double)(ctx->mean_q > kTbTallRows ? kTbTallBytes : kTbPairsBytes);
  bool wide = !all && pairs_ok && hc[5] > 0 && whole * (double)hc[14] <= (double)kTbWideBytes;
  uint8_t *pscratch = all || wide ? A.get<uint8_t>(all ? pair_bytes : hc[14]) : nullptr;
  if (!pscratch) all = wide = false;   // (the per-lane kernels' scratch is a few times smaller)
  const bool direct = few && all;
  auto by_pairs = [&](int c) { return all || (wide && c == 5); };
  if (few && (!direct || hc[6] > 0) && (rc = sort())) return rc;
  int64_t pos = hc[0];
  for (int c : {1, 2, 3, 5}) {
    if (hc[c] > 0 && by_pairs(c)) {
      tp.lo[tp.ranges] = pos;
      tp.cnt[tp.ranges++] = hc[c];
      pblocks += hc[c];
      tp.cap += hc[9 + c];
      hc[c] = -hc[c];   // done here
    }
    pos += hc[c] < 0 ? -hc[c] : hc[c];
  }
  if (pblocks > 0) {
    tp.sorted = direct ? nullptr : sorted;
    tp.cls = cls;
    tp.used = (unsigned long long *)(counts + 17);
    tp.scratch = pscratch;
    const int64_t blocks = direct ? np : pblocks;
    launches.push_back({(double)tp.cap * 2, [=](hipStream_t s_) { return tb_pairs(ta, tp, blocks, max_rows, s_); }});
  }
  pos = hc[0];
  for (int c = 1; c <= 3; ++c) {
    const int64_t nc = hc[c];
    if (nc < 0) pos -= nc;
    if (nc <= 0) continue;
    const int32_t bw = 8 << (c - 1);
    const int64_t nt = (nc + 63) / 64;
    TbTask *tasks = A.get<TbTask>(nt);
    int64_t *dsz = A.get<int64_t>(nt + 1), *doff = A.get<int64_t>(nt + 1);
    if (!tasks || !dsz || !doff) return fail(SWX_ENOMEM, "device pool exhausted (traceback tasks)");
    HIP_TRY(hipMemsetAsync(dsz + nt, 0, 8, st));
    HIP_TRY(tb_tasks(pos, pos + nc, sorted, ta, bw, tasks, dsz, st));
    if ((rc = scan(ctx, dsz, doff, nt + 1))) return rc;
    HIP_TRY(tb_offsets(nt, tasks, doff, st));
    HIP_TRY(hipMemcpyAsync(totals + (c - 1), doff + nt, sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    bands[nbands++] = BandPlan{tasks, nt, bw};
    pos += nc;
  }
  if (hc[5] < 0) pos -= hc[5];
  if (hc[5] > 0) {   // bands wider than 64 diagonals: row strips, columns swept
    const int64_t nc = hc[5];
    const int64_t nt = (nc + kTbwSlots - 1) / kTbwSlots;
    TbwTask *tasks = A.get<TbwTask>(nt);
    int64_t *dsz = A.get<int64_t>(nt + 1), *doff = A.get<int64_t>(nt + 1);
    int64_t *bsz = A.get<int64_t>(nt + 1), *boff = A.get<int64_t>(nt + 1);
    if (!tasks || !dsz || !doff || !bsz || !boff)
      return fail(SWX_ENOMEM, "device pool exhausted (wide traceback tasks)");
    HIP_TRY(hipMemsetAsync(dsz + nt, 0, 8, st));
    HIP_TRY(hipMemsetAsync(bsz + nt, 0, 8, st));
    HIP_TRY(tbw_tasks(pos, pos + nc, sorted, ta, tasks, dsz, bsz, st));
    if ((rc = scan(ctx, dsz, doff, nt + 1))) return rc;
    if ((rc = scan(ctx, bsz, boff, nt + 1))) return rc;
    HIP_TRY(tbw_offsets(nt, tasks, doff, boff, st));
    HIP_TRY(hipMemcpyAsync(totals + 3, doff + nt, sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipMemcpyAsync(totals + 4, boff + nt, sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    wtasks = tasks;
    wnt = nt;
    pos += nc;
  }
  if (nbands > 0 || wnt > 0) {
    int64_t ht[5];
    if ((rc = read_i64(ctx, totals, ht, 5))) return rc;
    for (int k = 0; k < nbands; ++k) {
      const BandPlan bp = bands[k];
      const int64_t words = ht[(bp.bw == 8 ? 1 : bp.bw == 16 ? 2 : 3) - 1];
      TbArgs tc = ta;
      tc.dir = A.get<uint32_t>(words);
      if (!tc.dir) return fail(SWX_ENOMEM, "device pool exhausted (choice codes)");
      // measured time per cell alone on the device, relative: 8-wide bands
      // pay the most per-row overhead per cell, 16-wide the least
      const double per_cell = bp.bw == 8 ? 2.0 : (bp.bw == 16 ? 1.2 : 1.5);
      launches.push_back({(double)words * 8 * per_cell, [=](hipStream_t s_) {
                            return tb_band(tc, bp.tasks, bp.nt, sorted, bp.bw, s_);
                          }});
    }
    if (wnt > 0) {
      TbArgs tc = ta;
      tc.dir = A.get<uint32_t>(ht[3]);
      int32_t *bnd = A.get<int32_t>(ht[4]);
      if (!tc.dir || !bnd) return fail(SWX_ENOMEM, "device pool exhausted (wide band)");
      launches.push_back({(double)ht[3] * 8 * 1.7,
                          [=](hipStream_t s_) { return tb_strip(tc, wtasks, wnt, sorted, bnd, s_); },
                          true});
    }
  }
  if (hc[6] > 0) {   // long pairs with wide bands: one pair per wave
    const int64_t nc = hc[6];
    std::vector<int64_t> info;
    // gather_pairs fields: qbeg, rbeg, score, qend, rend
    if ((rc = gather_info(ctx, nc, sorted + pos, qbeg, rbeg, score, qend, rend, nullptr, info)))
      return rc;
    std::vector<int64_t> ids(nc);
    if ((rc = read_i64(ctx, sorted + pos, ids.data(), nc))) return rc;
    std::vector<TbWaveJob> jobs(nc);
    std::vector<TbShape> shape(nc);
    int64_t dbytes = 0, bwords = 0;
    int64_t mmax = 0, wmax = 0, bwmax = 0;
    for (int64_t k = 0; k < nc; ++k) {
      TbWaveJob &jb = jobs[k];
      jb.pair = ids[k];
      jb.m = info[6 * k + 3] - info[6 * k + 0] + 1;
      jb.w = info[6 * k + 4] - info[6 * k + 1] + 1;
      safe_band(jb.m, jb.w, info[6 * k + 2], sc.smax, sc.o, sc.e, &jb.dlo, &jb.bw);
      mmax = std::max(mmax, jb.m);
      wmax = std::max(wmax, jb.w);
      bwmax = std::max(bwmax, jb.bw);
    }
    std::vector<int64_t> order(nc);
    std::vector<TbWaveJob> sorted_jobs(nc);
    TbWaveJob *dj = nullptr;
    uint8_t *dirw = nullptr;
    int32_t *bnd = nullptr;
    IntraSync *sync = nullptr;
    int64_t nspread = 0;
    const DevArena::Mark mark = A.mark();
    for (int lean = 0;; ++lean) {   // (kLean: the fastest shapes first)
      // few pairs share one shape, the largest one's, and so one launch (by their
      // own shapes 100 pairs made two, 4.6 ms instead of 4.2)
      const int rl_lo = lean == 0 ? 2 : 4;
      const TbShape common = tb_wave_shape(mmax, wmax, bwmax, sc.n, nc, ctx->cus, rl_lo, 16);
      dbytes = bwords = nspread = 0;
      for (int64_t k = 0; k < nc; ++k) {
        TbWaveJob &jb = jobs[k];
        shape[k] = lean == kLean                         ? tb_wave_least(jb, sc.n, nc, ctx->cus)
                   : nc < ctx->cus && common.rl != 0 ? common
                                                         : tb_wave_shape(jb.m, jb.w, jb.bw, sc.n, nc, ctx->cus, rl_lo, 16);
        if (shape[k].rl == 0) return fail(SWX_EINVAL, "alignment too long for the wave traceback");
        int64_t d, w;
        tb_wave_scratch(jb, shape[k].rl, &d, &w);
        jb.dir_off = dbytes;
        jb.bnd_off = bwords;
        dbytes += d;
        bwords += w;
        nspread += shape[k].segs > 1 ? 1 : 0;
      }
      dj = A.get<TbWaveJob>(nc);
      dirw = A.get<uint8_t>(std::max<int64_t>(dbytes, 256));
      bnd = A.get<int32_t>(std::max<int64_t>(bwords, 1));
      sync = nspread ? A.get<IntraSync>(nspread) : nullptr;
      if (dj && dirw && bnd && (!nspread || sync)) break;
      if (lean == kLean) return fail(SWX_ENOMEM, "device pool exhausted (wave traceback)");
      A.rewind(mark);
    }
    // launch groups of equal shape
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int64_t x, int64_t y) { return shape[x] < shape[y]; });
    for (int64_t k = 0; k < nc; ++k) sorted_jobs[k] = jobs[order[k]];
    HIP_TRY(hipMemcpyAsync(dj, sorted_jobs.data(), sizeof(TbWaveJob) * nc, hipMemcpyHostToDevice, st));
    if (nspread)   // the hand-over words of spread pairs start out invalid
      HIP_TRY(hipMemsetAsync(bnd, 0, sizeof(int32_t) * std::max<int64_t>(bwords, 1), st));
    HIP_TRY(hipStreamSynchronize(st));   // the host job table must outlive the copy
    for (int64_t k0 = 0; k0 < nc;) {
      int64_t k1 = k0;
      while (k1 < nc && shape[order[k1]] == shape[order[k0]]) ++k1;
      const TbShape sh = shape[order[k0]];
      const TbWaveJob *jp = dj + k0;
      const int64_t cnt = k1 - k0;
      IntraSync *gs = nullptr;
      if (sh.segs > 1) {   // one progress record per spread pair
        gs = sync;
        sync += cnt;
      }
      launches.push_back({(double)dbytes * 32, [=](hipStream_t s_) {
                            return tb_wave(ta, jp, cnt, sh.rl, sh.waves, sh.segs, gs, dirw, bnd, s_);
                          }});
      k0 = k1;
    }
    pos += nc;
  }
  if ((rc = run_side_by_side(ctx, launches))) return rc;
  // final CIGAR offsets and compaction into the caller's arena
  if (np <= kScanLensMax) {
    HIP_TRY(scan_lens(np, cig_len, cig_off_final, st));
  } else {
    int64_t *len64 = A.get<int64_t>(np + 1);
    if (!len64) return fail(SWX_ENOMEM, "device pool exhausted");
    HIP_TRY(hipMemsetAsync(len64 + np, 0, 8, st));
    HIP_TRY(lens_to_i64(np, cig_len, len64, st));
    if ((rc = scan(ctx, len64, cig_off_final, np + 1))) return rc;
  }
  return place_cigars(ctx, np, ta, coff, cls, cig_off_final, nullptr, out, flags, rc_range);
}

static int place_cigars(swx_ctx *ctx, int64_t np, const TbArgs &ta, const int64_t *coff,
                        const uint8_t *cls, const int64_t *cig_off_final, TbDirect *direct,
                        swx_batch_out *out, uint32_t *flags, int *rc_range) {
  DevArena &A = ctx->arena;
  hipStream_t st = ctx->stream;
  const int32_t *cig_len = ta.cig_len;
  if (direct && direct->defer) {
    uint32_t *dst = out->cigar;
    direct->room = out->cigar_cap;
    if (out->out_mem != SWX_MEM_DEVICE && dst) {
      // (room kept for the records behind it)
      const int64_t bytes = swx_ctx::kStage - ctx->out_used - round_up((int64_t)sizeof(swx_rec) * np, 256) - 256;
      dst = bytes >= 4096 ? (uint32_t *)host_place(ctx, bytes / 256 * 256) : nullptr;
      if (dst) {
        direct->pin = dst;
        direct->room = std::min<int64_t>(out->cigar_cap, bytes / 256 * 64);
      } else {
        direct->defer = false;
      }
    }
    if (direct->defer) {
      direct->total = cig_off_final + np;
      direct->cscr = ta.cig;
      if (dst)
        HIP_TRY(launch_cigar_compact(np, ta.cig, nullptr, cig_len, cig_off_final, nullptr, ta.qbeg,
                                     ta.qend, dst, ta.cig_stride, direct->room, st));
      return SWX_OK;
    }
  }
  int rc;
  int64_t total = 0;
  if ((rc = read_i64(ctx, cig_off_final + np, &total))) return rc;
  out->cigar_used = total;
  if (total > out->cigar_cap || (total > 0 && !out->cigar)) {
    *flags &= ~SWX_CIGAR;   // records are still produced; CIGARs are not copied
    *rc_range = SWX_ERANGE;
    g_last_error = "CIGAR arena too small";
    return SWX_OK;
  }
  uint32_t *dst = out->cigar, *dtmp = nullptr;
  if (out->out_mem != SWX_MEM_DEVICE && total) {
    dst = (uint32_t *)host_out(ctx, out->cigar, sizeof(uint32_t) * total);
    if (!dst) {
      dtmp = A.get<uint32_t>(total);
      if (!dtmp) return fail(SWX_ENOMEM, "device pool exhausted");
      dst = dtmp;
    }
  }
  HIP_TRY(launch_cigar_compact(np, ta.cig, coff, cig_len, cig_off_final, cls, ta.qbeg, ta.qend, dst,
                               ta.cig_stride, INT64_MAX, st));
  if (dtmp && total)
    HIP_TRY(hipMemcpyAsync(out->cigar, dtmp, sizeof(uint32_t) * total, hipMemcpyDeviceToHost, st));
  return SWX_OK;
}

// ---- the pipeline -----------------------------------------------------------

// ---- long pairs: intra-sequence path ----------------------------------------
struct LongPath {
  int64_t nlong = 0, nshort = 0;
  int64_t *d_long = nullptr;    // long pair ids (device)
  int64_t *d_short = nullptr;   // short pair ids (device; null: every pair is short)
  uint8_t *is_long = nullptr, *is_short = nullptr;   // per pair (device)
  std::vector<int64_t> ids;     // long pair ids (host)
  std::vector<int64_t> info;    // gather_pairs fields per long pair
  std::vector<IntraPair> pairs;
  int64_t max_rlen = 0;
  IntraPair *d_pairs = nullptr;
  uint32_t *d_maxcol = nullptr;
  int32_t *d_part_v = nullptr;  // partial bests of the max-array reductions
  int64_t *d_part_j = nullptr;
};

// Rows per lane of the intra kernel: the fewest instruction slots per column,
// counting padded rows and about 20 instructions of per-step overhead.
static int pick_rl(int64_t rows, int n) {
  int best = 4;
  int64_t best_cost = INT64_MAX;
  for (int RL : {4, 8, 16, 32}) {
    if (intra_lds_bytes(n, RL) + intra_static_lds() > 65536) continue;
    const int64_t strips = (rows + 64 * RL - 1) / (64 * RL);
    const int64_t cost = strips * (12 * RL + 20);
    if (cost < best_cost) { best_cost = cost; best = RL; }
  }
  return best;
}

// Most rows per lane, and so fewest strips, that the profiles leave room for
// (kLean); with two profiles per wave, as in the 16-bit pass, no fewer than pick_rl.
static int most_rl(int n) {
  int best = 4;
  for (int RL : {8, 16, 32})
    if (intra_lds_bytes(n, RL) + intra_static_lds() <= 65536) best = RL;
  return best;
}
static int most_rl16(int64_t rows, int n) {
  int best = pick_rl(rows, n);
  for (int RL : {8, 16, 32})
    if (RL > best && intra_lds_bytes16(n, RL) + 4096 <= 65536) best = RL;
  return best;
}

// Pairs above this many cells go to the intra-sequence path.  In the batched
// path a pair occupies one 16-bit lane half for cells * t; a full GPU holds
// about 2048 waves * 128 halves, so a pair larger than twice the batch's
// average work per half would finish last -- it is faster spread over a wave.
// A batch of few tasks runs each on four waves (cooperative strips), which
// shortens a task's time about four times.
// (k_split_long computes it from the batch's cells; this is its factor.)
static int64_t long_factor(const swx_ctx *ctx, int64_t npairs) {
  const int64_t tasks = (npairs + kSlots16 - 1) / kSlots16;
  return coop_waves(ctx->fill_coop, tasks, ctx->cus) > 1 ? kCoopWaves : 1;
}

static int code_bits(int64_t rows_padded) {
  int k = 1;
  while ((int64_t(1) << k) < rows_padded) ++k;
  return k;
}

static int gather_info(swx_ctx *ctx, int64_t n, const int64_t *d_ids, const int32_t *qlen,
                       const int64_t *rlen, const int32_t *score, const int32_t *qend,
                       const int64_t *rend, const int32_t *band, std::vector<int64_t> &info) {
  int64_t *d = ctx->arena.get<int64_t>(6 * n);
  if (!d) return fail(SWX_ENOMEM, "device pool exhausted (gather)");
  HIP_TRY(gather_pairs(n, d_ids, qlen, rlen, score, qend, rend, band, d, ctx->stream));
  info.resize(6 * n);
  return read_i64(ctx, d, info.data(), 6 * n);
}

// the long and the short pairs' lists, once their counts are known
static int list_pairs(swx_ctx *ctx, int64_t np, LongPath &lp) {
  if (lp.nlong == 0 || lp.d_long) return SWX_OK;
  int rc;
  const int64_t *count = nullptr;
  if ((rc = select_flagged_dev(ctx, lp.is_long, np, &lp.d_long, &count))) return rc;
  return lp.nshort > 0 ? select_flagged_dev(ctx, lp.is_short, np, &lp.d_short, &count) : SWX_OK;
}

// the long pairs' ids and lengths on the host
static int read_long(swx_ctx *ctx, const int32_t *qlen, const int64_t *rlen, LongPath &lp) {
  if (!lp.ids.empty()) return SWX_OK;
  int rc;
  lp.ids.resize(lp.nlong);
  if ((rc = read_i64(ctx, lp.d_long, lp.ids.data(), lp.nlong))) return rc;
  return gather_info(ctx, lp.nlong, lp.d_long, qlen, rlen, nullptr, nullptr, nullptr, nullptr,
                     lp.info);
}

// Most column chunks per pair of a graph's intra-sequence forward pass.
constexpr int64_t kGraphMaxChunks = 16;

// Waves per workgroup of an intra job: one per strip, within the LDS budget
// (a profile of (n + 1) * 64 * RL bytes per wave) and the kernel's maximum.
static int intra_waves(int64_t nstrips, int n, int RL) {
  const int64_t per = (int64_t)intra_lds_bytes(n, RL);
  const int64_t room = (65536 - (int64_t)intra_static_lds()) / per;
  int64_t w = std::min<int64_t>({nstrips, (int64_t)intra_max_waves(), room});
  return (int)std::max<int64_t>(w, 1);
}

// Waves per workgroup of a 16-bit job pair (two profiles per wave in LDS).
static int intra_waves16(int64_t nstrips, int n, int RL) {
  const int64_t per = (int64_t)intra_lds_bytes16(n, RL);
  const int64_t room = (65536 - 4096) / per;
  int64_t w = std::min<int64_t>({nstrips, (int64_t)intra_max_waves(), room});
  return (int)std::max<int64_t>(w, 1);
}

// Widest span of a positive-scoring path (the warm-up of every chunk of a
// long pair): the reference length when gaps cost nothing to extend.
static int64_t intra_warmup(const Scoring &sc, int64_t Lq, int64_t Lr) {
  if (sc.e <= 0) return Lr;
  return Lq + std::max<int64_t>((int64_t)sc.smax * Lq - sc.o, 0) / sc.e + 1;
}

// Column chunk width of a long pair: its share (by reference length) of
// `target` chunks over all long pairs, at least 256 columns and half the
// warm-up, and the whole reference when the warm-up spans it.
static int64_t intra_chunk(const Scoring &sc, int64_t Lq, int64_t Lr, int64_t target,
                           int64_t total_r) {
  const int64_t W = intra_warmup(sc, Lq, Lr);
  if (W >= Lr) return std::max<int64_t>(Lr, 1);
  const int64_t want = std::max<int64_t>(1, target * Lr / std::max<int64_t>(total_r, 1));
  const int64_t C = (Lr + want - 1) / want;
  return std::max<int64_t>(C, std::max<int64_t>(256, W / 2));
}

// Packed 16-bit lanes hold a long pair when no score can pass 2^15 - 2 (the
// a-priori bound smax * min(qlen, rlen) with the bias added on the way: T6)
// and its padded height fits a 16-bit row code.
static bool intra_fits16(const Scoring &sc, int64_t Lq, int64_t Lr, int RL) {
  const int64_t bound = (int64_t)std::max(sc.smax, 0) * std::min(Lq, Lr);
  return bound + sc.bias <= 32766 && round_up(Lq, 64 * RL) <= 65536;
}

// Largest 16-bit lane value for which the packed f16 three-way maximum is the
// unsigned maximum (0x7C00 and above are f16 infinities and NaNs).
static constexpr int64_t kMax3Lane = 0x7BFF;

// 16-bit waves per compute unit from which the automatic choice takes them.
static constexpr int64_t kIntra16MinWavesPerCu = 4;

// Launch shape of intra-sequence jobs: rows per lane, waves per workgroup and
// workgroups per job (segs > 1: the job's strips spread over that many).
struct IntraShape {
  int rl, waves, segs;
  bool operator<(const IntraShape &o) const {
    return std::tie(rl, waves, segs) < std::tie(o.rl, o.waves, o.segs);
  }
};
typedef std::map<IntraShape, std::vector<IntraJob>> IntraGroups;

// Shape of a job of `rows` query rows over `width` columns (band >= 0: the
// reversed pass's strip windows, SH + 2 * band wide and SH apart) when `jobs`
// such jobs share the device.  With at least one job per compute unit the
// device is full: the fewest instructions over all strips (pick_rl).  With
// fewer, a job is as slow as its longer of two paths: the chain of strips,
// each starting about 110 columns (banded: SH + 110) after the one above, and
// the strips each wave runs in turn.  Measured against it, 10,000 x 20,000
// forward in ms at 2 / 4 / 8 rows per lane: one pair 2.30 / 2.66 / 3.93, 30
// pairs 5.19 / 4.55 / 4.02, 100 pairs 16.4 / 11.0 / 10.9 (predicted 2.29 /
// 2.66 / 3.93, 4.8 / 4.4 / 3.9, 16.1 / 10.9 / 10.7).  Those jobs spread over up to four waves per
// workgroup (one per SIMD) and as many workgroups as fit at once: at most one
// per compute unit, and 32 (the compute units of one XCD) per XCD.
static IntraShape intra_shape(int64_t rows, int64_t width, int32_t band, int n, int64_t jobs,
                              int32_t cus, int lean) {
  jobs = std::max<int64_t>(jobs, 1);
  const int rl_lo = lean == 0 ? 2 : lean < kLean ? 4 : most_rl(n);
  if (jobs >= cus || cus <= 0) {
    const int RL = std::max(pick_rl(rows, n), rl_lo);
    return {RL, intra_waves((rows + 64 * RL - 1) / (64 * RL), n, RL), 1};
  }
  const int64_t segs_max =
      std::max<int64_t>(1, std::min<int64_t>(cus / jobs, 32 / ((jobs + 7) / 8)));
  IntraShape best{std::max(pick_rl(rows, n), rl_lo), 1, 1};
  double best_cost = -1;
  for (int RL : {2, 4, 8, 16, 32}) {
    if (RL < rl_lo || intra_lds_bytes(n, RL) + intra_static_lds() > 65536) continue;
    const int64_t SH = 64 * RL;
    const int64_t nstrips = std::max<int64_t>(1, (rows + SH - 1) / SH);
    if (nstrips > intra_max_strips()) continue;
    int64_t nw = std::min<int64_t>(4, intra_waves(nstrips, n, RL));
    const int64_t g = std::min<int64_t>(segs_max, (nstrips + nw - 1) / nw);
    if (g == 1 && RL == 2) continue;   // spread jobs only
    if (g == 1) nw = intra_waves(nstrips, n, RL);
    const int64_t win = band >= 0 ? std::min<int64_t>(width, SH + 2 * (int64_t)band) : width;
    const int64_t lag = (band >= 0 ? SH : 0) + (g > 1 ? 110 : 128);
    const int64_t tw = g * nw;
    const int64_t chain = (nstrips - 1) * lag + win;
    const int64_t turns = (nstrips + tw - 1) / tw * (win + 63);
    // (a step took 80 / 109 / 178 ns at 2 / 4 / 8 rows per lane); two waves
    // share a SIMD beyond four per workgroup
    const double cost = (double)std::max(chain, turns) * (31 * RL + 96) * (nw > 4 ? 1.5 : 1.0);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = {RL, (int)nw, (int)g};
    }
  }
  return best;
}

// How the forward pass of long pairs cuts up: rows per lane and, for one pair,
// columns per chunk, planned so that the waves of all jobs number one per SIMD
// (`lanes` jobs share a wave: two on 16-bit lanes).  A second wave on a SIMD
// halves both (the pass is bound by VALU issue), and only shortens the chunks,
// not their warm-up; short lanes cut a query into strips that run beside each
// other, so that fewer, longer chunks fill the device and repeat less warm-up.
// Only shapes whose workgroups put one wave on each SIMD of a compute unit:
// four strips or more, or (16-bit lanes) one strip, four pairs of jobs to a
// workgroup; workgroups of one or two waves pile up on some SIMDs (1,000 x
// 5,000,000 in two strips: 3.79 ms).  Measured, 16-bit lanes, 1,000 x
// 5,000,000: 1.6 waves per SIMD 3.85 ms, one 2.65; 300 x 5,000,000: 1.69,
// 1.02; 32-bit lanes, 1,000 x 1,000,000: one strip 1.58 ms, four 1.13.
struct FwdPlan {
  int rl = 0;
  int64_t jobs = 0;
  double est = 0;   // instructions of the longest path
};

constexpr int64_t kFwdPlanPairs = 64;

static int64_t fwd_chunk(const Scoring &sc, int64_t Lq, int64_t Lr, int RL, int64_t waves,
                         int64_t max_jobs, int64_t total_r) {
  if (intra_warmup(sc, Lq, Lr) >= Lr) return std::max<int64_t>(Lr, 1);
  const int64_t S = (Lq + 64 * RL - 1) / (64 * RL);
  const double share = (double)Lr / (double)std::max<int64_t>(total_r, 1);
  const int64_t want = std::max<int64_t>(
      1, (int64_t)std::min((double)waves * share / (double)S, (double)max_jobs * share));
  return std::max<int64_t>((Lr + want - 1) / want, 64);
}

// The cheapest plan over the pairs `ids` of info (gather_pairs fields): the
// longer of the longest job's chain of strips (each about 150 columns after
// the one above) and all the work over the SIMDs.
static FwdPlan plan_forward(const Scoring &sc, const std::vector<int64_t> &info,
                            const std::vector<int64_t> &ids, int lanes, int64_t max_jobs,
                            int32_t cus) {
  FwdPlan best;
  int64_t total_r = 0;
  for (int64_t k : ids) total_r += std::max<int64_t>(info[6 * k + 1], 1);
  const int64_t simds = 4 * (int64_t)std::max(cus, 1);
  for (int RL : {4, 8, 16, 32}) {
    const int64_t lds = lanes == 2 ? (int64_t)intra_lds_bytes16(sc.n, RL) + 4096
                                   : (int64_t)(intra_lds_bytes(sc.n, RL) + intra_static_lds());
    if (lds > 65536) continue;
    FwdPlan pl;
    pl.rl = RL;
    double work = 0, chain = 0;
    bool fits = true;
    const double cost = (12 * RL + (lanes == 2 ? 40 : 25));
    for (int64_t k : ids) {
      const int64_t Lq = info[6 * k], Lr = info[6 * k + 1];
      if (Lr == 0) continue;
      const int64_t S = (Lq + 64 * RL - 1) / (64 * RL);
      if (S > intra_max_strips() || (S < 4 && (lanes == 1 || S > 1)) ||
          (lanes == 2 && !intra_fits16(sc, Lq, Lr, RL))) {
        fits = false;
        break;
      }
      const int64_t wv = lanes == 2 ? intra_waves16(S, sc.n, RL) : intra_waves(S, sc.n, RL);
      const int64_t C = fwd_chunk(sc, Lq, Lr, RL, simds * lanes, max_jobs, total_r);
      const int64_t n = (Lr + C - 1) / C, width = std::min(Lr, C + intra_warmup(sc, Lq, Lr));
      pl.jobs += n;
      work += (double)n * (double)S * (double)(width + 63) * cost / lanes;
      const double turns = (double)((S + wv - 1) / wv) * (double)(width + 63);
      chain = std::max(chain, std::max((double)((S - 1) * 150 + width + 63), turns) * cost);
    }
    if (!fits) continue;
    pl.est = std::max(chain, work / (double)simds);
    if (best.rl == 0 || pl.est < best.est) best = pl;
  }
  return best;
}

// 16-bit forward jobs keyed by (rows per lane, strips): jobs of one key share
// their padded height, so any two of them can share a wave.
typedef std::map<std::pair<int, int64_t>, std::vector<IntraJob>> Jobs16;

// Device memory of a launch of long-pair jobs.
struct IntraMem {
  IntraJob *jobs = nullptr, *jobs16 = nullptr;
  IntraSync *sync = nullptr;
  uint32_t *bnd = nullptr;   // hand-over rows, bnd_words of them
  int64_t bnd_words = 0;
};
static bool intra_mem(DevArena &A, const IntraGroups &groups, const Jobs16 &jobs16, int64_t bnd_words,
                      IntraMem &m) {
  int64_t n32 = 0, nspread = 0, n16 = 0;
  for (const auto &kv : groups) {
    n32 += (int64_t)kv.second.size();
    if (kv.first.segs > 1) nspread += (int64_t)kv.second.size();
  }
  for (const auto &kv : jobs16) n16 += round_up((int64_t)kv.second.size(), 2);
  m = IntraMem{};
  m.bnd_words = std::max<int64_t>(bnd_words, 1);
  m.bnd = A.get<uint32_t>(m.bnd_words);
  bool ok = m.bnd != nullptr;
  if (n32) ok = (m.jobs = A.get<IntraJob>(n32)) != nullptr && ok;
  if (nspread) ok = (m.sync = A.get<IntraSync>(nspread)) != nullptr && ok;
  if (n16) ok = (m.jobs16 = A.get<IntraJob>(n16)) != nullptr && ok;
  return ok;
}

// Upload the 16-bit jobs (each key's list padded to an even count with an
// empty job) and launch them, a pair of jobs per workgroup; the stream is waited for.
// packed: jobs of one strip go four waves to a workgroup, a pair of jobs each
// (planned chunks of equal width: a workgroup ends with its longest wave).
static int launch_intra16_jobs(swx_ctx *ctx, const Jobs16 &jobs, IntraArgs a, const IntraMem &mem,
                               const Scoring &sc, bool m3, bool packed) {
  if (jobs.empty()) return SWX_OK;
  std::vector<IntraJob> all;
  std::vector<std::pair<int64_t, int64_t>> span;   // per key: first job, count
  for (const auto &kv : jobs) {
    const int64_t first = (int64_t)all.size();
    all.insert(all.end(), kv.second.begin(), kv.second.end());
    if (all.size() & 1) {
      IntraJob none{};
      none.pair = -1;
      all.push_back(none);
    }
    span.push_back({first, (int64_t)all.size() - first});
  }
  HIP_TRY(hipMemcpyAsync(mem.jobs16, all.data(), sizeof(IntraJob) * all.size(), hipMemcpyHostToDevice,
                         ctx->stream));
  a.bnd = mem.bnd;
  size_t k = 0;
  for (const auto &kv : jobs) {
    const int RL = kv.first.first;
    a.jobs = mem.jobs16 + span[k].first;
    a.njobs = span[k].second;
    int waves = intra_waves16(kv.first.second, sc.n, RL);
    a.segs = 1;
    if (packed && kv.first.second == 1) a.segs = waves = intra_waves16(4, sc.n, RL);
    HIP_TRY(intra_fill16(a, RL, waves, m3, ctx->stream));
    ++k;
  }
  HIP_TRY(hipStreamSynchronize(ctx->stream));   // the host job table must outlive the copy
  return SWX_OK;
}

// Upload jobs (grouped by launch shape) and launch them; the stream is waited for.
static int launch_intra_jobs(swx_ctx *ctx, const IntraGroups &groups, IntraArgs a, const IntraMem &mem,
                             bool rev) {
  std::vector<IntraJob> all;
  int64_t nspread = 0;
  for (const auto &kv : groups) {
    all.insert(all.end(), kv.second.begin(), kv.second.end());
    if (kv.first.segs > 1) nspread += (int64_t)kv.second.size();
  }
  if (all.empty()) return SWX_OK;
  HIP_TRY(hipMemcpyAsync(mem.jobs, all.data(), sizeof(IntraJob) * all.size(), hipMemcpyHostToDevice,
                         ctx->stream));
  if (nspread) {   // the words of spread jobs start out invalid
    HIP_TRY(intra_sync_init(mem.sync, nspread, ctx->stream));
    HIP_TRY(hipMemsetAsync(mem.bnd, 0, sizeof(uint32_t) * mem.bnd_words, ctx->stream));
  }
  a.bnd = mem.bnd;
  int64_t off = 0, soff = 0;
  for (const auto &kv : groups) {
    a.jobs = mem.jobs + off;
    a.njobs = (int64_t)kv.second.size();
    a.segs = kv.first.segs;
    a.sync = kv.first.segs > 1 ? mem.sync + soff : nullptr;
    HIP_TRY(intra_fill(a, kv.first.rl, kv.first.waves, rev, ctx->stream));
    off += a.njobs;
    if (kv.first.segs > 1) soff += a.njobs;
  }
  // the host job table must outlive the copy
  HIP_TRY(hipStreamSynchronize(ctx->stream));
  return SWX_OK;
}

// Forward pass of the long pairs: column chunks with a warm-up overlap, the
// encoded max array per pair, then the end (T1) of each pair.
static int64_t long_rlen(const LongPath &lp) {
  int64_t total = 0;
  for (int64_t k = 0; k < lp.nlong; ++k) total += std::max<int64_t>(lp.info[6 * k + 1], 1);
  return total;
}

// Packed 16-bit lanes run two chunks per wave, with half the waves per
// workgroup (two profiles each in LDS), on twice the chunk target. Chosen
// automatically only when those waves still cover every SIMD of the device:
// a few long pairs in few chunks finish sooner on 32-bit lanes.
static bool choose16(const swx_ctx *ctx, const Scoring &sc, const LongPath &lp) {
  if (ctx->intra_bits != 0) return ctx->intra_bits == 16;
  const int64_t total_r = long_rlen(lp);
  std::map<std::pair<int, int64_t>, int64_t> count;
  for (int64_t k = 0; k < lp.nlong; ++k) {
    const int64_t Lq = lp.info[6 * k], Lr = lp.info[6 * k + 1];
    const int RL = pick_rl(Lq, sc.n);
    if (Lr == 0 || !intra_fits16(sc, Lq, Lr, RL)) continue;
    const int64_t C = intra_chunk(sc, Lq, Lr, 2 * ctx->intra_jobs, total_r);
    count[{RL, round_up(Lq, 64 * RL) / (64 * RL)}] += (Lr + C - 1) / C;
  }
  int64_t waves = 0;
  for (const auto &kv : count)
    waves += (kv.second + 1) / 2 * intra_waves16(kv.first.second, sc.n, kv.first.first);
  return waves >= kIntra16MinWavesPerCu * (int64_t)ctx->cus;
}

// ---- short queries of the long-pair path (AloneArgs) -------------------------
// The long pairs of a batch whose queries have at most kAloneMaxQ rows and
// whose references at most kAloneMaxR columns, each on a wave (or half a
// wave's 16-bit lanes) over its whole reference.
struct AlonePath {
  bool on = false, all = false;   // all: the batched passes are empty
  bool label = false;             // ... and short pairs may reach the batched pass's limit
  int64_t *ids = nullptr;         // (null: every pair in turn)
  int64_t count = 0, n32 = 0;     // the first n32 on 32-bit lanes
  uint32_t *maxcol = nullptr;
  int64_t stride = 0;
  int32_t max_q = 0;
};
// References above kAloneSweep columns keep the chunks of the general path
// until there is a job per pair anyway.
static constexpr int64_t kAloneMaxR = 8192, kAloneSweep = 1024;
// The short pairs of a batch go the same way, on 16-bit lanes too (which hold every
// score here; those that reach the batched pass's limit of them are labelled 32
// bits, as they run there), up to kAlonePairs pairs in all: nothing is batched then, so there is no plan to
// build and read back, no pack, and no fill with a few tasks.
// Measured, whole call, long ones alone / all alone / all batched: 20,000
// reads 3.04 / 2.06 / 3.57 ms, 30,000 3.74 / 2.79 / 3.87; the 4,950 overlaps of 100
// reads of 70 (none long) 0.98 / 0.50 / 0.98, 19,900 of 200 1.17 / 0.81 / 1.17.
// A protein of 300, forward and reversed stage, long ones alone or none / all
// alone: 5,000 targets 1.98 / 1.08 ms, 12,000 3.20 / 1.68, 25,000 4.56 / 3.19,
// 32,000 4.47 / 3.88, 48,000 4.41 / 5.45; of 80, 40,000 2.35 / 1.84.
static constexpr int64_t kAlonePairs = 32768, kAloneMost = 49152;
// With begins wanted, as the reversed passes gain most, batches of shorter
// queries go further.  Here every pair costs the forward sweep of 256 rows (64
// lanes of four), however short its query; batched, the cost does not depend on
// the number of pairs while their tasks all start at once, but on the strips of
// the query (beyond four, the four waves of a task take a second turn), on the
// profile, and on how many pairs are left once the long ones are taken out.
// Batched / all alone, references of 500, 1,000 and 5,000, 36,000 and 42,000
// pairs.  Scores from the selector table: queries of 40 0.84 0.72 0.59 and 0.69
// 0.61 0.52, of 150 1.05 1.02 0.90 and 0.96 0.92 0.87, of 250 1.01 1.09 0.96 and
// 1.04 1.13 1.15 (49,000: 0.90 0.97); 33,000, of which 0.45 are long, 40 1.11 1.01
// 0.91, 150 1.41 1.30 1.19.  One query's profile for all (300, 1,000, 3,000): of 60
// 0.98 1.02 0.62 (49,000 0.87 0.76 0.65), of 150 1.33 1.69 1.36 (49,000 1.18 1.42
// 1.18).  Profiles read per task (500, 1,000, 5,000): of 100 1.59 1.36 0.81 (49,000
// 1.43 1.27 0.72), of 250 2.21 2.12 1.67 (49,000 2.23 2.32).
static int64_t alone_limit(const swx_ctx *ctx, const Scoring &sc, int64_t np, uint32_t flags,
                           int64_t nlong, bool one_query) {
  if (!(flags & SWX_BEGIN) || ctx->mean_q > kTbTallRows) return kAlonePairs;
  const int64_t strips = (ctx->mean_q + 31) / 32;
  const bool brief = ctx->mean_r <= 1024;
  if (!sc.qsel) return strips >= 5 || (brief && !one_query) ? kAloneMost : brief ? 36864 : kAlonePairs;
  if ((strips >= 5 || brief) && 5 * nlong >= 2 * np) return kAloneMost;
  return strips >= 6 ? 43008 : strips == 5 && brief ? 36864 : kAlonePairs;
}

static int plan_alone(swx_ctx *ctx, const Scoring &sc, int64_t np, uint32_t flags, bool one_query,
                      const int64_t *stats, const int32_t *qlen, const int64_t *rlen, LongPath &lp,
                      AlonePath &al) {
  DevArena &A = ctx->arena;
  const int64_t max_q = stats[2], max_r = stats[3], sum_r = stats[4];
  const int64_t bound = (int64_t)std::max(sc.smax, 0) * stats[0];
  if (A.fixed() || max_q > kAloneMaxQ || max_r > kAloneMaxR) return SWX_OK;
  const int64_t rp = std::max(np, ctx->route_pairs);
  if (rp > np && rp > kAloneMost) return SWX_OK;
  // (a threshold set by the caller says itself which pairs are batched)
  const bool all = lp.nshort == 0 || (ctx->long_cells < 0 &&
                                      rp <= alone_limit(ctx, sc, np, flags, lp.nlong, one_query));
  if (lp.nlong == 0 && !all) return SWX_OK;
  const int64_t count = all ? np : lp.nlong;
  if (max_r > kAloneSweep && count < 2 * ctx->intra_jobs) return SWX_OK;
  if (bound + sc.bias > 32766) return SWX_OK;          // (16-bit lanes, 16 code bits)
  // max array words at a fixed stride: within 1 GiB, or few skewed pairs
  if (count * max_r > std::max(int64_t(1) << 28, 4 * sum_r + (int64_t(1) << 20))) return SWX_OK;
  // the lanes that the general path takes: by the number of its chunks, of
  // which a pair has at least one and at most one per 256 columns
  int rc;
  bool w16 = ctx->intra_bits == 16;
  if (ctx->intra_bits == 0) {
    const int64_t need = 2 * kIntra16MinWavesPerCu * (int64_t)ctx->cus;
    w16 = lp.nlong >= need;
    if (!w16 && lp.nlong * ((max_r + 255) / 256) + 2 >= need) {
      if ((rc = list_pairs(ctx, np, lp))) return rc;
      if ((rc = read_long(ctx, qlen, rlen, lp))) return rc;
      w16 = choose16(ctx, sc, lp);
    }
  }
  al.on = true;
  al.all = all;
  al.count = count;
  al.label = all && lp.nshort > 0 && bound >= kInter16Limit;
  al.n32 = w16 ? 0 : lp.nlong;
  al.stride = max_r;
  al.max_q = (int32_t)max_q;
  al.maxcol = A.get<uint32_t>(al.count * max_r);
  if (!al.maxcol) {   // device memory is short: the general path takes less
    al = AlonePath{};
    return SWX_OK;
  }
  if ((!al.all || (lp.nlong > 0 && lp.nshort > 0 && !w16)) && (rc = list_pairs(ctx, np, lp))) return rc;
  if (!al.all) {
    al.ids = lp.d_long;
  } else if (lp.nlong > 0 && lp.nshort > 0 && !w16) {   // the long pairs first
    al.ids = A.get<int64_t>(np);
    if (!al.ids) return fail(SWX_ENOMEM, "device pool exhausted (pair list)");
    HIP_TRY(hipMemcpyAsync(al.ids, lp.d_long, 8 * lp.nlong, hipMemcpyDeviceToDevice, ctx->stream));
    HIP_TRY(hipMemcpyAsync(al.ids + lp.nlong, lp.d_short, 8 * lp.nshort, hipMemcpyDeviceToDevice,
                           ctx->stream));
  }
  if (al.all) {   // none is left to batch
    lp.nshort = 0;
    lp.nlong = np;
  }
  return SWX_OK;
}

static AloneArgs alone_args(const Scoring &sc, const AlonePath &al, const PairView &view,
                            const FillOut &out) {
  AloneArgs a{};
  a.ids = al.ids;
  a.count = al.count;
  a.view = view;
  a.matrix = sc.dmat;
  a.n = sc.n; a.o = sc.o; a.e = sc.e; a.bias = sc.bias;
  a.max_q = al.max_q;
  a.maxcol = al.maxcol;
  a.stride = al.stride;
  a.out = out;
  return a;
}

static IntraPairArgs alone_pairs(const AlonePath &al, const int32_t *qlen, const int64_t *rlen) {
  IntraPairArgs e{};
  e.ids = al.ids;
  e.stride = al.stride;
  e.maxcol = al.maxcol;
  e.qlen = qlen;
  e.rlen = rlen;
  e.max_rlen = al.stride;
  return e;
}

// What follows the forward pass of a batch that takes this path as a whole:
// begins, and with SWX_SCORE2 score2, by the same wave (32-bit lanes) or one
// kernel (null arrays: the forward pass alone).
struct AloneRest {
  int32_t *qbeg = nullptr, *score2 = nullptr;
  int64_t *rbeg = nullptr, *rend2 = nullptr;
  uint8_t *err = nullptr;
  int32_t mask_len = 0;
};
static void add_rest(AloneArgs &a, const Scoring &sc, const AloneRest &r) {
  a.smax = sc.smax;
  a.mask_len = r.mask_len;
  a.qbeg = r.qbeg; a.score2 = r.score2; a.rbeg = r.rbeg; a.rend2 = r.rend2;
  a.err = r.err;
}

static int run_alone_forward(swx_ctx *ctx, const Scoring &sc, const AlonePath &al, int64_t bound,
                             const PairView &view, const FillOut &out, uint8_t *lanebits,
                             const uint8_t *is_long, const AloneRest &rest) {
  AloneArgs a = alone_args(sc, al, view, out);
  add_rest(a, sc, rest);
  if (al.n32 > 0) {
    AloneArgs w = a;
    w.count = al.n32;
    w.lanebits = lanebits;
    if (rest.qbeg) HIP_TRY(alone_pass(w, ctx->stream));
    else HIP_TRY(alone_forward(w, ctx->stream));
  }
  if (al.count > al.n32) {
    a.is_long = is_long;
    a.lanebits = lanebits;
    if (al.n32 > 0) a.ids += al.n32;   // (a list, then)
    a.maxcol += al.n32 * al.stride;
    a.count -= al.n32;
    HIP_TRY(alone_forward16(a, bound + sc.bias <= kMax3Lane, ctx->stream));
    if (rest.qbeg) HIP_TRY(alone_begin(a, ctx->stream));
  }
  return SWX_OK;
}

static int run_intra_forward(swx_ctx *ctx, const Scoring &sc, LongPath &lp, const PairView &view,
                             const FillOut &out, uint8_t *err, uint8_t *lanebits) {
  DevArena &A = ctx->arena;
  int rc;
  if ((rc = read_long(ctx, view.qlen, view.rlen, lp))) return rc;
  const int64_t total_r = long_rlen(lp);
  for (int64_t k = 0; k < lp.nlong; ++k) lp.max_rlen = std::max(lp.max_rlen, lp.info[6 * k + 1]);
  const bool auto16 = choose16(ctx, sc, lp);
  // lanes of each pair, and the 32-bit jobs that will share the device
  std::vector<uint8_t> is16(lp.nlong);
  std::vector<int64_t> k16, k32, ids16, ids32;
  int64_t jobs32 = 0, r16 = 0, r32 = 0, mc_words = 0;
  for (int64_t k = 0; k < lp.nlong; ++k) {
    const int64_t Lq = lp.info[6 * k], Lr = lp.info[6 * k + 1];
    is16[k] = auto16 && intra_fits16(sc, Lq, Lr, pick_rl(Lq, sc.n));
    (is16[k] ? k16 : k32).push_back(k);
    (is16[k] ? ids16 : ids32).push_back(lp.ids[k]);
    (is16[k] ? r16 : r32) += std::max<int64_t>(Lr, 1);
    mc_words += Lr;
    if (!is16[k] && Lr > 0) {
      const int64_t C = intra_chunk(sc, Lq, Lr, ctx->intra_jobs, total_r);
      jobs32 += (Lr + C - 1) / C;
    }
  }
  lp.d_maxcol = A.get<uint32_t>(std::max<int64_t>(mc_words, 1));
  lp.d_pairs = A.get<IntraPair>(lp.nlong);
  lp.d_part_v = A.get<int32_t>(lp.nlong * intra_slices());
  lp.d_part_j = A.get<int64_t>(lp.nlong * intra_slices());
  if (!lp.d_maxcol || !lp.d_pairs || !lp.d_part_v || !lp.d_part_j)
    return fail(SWX_ENOMEM, "device pool exhausted (max array)");
  if (mc_words > 0) HIP_TRY(hipMemsetAsync(lp.d_maxcol, 0, sizeof(uint32_t) * mc_words, ctx->stream));
  const int64_t simds = 4 * (int64_t)std::max(ctx->cus, 1);
  Jobs16 jobs16;
  IntraGroups groups;
  IntraMem mem;
  bool m3 = true;       // every 16-bit pair's lane values below 0x7C00
  bool plan16 = false;  // 16-bit chunks planned
  const DevArena::Mark mark = A.mark();
  for (int lean = 0;; ++lean) {   // (kLean: the fastest shapes first)
    jobs16.clear();
    groups.clear();
    lp.pairs.clear();
    // a few pairs are planned together (many fill the device by their number);
    // 32-bit jobs that leave compute units idle spread over several workgroups
    // each (intra_shape) instead
    FwdPlan f16, f32;
    if (lp.nlong <= kFwdPlanPairs && lean == 0) {
      f16 = plan_forward(sc, lp.info, k16, 2, 2 * ctx->intra_jobs, ctx->cus);
      f32 = plan_forward(sc, lp.info, k32, 1, ctx->intra_jobs, ctx->cus);
    }
    plan16 = f16.rl != 0;
    const bool plan32 = f32.rl != 0 && f32.jobs >= ctx->cus;
    IntraShape common32{};   // ... all in one launch, by the largest job's shape
    if (!plan32 && jobs32 > 0 && jobs32 < ctx->cus) {
      int64_t rows = 0, width = 0;
      for (int64_t k : k32) {
        const int64_t Lq = lp.info[6 * k], Lr = lp.info[6 * k + 1];
        rows = std::max(rows, Lq);
        width = std::max(width, std::min(Lr, intra_chunk(sc, Lq, Lr, ctx->intra_jobs, total_r) +
                                                 intra_warmup(sc, Lq, Lr)));
      }
      common32 = intra_shape(rows, width, -1, sc.n, jobs32, ctx->cus, lean);
    }
    int64_t mc_off = 0, bnd_words = 0;
    for (int64_t k = 0; k < lp.nlong; ++k) {
      const int64_t p = lp.ids[k], Lq = lp.info[6 * k], Lr = lp.info[6 * k + 1];
      const bool w16 = is16[k];
      const int64_t W = intra_warmup(sc, Lq, Lr);
      int64_t C = intra_chunk(sc, Lq, Lr, (w16 ? 2 : 1) * ctx->intra_jobs, total_r);
      IntraShape shape{};
      if (w16 && plan16) {
        C = fwd_chunk(sc, Lq, Lr, f16.rl, 2 * simds, 2 * ctx->intra_jobs, r16);
        shape = IntraShape{f16.rl, 0, 1};
      } else if (!w16 && plan32) {
        C = fwd_chunk(sc, Lq, Lr, f32.rl, simds, ctx->intra_jobs, r32);
        shape = IntraShape{f32.rl, intra_waves((Lq + 64 * f32.rl - 1) / (64 * f32.rl), sc.n, f32.rl), 1};
      } else if (w16) {
        shape = IntraShape{lean == kLean ? most_rl16(Lq, sc.n) : pick_rl(Lq, sc.n), 0, 1};
      } else {
        shape = common32.rl != 0 ? common32
                                 : intra_shape(Lq, std::min(Lr, C + W), -1, sc.n, jobs32, ctx->cus, lean);
      }
      const int RL = shape.rl;
      const int64_t SH = 64 * RL;
      const int64_t qp = (Lq + SH - 1) / SH * SH;
      const int64_t bound = (int64_t)std::max(sc.smax, 0) * std::min(Lq, Lr);
      const int kb = w16 ? 16 : code_bits(qp);
      if (kb > 30 || bound >= (int64_t(1) << (32 - kb)))
        return fail(SWX_EOVERFLOW, "long pair: score range and query length exceed the max-array word");
      if (w16 && bound + sc.bias > kMax3Lane) m3 = false;
      lp.pairs.push_back(IntraPair{p, mc_off, kb, (int32_t)SH});
      if (Lr > 0) {
        const int64_t nstrips = qp / SH;
        if (nstrips > intra_max_strips())
          return fail(SWX_EINVAL, "query too long for the intra-sequence path");
        for (int64_t c0 = 0; c0 < Lr; c0 += C) {
          IntraJob jb{};
          jb.pair = p;
          jb.c0 = c0;
          jb.c1 = std::min(Lr, c0 + C);
          jb.cw = std::max<int64_t>(0, c0 - W);
          jb.mc_off = mc_off;
          jb.bnd_off = bnd_words;
          jb.kbits = kb;
          jb.band = -1;
          bnd_words += 2 * (jb.c1 - jb.cw) * (nstrips - 1);
          if (w16) jobs16[{RL, nstrips}].push_back(jb);
          else groups[shape].push_back(jb);
        }
      }
      mc_off += Lr;
    }
    if (intra_mem(A, groups, jobs16, bnd_words, mem)) break;
    if (lean == kLean) return fail(SWX_ENOMEM, "device pool exhausted (hand-over rows)");
    A.rewind(mark);
  }
  HIP_TRY(hipMemcpyAsync(lp.d_pairs, lp.pairs.data(), sizeof(IntraPair) * lp.nlong,
                         hipMemcpyHostToDevice, ctx->stream));
  IntraArgs a{};
  a.view = view;
  a.matrix = sc.dmat;
  a.n = sc.n; a.o = sc.o; a.e = sc.e; a.bias = sc.bias;
  a.maxcol = lp.d_maxcol;
  a.err = err;
  if ((rc = launch_intra_jobs(ctx, groups, a, mem, false))) return rc;
  if ((rc = launch_intra16_jobs(ctx, jobs16, a, mem, sc, m3, plan16))) return rc;
  A.rewind(mark);   // (both have been waited for)
  // lane widths of the long pairs (diagnostic)
  for (int w = 0; w < 2; ++w) {
    const std::vector<int64_t> &ids = w ? ids32 : ids16;
    if (ids.empty()) continue;
    int64_t *d = A.get<int64_t>((int64_t)ids.size());
    if (!d) return fail(SWX_ENOMEM, "device pool exhausted (lane widths)");
    HIP_TRY(hipMemcpyAsync(d, ids.data(), 8 * ids.size(), hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(mark_lanes((int64_t)ids.size(), d, lanebits, w ? 32 : 16, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));   // the host list must outlive the copy
  }
  IntraPairArgs e{};
  e.pairs = lp.d_pairs; e.maxcol = lp.d_maxcol; e.qlen = view.qlen; e.rlen = view.rlen;
  e.score = out.score; e.qend = out.qend; e.rend = out.rend; e.overflow = out.overflow;
  e.part_v = lp.d_part_v; e.part_j = lp.d_part_j; e.max_rlen = lp.max_rlen;
  HIP_TRY(intra_end(e, lp.nlong, ctx->stream));
  return SWX_OK;
}

// Reversed pass of the long pairs with a positive score: one job per pair.
static int run_intra_reverse(swx_ctx *ctx, const Scoring &sc, LongPath &lp, const PairView &rview,
                             const int32_t *score, const int32_t *qend, const int64_t *rend,
                             const int32_t *band, const int32_t *tgt, const FillOut &rout,
                             uint8_t *err) {
  std::vector<int64_t> info;
  int rc;
  if ((rc = gather_info(ctx, lp.nlong, lp.d_long, nullptr, nullptr, score, qend, rend, band, info)))
    return rc;
  int64_t njobs = 0;
  int64_t max_rows = 0, max_cols = 0, max_band = 0;
  for (int64_t k = 0; k < lp.nlong; ++k) {
    if (info[6 * k + 2] <= 0) continue;
    ++njobs;
    max_rows = std::max(max_rows, info[6 * k + 3] + 1);
    max_cols = std::max(max_cols, info[6 * k + 4] + 1);
    const int64_t band = info[6 * k + 5];   // (none: negative)
    max_band = band < 0 || max_band < 0 ? -1 : std::max(max_band, band);
  }
  IntraGroups groups;
  IntraMem mem;
  DevArena &A = ctx->arena;
  const DevArena::Mark mark = A.mark();
  for (int lean = 0;; ++lean) {   // (kLean: the fastest shapes first)
    groups.clear();
    int64_t bnd_words = 0;
    // jobs that leave compute units idle share one shape, the largest job's, and
    // so one launch: by their own shapes 50 pairs made two, one after the other
    const IntraShape common = intra_shape(max_rows, max_cols, (int32_t)max_band, sc.n, njobs, ctx->cus, lean);
    for (int64_t k = 0; k < lp.nlong; ++k) {
      if (info[6 * k + 2] <= 0) continue;
      const int64_t rows = info[6 * k + 3] + 1, cols = info[6 * k + 4] + 1;
      const IntraShape shape =
          njobs < ctx->cus ? common
                           : intra_shape(rows, cols, (int32_t)info[6 * k + 5], sc.n, njobs, ctx->cus, lean);
      const int RL = shape.rl;
      const int64_t SH = 64 * RL;
      const int64_t qp = (rows + SH - 1) / SH * SH;
      const int kb = code_bits(qp);
      if (kb > 30 || info[6 * k + 2] >= (int64_t(1) << (32 - kb)))
        return fail(SWX_EOVERFLOW, "long pair: score range and query length exceed the max-array word");
      const int64_t nstrips = qp / SH;
      if (nstrips > intra_max_strips())
        return fail(SWX_EINVAL, "query too long for the intra-sequence path");
      IntraJob jb{};
      jb.pair = lp.ids[k];
      jb.cw = 0; jb.c0 = 0; jb.c1 = cols;
      jb.mc_off = 0;
      jb.bnd_off = bnd_words;
      jb.kbits = kb;
      jb.band = (int32_t)info[6 * k + 5];
      bnd_words += 2 * cols * (nstrips - 1);
      groups[shape].push_back(jb);
    }
    if (intra_mem(A, groups, Jobs16{}, bnd_words, mem)) break;
    if (lean == kLean) return fail(SWX_ENOMEM, "device pool exhausted (intra jobs)");
    A.rewind(mark);
  }
  IntraArgs a{};
  a.view = rview;
  a.matrix = sc.dmat;
  a.n = sc.n; a.o = sc.o; a.e = sc.e; a.bias = sc.bias;
  a.maxcol = nullptr;
  a.target = tgt;
  a.out = rout;
  a.err = err;
  if ((rc = launch_intra_jobs(ctx, groups, a, mem, true))) return rc;
  A.rewind(mark);   // (waited for)
  return SWX_OK;
}

// The CIGARs of a deferred traceback (TbDirect), whose total is known now.
static int finish_cigars(swx_ctx *ctx, int64_t np, const TbDirect &d, int64_t total,
                         const int32_t *cig_len, const int64_t *cig_off_final, const int32_t *qbeg,
                         const int32_t *qend, swx_batch_out *out, int *rc_range) {
  out->cigar_used = total;
  if (total > out->cigar_cap || (total > 0 && !out->cigar)) {
    *rc_range = SWX_ERANGE;
    g_last_error = "CIGAR arena too small";
    return SWX_OK;
  }
  if (out->out_mem == SWX_MEM_DEVICE || total == 0) return SWX_OK;
  if (total <= d.room) {
    memcpy(out->cigar, d.pin, sizeof(uint32_t) * (size_t)total);
    return SWX_OK;
  }
  uint32_t *tmp = ctx->arena.get<uint32_t>(total);   // more than the pinned memory holds
  if (!tmp) return fail(SWX_ENOMEM, "device pool exhausted");
  HIP_TRY(launch_cigar_compact(np, d.cscr, nullptr, cig_len, cig_off_final, nullptr, qbeg, qend, tmp,
                               d.max_q + d.max_r + 2, INT64_MAX, ctx->stream));
  HIP_TRY(hipMemcpyAsync(out->cigar, tmp, sizeof(uint32_t) * total, hipMemcpyDeviceToHost, ctx->stream));
  HIP_TRY(wait_stream(ctx->stream));
  return SWX_OK;
}

// the records' place: the caller's device memory, pinned memory, or (*copy) a
// device buffer that is copied at the end
static swx_rec_dev *out_records(swx_ctx *ctx, swx_rec *dst, uint32_t out_mem, int64_t np, bool *copy) {
  if (out_mem == SWX_MEM_DEVICE) return (swx_rec_dev *)dst;
  if (void *p = host_out(ctx, dst, (int64_t)sizeof(swx_rec) * np)) return (swx_rec_dev *)p;
  *copy = true;
  return ctx->arena.get<swx_rec_dev>(np);
}

static int run_pipeline(swx_ctx *ctx, const Scoring &sc, const DeviceBatch &b, uint32_t flags,
                        int32_t mask_len, swx_batch_out *out, const swx_profile *prof) {
  DevArena &A = ctx->arena;
  hipStream_t st = ctx->stream;
  const int64_t np = b.npairs;
  if (flags & SWX_SUBOPT) flags |= SWX_ALL;
  if (flags & (SWX_CIGAR | SWX_SCORE2)) flags |= SWX_BEGIN;
  int rc;
  HIP_TRY(hipEventRecord(ctx->ev[0], st));

  // per-pair arrays
  int64_t *qstart = A.get<int64_t>(np), *rstart = A.get<int64_t>(np), *rlen = A.get<int64_t>(np);
  int32_t *qlen = A.get<int32_t>(np);
  int32_t *score = A.get<int32_t>(np), *qend = A.get<int32_t>(np);
  int64_t *rend = A.get<int64_t>(np);
  uint8_t *ovf = A.get<uint8_t>(np), *lanebits = A.get<uint8_t>(np), *err = A.get<uint8_t>(np);
  int32_t *qbeg = A.get<int32_t>(np), *score2 = A.get<int32_t>(np);
  int64_t *rbeg = A.get<int64_t>(np), *rend2 = A.get<int64_t>(np);
  // [0 .. 4] the views' statistics, [5] long pairs, [6] validation flags,
  // [7] pairs that failed a consistency check
  int64_t *stats = A.get<int64_t>(8);
  LongPath lp;
  lp.is_long = A.get<uint8_t>(np);
  lp.is_short = A.get<uint8_t>(np);
  if (!qstart || !rstart || !rlen || !qlen || !score || !qend || !rend || !ovf || !lanebits ||
      !err || !qbeg || !score2 || !rbeg || !rend2 || !stats || !lp.is_long || !lp.is_short)
    return fail(SWX_ENOMEM, "device pool exhausted (pair arrays)");
  // Validation, views (clamped into the arrays whatever the input holds),
  // statistics and the split into long and short pairs with one read at the
  // end: nothing else runs before the input is known to be valid.  (Three
  // reads and eight small launches more took 0.1 ms of a batch of 500.)
  {
    FillSet fs{};
    fs.add(stats, 8, 8, 0);
    fs.add(err, np, 1, 0);
    fs.add(lanebits, np, 1, 16);
    HIP_TRY(fill_set(fs, st));
    ValidateArgs va{b.qcat, b.qcat_len, b.qoff, b.nq, b.rcat, b.rcat_len, b.roff, b.nr,
                    b.pair_q, b.pair_r, np, sc.n, (uint32_t *)(stats + 6)};
    HIP_TRY(launch_validate(va, st));
    if (b.nq >= 1 && b.nr >= 1) {   // (else every pair's index is out of range)
      const ViewCaps vc{b.nq, b.nr, b.qcat_len, b.rcat_len, INT32_MAX, 0, INT64_MAX};
      HIP_TRY(launch_views(np, b.qoff, b.roff, b.pair_q, b.pair_r, vc, qstart, qlen, rstart, rlen,
                           stats, st));
      HIP_TRY(split_long(np, qlen, rlen, ctx->long_cells, long_factor(ctx, np), ctx->long_rlen, stats,
                         lp.is_long, lp.is_short, stats + 5, st));
    }
  }
  int64_t hstats[8];
  if ((rc = read_i64(ctx, stats, hstats, 8))) return rc;
  const uint32_t bad = (uint32_t)hstats[6];
  if (bad & 1u) return fail(SWX_EINVAL, "offsets must be non-decreasing and within the code arrays");
  if (bad & 2u) return fail(SWX_EINVAL, "pair index out of range");
  if (bad & 12u) return fail(SWX_EINVAL, "symbol code outside [0, n)");
  ctx->max_q = hstats[2];
  ctx->max_r = hstats[3];
  ctx->mean_q = hstats[1] / std::max<int64_t>(hstats[4], 1);
  ctx->mean_r = hstats[4] / np;
  lp.nlong = hstats[5];
  lp.nshort = np - lp.nlong;
  // a score can reach smax * min(qlen, rlen); the 32-bit lanes hold < 2^26
  const int64_t score_bound = (int64_t)std::max(sc.smax, 0) * hstats[0];
  if (score_bound >= (1 << 26) - 1)
    return fail(SWX_EOVERFLOW, "a score could exceed the 32-bit lane range");
  PairView fview{qstart, rstart, qlen, rlen, b.qcat, b.rcat, 0};
  FillOut fout{score, qend, rend, ovf, err};

  // 24-row strips exist for the 4-symbol selector profile only
  const int R = (ctx->fill_rows == 24 && !sc.qsel) ? 32 : ctx->fill_rows;
  // every pair on one query (general alphabets): the query profile is built
  // once (or comes resident with the caller's profile) and every batched
  // pass reads it, instead of profile bytes per task
  SharedProf shp;
  const SharedProf *sp = nullptr;
  if (!sc.qsel && b.nq == 1) {
    if (prof && prof->dev) {
      shp.fwd = R == 32 ? prof->fwd32 : prof->fwd16;
      shp.fwd_row = R == 32 ? prof->qp32 : prof->qp16;
      shp.rev = prof->rev;
      shp.rev_row = prof->rev_row;
      shp.qlen = (int32_t)prof->query.size();
    } else {
      int64_t qo[2];
      if ((rc = read_i64(ctx, b.qoff, qo, 2))) return rc;
      const int64_t ql = qo[1] - qo[0];
      if (ql < 1 || ql > INT32_MAX / 4) return fail(SWX_EINVAL, "bad query length");
      shp.qlen = (int32_t)ql;
      shp.fwd_row = round_up(ql, R);
      shp.rev_row = qprof_rev_row(ql, 32);
      uint8_t *fw = A.get<uint8_t>((sc.n + 1) * shp.fwd_row);
      uint8_t *rv = A.get<uint8_t>(16 * (sc.n + 1) * shp.rev_row);
      if (!fw || !rv) return fail(SWX_ENOMEM, "device pool exhausted (query profile)");
      HIP_TRY(build_qprof(b.qcat + qo[0], shp.qlen, sc.dmat, sc.n, sc.bias, (int32_t)shp.fwd_row, fw,
                          shp.rev_row, rv, st));
      shp.fwd = fw;
      shp.rev = rv;
    }
    shp.R = R;
    sp = &shp;
  }

  // long pairs take the intra-sequence path, the rest the batched one
  AlonePath al;
  if ((rc = plan_alone(ctx, sc, np, flags, b.nq == 1, hstats, qlen, rlen, lp, al))) return rc;
  if (!al.on && (rc = list_pairs(ctx, np, lp))) return rc;
  AloneRest rest;
  if (al.all && (flags & SWX_BEGIN)) {
    rest.qbeg = qbeg;
    rest.rbeg = rbeg;
    rest.err = err;
    rest.mask_len = mask_len;
    if (flags & SWX_SCORE2) {
      rest.score2 = score2;
      rest.rend2 = rend2;
    }
  }
  auto long_forward = [&]() -> int {
    return al.on ? run_alone_forward(ctx, sc, al, score_bound, fview, fout, lanebits,
                                     al.label ? lp.is_long : nullptr, rest)
                 : run_intra_forward(ctx, sc, lp, fview, fout, err, lanebits);
  };

  // forward fill, 16-bit lanes (events 1 and 2 bracket the fill kernels)
  Plan p16, p32;
  if ((rc = plan_pass(ctx, sc, lp.d_short, lp.nshort, qlen, rlen, nullptr, nullptr, 16, R, p16, sp)))
    return rc;
  // With both kinds of pairs, the long pairs' pass runs on a side stream
  // beside the batched one (each ends on its own largest tasks, the other
  // fills the device meanwhile; the outputs are disjoint).
  const bool beside = lp.nlong > 0 && p16.ntasks > 0 && have_side_streams(ctx);
  if (beside) {
    HIP_TRY(hipEventRecord(ctx->fork_ev, st));
    HIP_TRY(hipStreamWaitEvent(ctx->aux[0], ctx->fork_ev, 0));
  }
  if ((rc = run_fill(ctx, p16, sc, fview, false, nullptr, fout, score_bound, 1, 0, 0, sp))) return rc;
  if (lp.nlong > 0) {
    if (beside) {
      {
        StreamScope on_side(ctx, ctx->aux[0]);   // the pass's launches and waits go there
        rc = long_forward();
      }
      if (rc) {   // nothing of the call may still run when it returns
        (void)hipStreamSynchronize(ctx->aux[0]);
        return rc;
      }
      HIP_TRY(hipEventRecord(ctx->join_ev[0], ctx->aux[0]));
      HIP_TRY(hipStreamWaitEvent(st, ctx->join_ev[0], 0));
    } else if ((rc = long_forward())) {
      return rc;
    }
    HIP_TRY(hipEventRecord(ctx->ev[2], st));
  }

  // saturated pairs: exact re-run on 32-bit lanes (none where no score of the
  // batch can reach the 16-bit limit, and none of the long pairs)
  int64_t *wide = nullptr, nwide = 0;
  if (lp.nshort > 0 && score_bound >= kInter16Limit &&
      (rc = select_flagged(ctx, ovf, np, &wide, &nwide)))
    return rc;
  if (nwide > 0) {
    if ((rc = plan_pass(ctx, sc, wide, nwide, qlen, rlen, nullptr, nullptr, 32, R, p32, sp))) return rc;
    if ((rc = run_fill(ctx, p32, sc, fview, false, nullptr, fout, score_bound, -1, 0, 0, sp))) return rc;
    HIP_TRY(mark_lanes(nwide, wide, lanebits, 32, st));
  }
  HIP_TRY(hipEventRecord(ctx->ev[3], st));

  // reversed pass: begin
  if ((flags & SWX_BEGIN) && !rest.qbeg) {
    int64_t *rqs = A.get<int64_t>(np), *rrs = A.get<int64_t>(np), *rrl = A.get<int64_t>(np);
    int32_t *rql = A.get<int32_t>(np), *tgt = A.get<int32_t>(np), *band = A.get<int32_t>(np);
    int32_t *band_q = A.get<int32_t>(np), *rsc = A.get<int32_t>(np), *rqe = A.get<int32_t>(np);
    int64_t *rre = A.get<int64_t>(np);
    uint8_t *rov = A.get<uint8_t>(np), *f16 = A.get<uint8_t>(np), *f32 = A.get<uint8_t>(np);
    if (!rqs || !rrs || !rrl || !rql || !tgt || !band || !band_q || !rsc || !rqe || !rre || !rov ||
        !f16 || !f32)
      return fail(SWX_ENOMEM, "device pool exhausted (reverse)");
    HIP_TRY(rev_setup(np, fview, score, qend, rend, lanebits, sc.smax, sc.o, sc.e,
                      RevSetup{rqs, rrs, rrl, rql, tgt, band, band_q, rsc, f16, f32}, err, st));
    if (lp.nlong > 0 && lp.nshort > 0) HIP_TRY(clear_flags(lp.nlong, lp.d_long, f16, f32, st));
    PairView rview{rqs, rrs, rql, rrl, b.qcat, b.rcat, 1};
    FillOut rout{rsc, rqe, rre, rov, err};
    // both lane widths' pair lists first, their counts in one read, so that
    // no read waits for a queued fill
    int64_t *rids[2] = {nullptr, nullptr}, rcnt[2] = {0, 0};
    const int64_t *rcd[2] = {nullptr, nullptr};
    int64_t *rc2 = A.get<int64_t>(2);
    if (!rc2) return fail(SWX_ENOMEM, "device pool exhausted (reverse counts)");
    // (without a pair above the 16-bit limit, the second list is empty)
    const int widths = lp.nshort == 0 ? 0 : score_bound >= kInter16Limit ? 2 : 1;
    for (int k = 0; k < widths; ++k) {
      if ((rc = select_flagged_dev(ctx, k == 0 ? f16 : f32, np, &rids[k], &rcd[k]))) return rc;
      HIP_TRY(hipMemcpyAsync(rc2 + k, rcd[k], sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    }
    if (widths > 0 && (rc = read_i64(ctx, rc2, rcnt, widths))) return rc;
    // as in the forward pass, the long pairs' reversed pass runs on a side
    // stream beside the batched one (16-bit lanes)
    const bool beside = lp.nlong > 0 && rcnt[0] > 0 && have_side_streams(ctx);
    bool long_done = false;
    auto long_reverse = [&]() -> int {
      if (!al.on) return run_intra_reverse(ctx, sc, lp, rview, score, qend, rend, band, tgt, rout, err);
      AloneArgs a = alone_args(sc, al, rview, rout);
      a.target = tgt;
      a.band = band;
      HIP_TRY(alone_reverse(a, ctx->stream));
      return SWX_OK;
    };
    for (int k = 0; k < 2; ++k) {
      if (rcnt[k] == 0) continue;
      Plan pr;
      if ((rc = plan_pass(ctx, sc, rids[k], rcnt[k], rql, rrl, band, band_q, k == 0 ? 16 : 32, R, pr,
                          sp)))
        return rc;
      if (k == 0 && beside) {
        HIP_TRY(hipEventRecord(ctx->fork_ev, st));
        HIP_TRY(hipStreamWaitEvent(ctx->aux[0], ctx->fork_ev, 0));
      }
      if ((rc = run_fill(ctx, pr, sc, rview, true, tgt, rout, score_bound, -1, 0, 0, sp))) return rc;
      if (k == 0 && beside) {
        {
          StreamScope on_side(ctx, ctx->aux[0]);
          rc = long_reverse();
        }
        if (rc) {   // nothing of the call may still run when it returns
          (void)hipStreamSynchronize(ctx->aux[0]);
          return rc;
        }
        HIP_TRY(hipEventRecord(ctx->join_ev[0], ctx->aux[0]));
        long_done = true;
      }
    }
    if (long_done) {
      HIP_TRY(hipStreamWaitEvent(st, ctx->join_ev[0], 0));
    } else if (lp.nlong > 0 && (rc = long_reverse())) {
      return rc;
    }
    HIP_TRY(launch_begins(np, score, qend, rend, rsc, rqe, rre, qbeg, rbeg, err, st));
  }
  HIP_TRY(hipEventRecord(ctx->ev[4], st));

  // banded traceback: CIGAR
  int64_t *cig_off_final = A.get<int64_t>(np + 1);
  int32_t *cig_len = A.get<int32_t>(np);
  if (!cig_off_final || !cig_len) return fail(SWX_ENOMEM, "device pool exhausted");
  int rc_range = SWX_OK;
  TbDirect direct{hstats[2], hstats[3],
                  round_up(tb_wave_dir_bytes(hstats[2], hstats[3], kTbPairRows), 256) +
                      tb_pair_bnd_bytes(hstats[2], hstats[3]),
                  (flags & SWX_SUBOPT) == 0, nullptr, nullptr, 0, nullptr};
  TbDirect *const tbd = al.all && np * direct.stride <= kTbGraphBytes ? &direct : nullptr;
  if (flags & SWX_CIGAR) {
    if ((rc = run_traceback(ctx, sc, b, np, hstats[0], tbd, score, qbeg, qend, rbeg, rend, qstart, rstart, qlen,
                            rlen, cig_len, cig_off_final, err, out, &flags, &rc_range)))
      return rc;
  } else {
    out->cigar_used = 0;
  }
  HIP_TRY(hipEventRecord(ctx->ev[5], st));

  // score2 from the max array (final CM plane of the forward tasks)
  if ((flags & SWX_SCORE2) && !rest.score2) {
    Score2InterArgs s2{};
    s2.rlen = rlen; s2.qlen = qlen; s2.score1 = score; s2.rbeg = rbeg; s2.rend = rend;
    s2.mask_len = mask_len; s2.score2 = score2; s2.rend2 = rend2;
    s2.tasks = p16.d_tasks; s2.ntasks = p16.ntasks; s2.slot_pair = p16.d_sorted;
    s2.bnd = p16.d_bnd; s2.halves = 2;
    HIP_TRY(launch_score2_inter(s2, st));
    if (p32.ntasks) {
      s2.tasks = p32.d_tasks; s2.ntasks = p32.ntasks; s2.slot_pair = p32.d_sorted;
      s2.bnd = p32.d_bnd; s2.halves = 1;
      HIP_TRY(launch_score2_inter(s2, st));
    }
    if (lp.nlong > 0) {
      IntraPairArgs e = alone_pairs(al, qlen, rlen);
      if (!al.on) {
        e.pairs = lp.d_pairs; e.maxcol = lp.d_maxcol;
        e.part_v = lp.d_part_v; e.part_j = lp.d_part_j; e.max_rlen = lp.max_rlen;
      }
      e.score = score; e.qend = qend; e.rend = rend; e.rbeg = rbeg;
      e.mask_len = mask_len; e.score2 = score2; e.rend2 = rend2;
      HIP_TRY(intra_score2(e, al.on ? al.count : lp.nlong, st));
    }
  }
  HIP_TRY(hipEventRecord(ctx->ev[6], st));

  // The suboptimal alignment behind score2: its end row (a forward pass over
  // a window of the reference ending at ref_end2, best taken in the last
  // column only), its begin (the reversed pass anchored at that end, on
  // 32-bit lanes offset by kAnchor so that only alignments starting at the
  // anchor cell can reach the target), its CIGAR (the banded traceback),
  // placed in the arena after every primary CIGAR.
  if (flags & SWX_SUBOPT) {
    // Where nothing was batched these passes take a wave per pair too, 32-bit
    // lanes as here, over every pair (those without a score2 have no columns):
    // no selection, plan, pack or read.  20,000 reads, 14,000 with a score2:
    // 2.07 + 1.60 ms for the two passes with their planning -> 0.46 + 0.36.
    const bool sub_alone = al.all && al.max_q < kAloneMaxQ;
    const uint32_t kAnchor = sub_alone ? kAloneAnchor : 1u << 25;
    if (score_bound >= (int64_t(1) << 24))
      return fail(SWX_EOVERFLOW, "scores too large for the suboptimal alignment's anchored pass");
    int64_t *wrs = A.get<int64_t>(np), *wrl = A.get<int64_t>(np), *wre = A.get<int64_t>(np);
    int32_t *wsc = A.get<int32_t>(np), *wqe = A.get<int32_t>(np);
    uint8_t *wov = A.get<uint8_t>(np), *sfl = A.get<uint8_t>(np), *slb = A.get<uint8_t>(np);
    int64_t *rqs = A.get<int64_t>(np), *rrs = A.get<int64_t>(np), *rrl = A.get<int64_t>(np);
    int32_t *rql = A.get<int32_t>(np), *tgt = A.get<int32_t>(np), *rsc = A.get<int32_t>(np);
    int32_t *rqe = A.get<int32_t>(np);
    int64_t *rre = A.get<int64_t>(np);
    uint8_t *rov = A.get<uint8_t>(np);
    int32_t *s_score = A.get<int32_t>(np), *s_qbeg = A.get<int32_t>(np), *s_qend = A.get<int32_t>(np);
    int64_t *s_rbeg = A.get<int64_t>(np), *s_rend = A.get<int64_t>(np);
    int32_t *s_cig_len = A.get<int32_t>(np);
    int64_t *s_cig_off = A.get<int64_t>(np + 1);
    if (!wrs || !wrl || !wre || !wsc || !wqe || !wov || !sfl || !slb || !rqs || !rrs || !rrl ||
        !rql || !tgt || !rsc || !rqe || !rre || !rov || !s_score || !s_qbeg || !s_qend ||
        !s_rbeg || !s_rend || !s_cig_len || !s_cig_off)
      return fail(SWX_ENOMEM, "device pool exhausted (suboptimal)");
    HIP_TRY(launch_sub_window(np, rstart, qlen, score2, rend2, sc.smax, sc.o, sc.e, wrs, wrl, sfl,
                              st));
    HIP_TRY(hipMemsetAsync(wsc, 0, sizeof(int32_t) * np, st));
    HIP_TRY(hipMemsetAsync(wqe, 0xFF, sizeof(int32_t) * np, st));
    int64_t *ids = nullptr, cnt = 0;
    if (sub_alone) {
      const PairView wview{qstart, wrs, qlen, wrl, b.qcat, b.rcat, 0};
      HIP_TRY(alone_last(alone_args(sc, al, wview, FillOut{wsc, wqe, wre, wov, err}), st));
    } else if ((rc = select_flagged(ctx, sfl, np, &ids, &cnt))) {
      return rc;
    }
    if (cnt > 0) {
      Plan pw;
      if ((rc = plan_pass(ctx, sc, ids, cnt, qlen, wrl, nullptr, nullptr, 32, R, pw, sp))) return rc;
      PairView wview{qstart, wrs, qlen, wrl, b.qcat, b.rcat, 0};
      FillOut wout{wsc, wqe, wre, wov, err};
      if ((rc = run_fill(ctx, pw, sc, wview, false, nullptr, wout, score_bound, -1, 0, 1, sp)))
        return rc;
    }
    HIP_TRY(launch_sub_rev_views(np, qstart, rstart, qlen, score2, rend2, wsc, wqe, kAnchor, rqs,
                                 rql, rrs, rrl, tgt, sfl, err, st));
    HIP_TRY(hipMemsetAsync(rsc, 0, sizeof(int32_t) * np, st));
    cnt = 0;
    if (sub_alone) {
      const PairView rview{rqs, rrs, rql, rrl, b.qcat, b.rcat, 1};
      AloneArgs a = alone_args(sc, al, rview, FillOut{rsc, rqe, rre, rov, err});
      a.target = tgt;
      a.anchor = kAnchor;
      a.max_q += 1;
      HIP_TRY(alone_reverse(a, st));
    } else if ((rc = select_flagged(ctx, sfl, np, &ids, &cnt))) {
      return rc;
    }
    if (cnt > 0) {
      Plan pr;
      if ((rc = plan_pass(ctx, sc, ids, cnt, rql, rrl, nullptr, nullptr, 32, R, pr, sp))) return rc;
      PairView rview{rqs, rrs, rql, rrl, b.qcat, b.rcat, 1};
      FillOut rout{rsc, rqe, rre, rov, err};
      if ((rc = run_fill(ctx, pr, sc, rview, true, tgt, rout, score_bound + kAnchor, -1, kAnchor,
                         0, sp)))
        return rc;
    }
    HIP_TRY(launch_sub_begins(np, score2, rend2, wqe, sfl, tgt, rsc, rqe, rre, s_score, s_qbeg,
                              s_qend, s_rbeg, s_rend, err, st));
    // CIGARs after the primaries (cigar_used holds their total even when they did not fit)
    const int64_t base = out->cigar_used;
    swx_batch_out so = *out;
    so.cigar = (out->cigar && base <= out->cigar_cap) ? out->cigar + base : nullptr;
    so.cigar_cap = out->cigar_cap > base ? out->cigar_cap - base : 0;
    uint32_t sflags = SWX_BEGIN | SWX_CIGAR;
    int rc_sub = SWX_OK;
    if ((rc = run_traceback(ctx, sc, b, np, hstats[0], tbd, s_score, s_qbeg, s_qend, s_rbeg, s_rend, qstart,
                            rstart, qlen, rlen, s_cig_len, s_cig_off, err, &so, &sflags, &rc_sub)))
      return rc;
    out->cigar_used = base + so.cigar_used;
    if (rc_sub != SWX_OK) rc_range = rc_sub;
    if (!(flags & SWX_CIGAR)) sflags &= ~SWX_CIGAR;   // the primaries did not fit either
    HIP_TRY(hipMemsetAsync(slb, 32, np, st));
    bool scopy = false;
    swx_rec_dev *srec = out_records(ctx, out->sub_recs, out->out_mem, np, &scopy);
    if (!srec) return fail(SWX_ENOMEM, "device pool exhausted");
    HIP_TRY(launch_records(np, s_score, s_score, s_qbeg, s_qend, s_rbeg, s_rend, s_rend, s_cig_off,
                           s_cig_len, slb, sflags, srec, nullptr, nullptr, INT64_MAX, st));
    if (sflags & SWX_CIGAR) HIP_TRY(shift_cigar_offsets(np, base, srec, st));
    if (scopy)
      HIP_TRY(hipMemcpyAsync(out->sub_recs, srec, sizeof(swx_rec) * np, hipMemcpyDeviceToHost, st));
  }

  // records
  bool rcopy = false;
  swx_rec_dev *drec = out_records(ctx, out->recs, out->out_mem, np, &rcopy);
  if (!drec) return fail(SWX_ENOMEM, "device pool exhausted");
  HIP_TRY(launch_records(np, score, score2, qbeg, qend, rbeg, rend, rend2, cig_off_final, cig_len,
                         lanebits, flags, drec, err, stats + 7,
                         direct.total ? (out->cigar ? out->cigar_cap : 0) : INT64_MAX, st));
  if (rcopy && np)
    HIP_TRY(hipMemcpyAsync(out->recs, drec, sizeof(swx_rec) * np, hipMemcpyDeviceToHost, st));
  HIP_TRY(hipEventRecord(ctx->ev[7], st));
  // consistency: any per-pair error flag
  int64_t nerr = 0;
  if (direct.total) {
    int64_t h[2];
    if ((rc = read_two(ctx, stats + 7, 1, direct.total, 1, h))) return rc;
    nerr = h[0];
    if ((rc = finish_cigars(ctx, np, direct, h[1], cig_len, cig_off_final, qbeg, qend, out, &rc_range)))
      return rc;
  } else if ((rc = read_i64(ctx, stats + 7, &nerr))) {
    return rc;
  }
  finish_outputs(ctx);
  ctx->nstages = 7;
  for (int k = 0; k < 7; ++k) {
    float ms = 0.f;
    hipError_t e = hipEventElapsedTime(&ms, ctx->ev[k], ctx->ev[k + 1]);
    if (e == hipErrorNotReady) {   // done on the device, not yet seen by the runtime
      HIP_TRY(hipEventSynchronize(ctx->ev[k + 1]));
      e = hipEventElapsedTime(&ms, ctx->ev[k], ctx->ev[k + 1]);
    }
    HIP_TRY(e);
    ctx->stage_ms[k] = ms;
  }
  if (nerr) return fail(SWX_EINTERNAL, "internal consistency check failed for " +
                                           std::to_string(nerr) + " pairs");
  return rc_range;
}

// ============================================================================
// Fixed-capacity path for hipGraph capture.
//
// The same stages as run_pipeline, for batches of exactly B pairs with
// qlen <= QM and rlen <= RM, with every buffer sized from those capacities
// when the graph is made and every count that depends on the data (pairs
// re-run on 32-bit lanes, pairs per reversed pass, pairs per traceback class)
// kept on the device: plans take their pair count from device memory and
// form empty tasks past it, kernels skip empty tasks.  Nothing in it waits on
// the host, so the whole chain is captured once and replayed per batch.
// Long pairs are not routed to the intra-sequence path here (its job tables
// are built on the host), and wide bands stay on the strip kernel.
// ============================================================================
struct FixedPlan {
  int lane_bits = 16, R = 32, slots = 128;
  int64_t cap_n = 0, ntasks = 0;
  uint64_t *k0 = nullptr, *k1 = nullptr;
  int64_t *v0 = nullptr, *v1 = nullptr;
  void *sort_tmp = nullptr;
  size_t sort_bytes = 0;
  int64_t *sorted = nullptr;
  InterTask *tasks = nullptr;
  int64_t *bsz = nullptr, *boff = nullptr, *qsz = nullptr, *qoff = nullptr;
  uint32_t *bnd = nullptr;
  uint2 *rsym = nullptr;
  uint8_t *prof = nullptr;
};

struct FixedTb {   // one traceback class
  int64_t cap_tasks = 0;
  void *tasks = nullptr;     // TbTask or TbwTask
  int64_t *dsz = nullptr, *doff = nullptr, *bsz = nullptr, *boff = nullptr;
  uint32_t *dir = nullptr;
  int32_t *bnd = nullptr;
};

struct GraphState {
  swx_graph_cfg cfg{};
  int32_t fill_sched = 1, cus = 0;    // the creating context's fill schedule
  int32_t fill_coop = 0;
  unsigned long long *queue = nullptr;
  std::vector<int8_t> matrix;
  Scoring sc{};
  DevArena A;
  int64_t B = 0, QM = 0, RM = 0;
  bool clamp = false, need32 = false, pair3 = false;
  // inputs / outputs
  int8_t *qcat = nullptr, *rcat = nullptr;
  int64_t *qoff = nullptr, *roff = nullptr, *pair_q = nullptr, *pair_r = nullptr;
  swx_rec_dev *recs = nullptr;
  uint32_t *cigar = nullptr;
  int64_t cigar_cap = 0;
  // per pair
  int64_t *qstart, *rstart, *rlen, *rend, *rbeg, *rend2, *rqs, *rrs, *rrl, *rre;
  int32_t *qlen, *score, *qend, *qbeg, *score2, *rql, *tgt, *band, *band_q, *rsc, *rqe, *cig_len;
  uint8_t *ovf, *lanebits, *err, *rov, *f16, *f32, *cls;
  uint32_t *bad;
  int64_t *status;            // [0] pairs with an error flag
  // compaction of flagged pairs
  int64_t *f64, *pos, *ids;
  void *scan_tmp = nullptr;
  size_t scan_bytes = 0;
  FixedPlan p16, p32, r16, r32;
  // traceback
  uint64_t *tk0, *tk1;
  int64_t *tv0, *tv1, *coff, *counts, *ranges, *len64, *cig_off_final;
  int64_t *tb_sorted = nullptr;
  void *tb_sort_tmp = nullptr;
  size_t tb_sort_bytes = 0;
  FixedTb tb[6];
  // graphs of up to kTbGraphPairs pairs: a workgroup per pair instead
  bool tb_by_pairs = false;
  int64_t tbp_stride = 0;
  uint8_t *tbp_scratch = nullptr;
  uint32_t *cscr = nullptr;
  // intra route: every pair spread over a wave (one job per pair)
  bool intra = false;
  int RL = 16, waves = 1;
  int32_t kbits = 1, sh = 1024;
  AlonePath alone;             // ... of short queries: no jobs
  int64_t bnd_stride = 0;      // reversed pass: hand-over rows per pair
  int32_t nc = 1;              // forward pass: column chunks per pair ...
  int64_t chunk = 0;           // ... of this many columns ...
  int64_t fbnd_stride = 0;     // ... and hand-over rows per chunk
  IntraJob *jobs = nullptr, *rjobs = nullptr;
  IntraPair *ipairs = nullptr;
  uint32_t *maxcol = nullptr, *ibnd = nullptr;
  int32_t *part_v = nullptr;
  int64_t *part_j = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

static int fixed_scan(GraphState &g, const int64_t *in, int64_t *out, int64_t n, hipStream_t st) {
  size_t need = 0;
  HIP_TRY(launch_exclusive_scan(in, out, n, nullptr, &need, st));
  if (need > g.scan_bytes) return fail(SWX_EINTERNAL, "scan scratch too small");
  size_t have = g.scan_bytes;
  HIP_TRY(launch_exclusive_scan(in, out, n, g.scan_tmp, &have, st));
  return SWX_OK;
}

// allocate a plan's buffers for up to cap_n pairs (create time)
static int fixed_plan_alloc(GraphState &g, FixedPlan &pl, int lane_bits, int R) {
  DevArena &A = g.A;
  pl.lane_bits = lane_bits;
  pl.R = R;
  pl.slots = lane_bits == 16 ? kSlots16 : kSlots32;
  pl.cap_n = g.B;
  pl.ntasks = (g.B + pl.slots - 1) / pl.slots;
  const int halves = lane_bits == 16 ? 2 : 1;
  pl.k0 = A.get<uint64_t>(g.B); pl.k1 = A.get<uint64_t>(g.B);
  pl.v0 = A.get<int64_t>(g.B); pl.v1 = A.get<int64_t>(g.B);
  pl.tasks = A.get<InterTask>(pl.ntasks);
  pl.bsz = A.get<int64_t>(pl.ntasks + 1); pl.boff = A.get<int64_t>(pl.ntasks + 1);
  pl.qsz = A.get<int64_t>(pl.ntasks + 1); pl.qoff = A.get<int64_t>(pl.ntasks + 1);
  const int64_t rp_cap = (g.RM + 7) / 8 * 8 + 8;
  const int64_t qp_cap = (g.QM + R - 1) / R * R + R;
  const int64_t bnd_words = pl.ntasks * 3 * 64 * rp_cap;
  pl.bnd = A.get<uint32_t>(bnd_words);
  pl.rsym = A.get<uint2>(rsym_offset(bnd_words) + 16);
  if (!g.sc.qsel) pl.prof = A.get<uint8_t>(pl.ntasks * qp_cap * (g.sc.n + 1) * halves * 64 + 16);
  size_t sb = 0;
  HIP_TRY(plan_sort(g.B, nullptr, nullptr, nullptr, nullptr, nullptr, R, 0, 0, pl.k0, pl.k1, pl.v0, pl.v1,
                    nullptr, &sb, nullptr, nullptr, true));
  pl.sort_bytes = sb;
  pl.sort_tmp = A.alloc(sb);
  if (!pl.k0 || !pl.k1 || !pl.v0 || !pl.v1 || !pl.tasks || !pl.bsz || !pl.boff || !pl.qsz ||
      !pl.qoff || !pl.bnd || !pl.rsym || (!g.sc.qsel && !pl.prof) || !pl.sort_tmp)
    return fail(SWX_ENOMEM, "device pool exhausted (graph plan)");
  return SWX_OK;
}

// plan + fill of one pass over ids[0 .. *n_dev) (ids null: all B pairs)
static int fixed_fill(GraphState &g, FixedPlan &pl, const int64_t *ids, const int64_t *n_dev,
                      const int32_t *qlen, const int64_t *rlen, const int32_t *band,
                      const int32_t *band_q, const PairView &view, bool rev,
                      const int32_t *target, FillOut out, hipStream_t st) {
  size_t sb = pl.sort_bytes;
  HIP_TRY(plan_sort(pl.cap_n, n_dev, ids, qlen, rlen, band, pl.R, 0, 0, pl.k0, pl.k1, pl.v0, pl.v1,
                    pl.sort_tmp, &sb, &pl.sorted, st, true));
  const int halves = pl.lane_bits == 16 ? 2 : 1;
  const int64_t per_row = g.sc.qsel ? 0 : (int64_t)(g.sc.n + 1) * halves * 64;
  HIP_TRY(plan_tasks_dev(   // also clears bsz[ntasks], qsz[ntasks]
                         pl.cap_n, n_dev, pl.ntasks, pl.slots, pl.R, per_row, pl.sorted, qlen, rlen,
                         band, band_q, pl.tasks, pl.bsz, pl.qsz, st));
  int rc;
  if ((rc = fixed_scan(g, pl.bsz, pl.boff, pl.ntasks + 1, st))) return rc;
  if ((rc = fixed_scan(g, pl.qsz, pl.qoff, pl.ntasks + 1, st))) return rc;
  HIP_TRY(plan_offsets_dev(pl.ntasks, pl.tasks, pl.boff, pl.qoff, st));
  PackArgs pk{};
  pk.tasks = pl.tasks; pk.ntasks = pl.ntasks; pk.slot_pair = pl.sorted; pk.view = view;
  pk.prof = pl.prof; pk.rsym = pl.rsym; pk.matrix = g.sc.dmat; pk.n = g.sc.n; pk.bias = g.sc.bias;
  pk.halves = halves; pk.strip_rows = pl.R; pk.rev = rev ? 1 : 0;
  HIP_TRY(inter_pack_ref(pk, st));
  if (!g.sc.qsel) HIP_TRY(inter_pack(pk, st));
  InterArgs a{};
  a.tasks = pl.tasks; a.ntasks = pl.ntasks; a.slot_pair = pl.sorted; a.view = view;
  a.prof = g.sc.qsel ? nullptr : pl.prof; a.bnd = pl.bnd; a.rsym = pl.rsym;
  for (int k = 0; k < 8; ++k) a.lut[k] = g.sc.lut[k];
  a.n = g.sc.n; a.o = g.sc.o; a.e = g.sc.e; a.bias = g.sc.bias;
  a.rev = rev ? 1 : 0;
  a.clamp = g.clamp ? 1 : 0;
  a.pair3 = g.pair3 ? 1 : 0;
  a.code_top = pl.R - 1;
  a.dummy = g.sc.dmat;
  a.target = target;
  a.out = out;
  a.sched = g.fill_sched;
  a.cus = g.cus;
  a.queue = g.queue;
  a.coop = coop_waves(g.fill_coop, pl.ntasks, g.cus);
  HIP_TRY(inter_fill(a, pl.lane_bits, pl.R, st));
  return SWX_OK;
}

// flagged pairs -> ids[0 .. *count) with the count on the device (pos[B])
static int fixed_select(GraphState &g, const uint8_t *flag, const int64_t **count, hipStream_t st) {
  HIP_TRY(flags_to_i64(g.B, flag, g.f64, st));   // also clears g.f64[B]
  int rc;
  if ((rc = fixed_scan(g, g.f64, g.pos, g.B + 1, st))) return rc;
  HIP_TRY(compact_flags(g.B, flag, g.pos, g.ids, st));
  *count = g.pos + g.B;
  return SWX_OK;
}

static int fixed_issue(GraphState &g, hipStream_t st) {
  const int64_t B = g.B;
  const uint32_t flags = g.cfg.flags & (SWX_CIGAR | SWX_SCORE2) ? (g.cfg.flags | SWX_BEGIN) : g.cfg.flags;
  int rc;
  if (g.intra) {
    // the intra route clears all its per-call buffers in one launch (the
    // lanes are 32-bit throughout)
    FillSet fs{};
    fs.add(g.bad, 2, 4, 0);
    fs.add(g.status, 1, 8, 0);
    fs.add(g.err, B, 1, 0);
    fs.add(g.lanebits, B, 1, 32);
    if (!g.alone.on) fs.add(g.maxcol, B * g.RM, 4, 0);
    fs.add(g.counts, 9, 8, 0);
    HIP_TRY(fill_set(fs, st));
  } else {
    HIP_TRY(fill_u8(8, (uint8_t *)g.bad, 0, st));
    HIP_TRY(fill_i64(1, g.status, 0, st));
    HIP_TRY(fill_u8(B, g.err, 0, st));
    HIP_TRY(fill_u8(B, g.lanebits, 16, st));
  }
  ValidateArgs va{g.qcat, g.cfg.qcat_cap, g.qoff, g.cfg.nq_cap, g.rcat, g.cfg.rcat_cap, g.roff,
                  g.cfg.nr_cap, g.pair_q, g.pair_r, B, g.sc.n, g.bad};
  HIP_TRY(launch_validate(va, st));
  {
    const ViewCaps vc{g.cfg.nq_cap, g.cfg.nr_cap, g.cfg.qcat_cap, g.cfg.rcat_cap,
                      (int32_t)g.QM, 0, g.RM};
    HIP_TRY(launch_views(B, g.qoff, g.roff, g.pair_q, g.pair_r, vc, g.qstart, g.qlen, g.rstart,
                         g.rlen, nullptr, st));
  }
  PairView fview{g.qstart, g.rstart, g.qlen, g.rlen, g.qcat, g.rcat, 0};
  FillOut fout{g.score, g.qend, g.rend, g.ovf, g.err};
  IntraArgs ia{};
  if (g.alone.on) {
    AloneArgs a = alone_args(g.sc, g.alone, fview, fout);
    AloneRest rest;
    rest.qbeg = g.qbeg;
    rest.rbeg = g.rbeg;
    rest.err = g.err;
    rest.mask_len = g.cfg.mask_len;
    if (flags & SWX_SCORE2) {
      rest.score2 = g.score2;
      rest.rend2 = g.rend2;
    }
    add_rest(a, g.sc, rest);
    if (flags & SWX_BEGIN) HIP_TRY(alone_pass(a, st));
    else HIP_TRY(alone_forward(a, st));
  } else if (g.intra) {
    HIP_TRY(intra_jobs_chunked(B, g.nc, g.chunk, g.qlen, g.rlen, g.sc.smax, g.sc.o, g.sc.e,
                               g.kbits, g.sh, g.RM, g.fbnd_stride, g.jobs, g.ipairs, st));
    ia.jobs = g.jobs; ia.njobs = B * g.nc; ia.view = fview; ia.matrix = g.sc.dmat;
    ia.n = g.sc.n; ia.o = g.sc.o; ia.e = g.sc.e; ia.bias = g.sc.bias;
    ia.maxcol = g.maxcol; ia.bnd = g.ibnd; ia.err = g.err;
    HIP_TRY(intra_fill(ia, g.RL, g.waves, false, st));
    IntraPairArgs e{};
    e.pairs = g.ipairs; e.maxcol = g.maxcol; e.qlen = g.qlen; e.rlen = g.rlen;
    e.score = g.score; e.qend = g.qend; e.rend = g.rend; e.overflow = g.ovf;
    e.part_v = g.part_v; e.part_j = g.part_j; e.max_rlen = g.RM;
    HIP_TRY(intra_end(e, B, st));
  } else if ((rc = fixed_fill(g, g.p16, nullptr, nullptr, g.qlen, g.rlen, nullptr, nullptr, fview, false,
                              nullptr, fout, st))) {
    return rc;
  }
  if (g.need32 && !g.intra) {
    const int64_t *nw = nullptr;
    if ((rc = fixed_select(g, g.ovf, &nw, st))) return rc;
    if ((rc = fixed_fill(g, g.p32, g.ids, nw, g.qlen, g.rlen, nullptr, nullptr, fview, false, nullptr,
                         fout, st)))
      return rc;
    HIP_TRY(mark_lanes_dev(B, nw, g.ids, g.lanebits, 32, st));
  }
  if ((flags & SWX_BEGIN) && !g.alone.on) {
    HIP_TRY(rev_setup(B, fview, g.score, g.qend, g.rend, g.lanebits, g.sc.smax, g.sc.o, g.sc.e,
                      RevSetup{g.rqs, g.rrs, g.rrl, g.rql, g.tgt, g.band, g.band_q, g.rsc, g.f16, g.f32},
                      g.err, st));
    PairView rview{g.rqs, g.rrs, g.rql, g.rrl, g.qcat, g.rcat, 1};
    FillOut rout{g.rsc, g.rqe, g.rre, g.rov, g.err};
    if (g.intra) {
      HIP_TRY(intra_rev_jobs_fixed(B, g.score, g.rend, g.band, g.kbits, g.bnd_stride, g.rjobs, st));
      IntraArgs ra = ia;
      ra.jobs = g.rjobs;
      ra.njobs = B;   // one reversed job per pair (the forward pass had g.nc per pair)
      ra.view = rview;
      ra.maxcol = nullptr;
      ra.target = g.tgt;
      ra.out = rout;
      HIP_TRY(intra_fill(ra, g.RL, g.waves, true, st));
    }
    const int64_t *n16 = nullptr;
    if (!g.intra && (rc = fixed_select(g, g.f16, &n16, st))) return rc;
    if (!g.intra && (rc = fixed_fill(g, g.r16, g.ids, n16, g.rql, g.rrl, g.band, g.band_q, rview,
                                     true, g.tgt, rout, st)))
      return rc;
    if (g.need32 && !g.intra) {
      const int64_t *n32 = nullptr;
      if ((rc = fixed_select(g, g.f32, &n32, st))) return rc;
      if ((rc = fixed_fill(g, g.r32, g.ids, n32, g.rql, g.rrl, g.band, g.band_q, rview, true,
                           g.tgt, rout, st)))
        return rc;
    }
    HIP_TRY(launch_begins(B, g.score, g.qend, g.rend, g.rsc, g.rqe, g.rre, g.qbeg, g.rbeg, g.err, st));
  }
  if (flags & SWX_CIGAR) {
    TbArgs ta{};
    ta.score = g.score; ta.qbeg = g.qbeg; ta.qend = g.qend; ta.rbeg = g.rbeg; ta.rend = g.rend;
    ta.qstart = g.qstart; ta.rstart = g.rstart; ta.qlen = g.qlen; ta.rlen = g.rlen;
    ta.qcat = g.qcat; ta.rcat = g.rcat; ta.matrix = g.sc.dmat;
    ta.n = g.sc.n; ta.o = g.sc.o; ta.e = g.sc.e; ta.smax = g.sc.smax;
    ta.cig_len = g.cig_len; ta.err = g.err;
    ta.wave_cells = INT64_MAX;   // no host-planned wave traceback in a graph
    ta.cig = g.cscr;
    ta.cig_stride = g.QM + g.RM + 2;
    if (!g.tb_by_pairs) {
      ta.cig_off = g.coff;
      if (!g.intra) HIP_TRY(fill_i64(9, g.counts, 0, st));
      HIP_TRY(tb_classify(ta, B, g.cls, g.tk0, g.tv0, g.coff, g.counts, g.counts + 8, nullptr, st));
    }
    if (g.tb_by_pairs) {
      TbPairs tp{};
      tp.stride = g.tbp_stride;
      tp.scratch = g.tbp_scratch;
      HIP_TRY(tb_pairs(ta, tp, B, std::min<int64_t>(g.QM, g.RM), st));
    } else {
    size_t sb = g.tb_sort_bytes;
    HIP_TRY(sort_keys(B, g.tk0, g.tk1, g.tv0, g.tv1, g.tb_sort_tmp, &sb, &g.tb_sorted, st, kTbKeyBits,
                      true));
    HIP_TRY(class_ranges(g.counts, g.ranges, st));
    for (int c = 1; c <= 3; ++c) {
      FixedTb &t = g.tb[c];
      const int32_t bw = 8 << (c - 1);
      TbTask *tasks = (TbTask *)t.tasks;
      HIP_TRY(fill_i64(1, t.dsz + t.cap_tasks, 0, st));
      HIP_TRY(tb_tasks_range(g.ranges + 2 * c, t.cap_tasks, g.tb_sorted, ta, bw, tasks, t.dsz, st));
      if ((rc = fixed_scan(g, t.dsz, t.doff, t.cap_tasks + 1, st))) return rc;
      HIP_TRY(tb_offsets(t.cap_tasks, tasks, t.doff, st));
      TbArgs tc = ta;
      tc.dir = t.dir;
      HIP_TRY(tb_band(tc, tasks, t.cap_tasks, g.tb_sorted, bw, st));
    }
    {
      FixedTb &t = g.tb[5];
      TbwTask *tasks = (TbwTask *)t.tasks;
      HIP_TRY(fill_i64(1, t.dsz + t.cap_tasks, 0, st));
      HIP_TRY(fill_i64(1, t.bsz + t.cap_tasks, 0, st));
      HIP_TRY(tbw_tasks_range(g.ranges + 10, t.cap_tasks, g.tb_sorted, ta, tasks, t.dsz, t.bsz, st));
      if ((rc = fixed_scan(g, t.dsz, t.doff, t.cap_tasks + 1, st))) return rc;
      if ((rc = fixed_scan(g, t.bsz, t.boff, t.cap_tasks + 1, st))) return rc;
      HIP_TRY(tbw_offsets(t.cap_tasks, tasks, t.doff, t.boff, st));
      TbArgs tc = ta;
      tc.dir = t.dir;
      HIP_TRY(tb_strip(tc, tasks, t.cap_tasks, g.tb_sorted, t.bnd, st));
    }
    }
    if (B <= kScanLensMax) {
      HIP_TRY(scan_lens(B, g.cig_len, g.cig_off_final, st));
    } else {
      HIP_TRY(fill_i64(1, g.len64 + B, 0, st));
      HIP_TRY(lens_to_i64(B, g.cig_len, g.len64, st));
      if ((rc = fixed_scan(g, g.len64, g.cig_off_final, B + 1, st))) return rc;
    }
    HIP_TRY(launch_cigar_compact(B, g.cscr, ta.cig_off, g.cig_len, g.cig_off_final,
                                 g.tb_by_pairs ? nullptr : g.cls, g.qbeg, g.qend, g.cigar,
                                 ta.cig_stride, INT64_MAX, st));
  }
  if ((flags & SWX_SCORE2) && g.alone.on) {
    // (with the forward pass)
  } else if ((flags & SWX_SCORE2) && g.intra) {
    IntraPairArgs e{};
    e.pairs = g.ipairs; e.maxcol = g.maxcol; e.qlen = g.qlen; e.rlen = g.rlen;
    e.part_v = g.part_v; e.part_j = g.part_j; e.max_rlen = g.RM;
    e.score = g.score; e.qend = g.qend; e.rend = g.rend; e.rbeg = g.rbeg;
    e.mask_len = g.cfg.mask_len; e.score2 = g.score2; e.rend2 = g.rend2;
    HIP_TRY(intra_score2(e, B, st));
  } else if (flags & SWX_SCORE2) {
    Score2InterArgs s2{};
    s2.rlen = g.rlen; s2.qlen = g.qlen; s2.score1 = g.score; s2.rbeg = g.rbeg; s2.rend = g.rend;
    s2.mask_len = g.cfg.mask_len; s2.score2 = g.score2; s2.rend2 = g.rend2;
    s2.tasks = g.p16.tasks; s2.ntasks = g.p16.ntasks; s2.slot_pair = g.p16.sorted;
    s2.bnd = g.p16.bnd; s2.halves = 2;
    HIP_TRY(launch_score2_inter(s2, st));
    if (g.need32) {
      s2.tasks = g.p32.tasks; s2.ntasks = g.p32.ntasks; s2.slot_pair = g.p32.sorted;
      s2.bnd = g.p32.bnd; s2.halves = 1;
      HIP_TRY(launch_score2_inter(s2, st));
    }
  }
  HIP_TRY(launch_records(B, g.score, g.score2, g.qbeg, g.qend, g.rbeg, g.rend, g.rend2,
                         g.cig_off_final, g.cig_len, g.lanebits, flags, g.recs, g.err, g.status,
                         INT64_MAX, st));
  return SWX_OK;
}

static int graph_alloc(GraphState &g) {
  DevArena &A = g.A;
  const int64_t B = g.B;
  g.queue = A.get<unsigned long long>(1);
  g.qcat = A.get<int8_t>(g.cfg.qcat_cap);
  g.rcat = A.get<int8_t>(g.cfg.rcat_cap);
  g.qoff = A.get<int64_t>(g.cfg.nq_cap + 1);
  g.roff = A.get<int64_t>(g.cfg.nr_cap + 1);
  g.pair_q = A.get<int64_t>(B);
  g.pair_r = A.get<int64_t>(B);
  g.recs = A.get<swx_rec_dev>(B);
  g.cigar_cap = B * (g.QM + g.RM + 2);
  g.cigar = A.get<uint32_t>(g.cigar_cap);
  g.cscr = A.get<uint32_t>(g.cigar_cap);
  bool per_pair = true;
  for (int64_t **p : {&g.qstart, &g.rstart, &g.rlen, &g.rend, &g.rbeg, &g.rend2, &g.rqs, &g.rrs,
                      &g.rrl, &g.rre, &g.tv0, &g.tv1})
    per_pair = (*p = A.get<int64_t>(B)) != nullptr && per_pair;
  for (int32_t **p : {&g.qlen, &g.score, &g.qend, &g.qbeg, &g.score2, &g.rql, &g.tgt, &g.band,
                      &g.band_q, &g.rsc, &g.rqe, &g.cig_len})
    per_pair = (*p = A.get<int32_t>(B)) != nullptr && per_pair;
  for (uint8_t **p : {&g.ovf, &g.lanebits, &g.err, &g.rov, &g.f16, &g.f32, &g.cls})
    per_pair = (*p = A.get<uint8_t>(B)) != nullptr && per_pair;
  if (!per_pair) return fail(SWX_ENOMEM, "device pool exhausted (graph)");
  g.bad = A.get<uint32_t>(2);   // (read as one 64-bit word)
  g.status = A.get<int64_t>(1);
  g.f64 = A.get<int64_t>(B + 1);
  g.pos = A.get<int64_t>(B + 1);
  g.ids = A.get<int64_t>(B);
  g.tk0 = A.get<uint64_t>(B);
  g.tk1 = A.get<uint64_t>(B);
  g.coff = A.get<int64_t>(B);
  g.counts = A.get<int64_t>(9);
  g.ranges = A.get<int64_t>(16);
  g.len64 = A.get<int64_t>(B + 1);
  g.cig_off_final = A.get<int64_t>(B + 1);
  int rc;
  const int R = 32;
  if (g.intra) {
    g.RL = pick_rl(g.QM, g.sc.n);
    g.sh = 64 * g.RL;
    const int64_t qp = (g.QM + g.sh - 1) / g.sh * g.sh;
    const int64_t nstrips = qp / g.sh;
    if (nstrips > intra_max_strips()) return fail(SWX_EINVAL, "max_qlen too long for the intra route");
    g.kbits = code_bits(qp);
    const int64_t bound = (int64_t)std::max(g.sc.smax, 0) * std::min<int64_t>(g.QM, g.RM);
    if (g.kbits > 30 || bound >= (int64_t(1) << (32 - g.kbits)))
      return fail(SWX_EOVERFLOW, "score range and query length exceed the max-array word");
    g.waves = intra_waves(nstrips, g.sc.n, g.RL);
    g.bnd_stride = 2 * (nstrips - 1) * g.RM;
    // the forward pass cuts each reference into column chunks that start the
    // widest positive-scoring span early (for the capacity's query length;
    // a shorter query starts later), so that a pair spreads over several
    // workgroups instead of sweeping its reference on one
    g.nc = 1;
    g.chunk = std::max<int64_t>(g.RM, 1);
    int64_t wcap = g.RM;
    if (g.sc.e > 0) {
      wcap = g.QM + std::max<int64_t>((int64_t)g.sc.smax * g.QM - g.sc.o, 0) / g.sc.e + 1;
      // (a one-pair graph is latency-bound: its chunks only need to fill a
      // few compute units, so it takes the most of them)
      const int64_t C = B == 1 ? 128 : std::max<int64_t>(256, (wcap + 1) / 2);
      const int64_t nc = std::min<int64_t>(kGraphMaxChunks, (g.RM + C - 1) / C);
      if (nc > 1) {
        g.nc = (int32_t)nc;
        g.chunk = (g.RM + nc - 1) / nc;
      }
    }
    // short queries: a wave per pair (as in plan_alone, for the capacities)
    g.alone.on = g.QM <= kAloneMaxQ && g.RM <= kAloneMaxR && g.RM >= 1 && bound + g.sc.bias <= 32766 &&
                 (g.RM <= kAloneSweep || B >= 16 * (int64_t)g.cus);
    g.fbnd_stride = 2 * (nstrips - 1) * std::min<int64_t>(g.RM, g.chunk + wcap);
    g.jobs = A.get<IntraJob>(B * g.nc);
    g.rjobs = A.get<IntraJob>(B);
    g.ipairs = A.get<IntraPair>(B);
    g.maxcol = A.get<uint32_t>(B * std::max<int64_t>(g.RM, 1));
    g.ibnd = A.get<uint32_t>(std::max<int64_t>(
        {B * g.bnd_stride, B * g.nc * g.fbnd_stride, int64_t(1)}));
    g.part_v = A.get<int32_t>(B * intra_slices());
    g.part_j = A.get<int64_t>(B * intra_slices());
    g.alone.count = g.alone.n32 = B;
    g.alone.maxcol = g.maxcol;
    g.alone.stride = g.RM;
    g.alone.max_q = (int32_t)g.QM;
    if (!g.jobs || !g.rjobs || !g.ipairs || !g.maxcol || !g.ibnd || !g.part_v || !g.part_j)
      return fail(SWX_ENOMEM, "device pool exhausted (graph intra route)");
  } else {
    if ((rc = fixed_plan_alloc(g, g.p16, 16, R))) return rc;
    if ((rc = fixed_plan_alloc(g, g.r16, 16, R))) return rc;
  }
  if (g.need32 && !g.intra) {
    if ((rc = fixed_plan_alloc(g, g.p32, 32, R))) return rc;
    if ((rc = fixed_plan_alloc(g, g.r32, 32, R))) return rc;
  }
  // traceback: a workgroup per pair where its fixed scratch stays small (and can
  // be had: for queries of less than 256 rows it is more than the classes'), else
  // the band classes, up to every pair in one class
  const int64_t tbp_stride = round_up(tb_wave_dir_bytes(g.QM, g.RM, kTbPairRows), 256) +
                             tb_pair_bnd_bytes(g.QM, g.RM);
  g.tb_by_pairs = B <= kTbGraphPairs && B * tbp_stride <= kTbGraphBytes &&
                  (g.QM + 64 * kTbPairRows - 1) / (64 * kTbPairRows) <= tb_wave_max_strips();
  if (g.tb_by_pairs) {
    g.tbp_stride = tbp_stride;
    g.tbp_scratch = A.get<uint8_t>(B * tbp_stride);
    g.tb_by_pairs = g.tbp_scratch != nullptr;
  }
  const int64_t capT = (B + 63) / 64;
  for (int c = 1; c <= 3 && !g.tb_by_pairs; ++c) {
    FixedTb &t = g.tb[c];
    t.cap_tasks = capT;
    t.tasks = A.get<TbTask>(capT);
    t.dsz = A.get<int64_t>(capT + 1);
    t.doff = A.get<int64_t>(capT + 1);
    t.dir = A.get<uint32_t>(capT * (g.QM + 2) * ((8 << (c - 1)) / 8) * 64);
    if (!t.tasks || !t.dsz || !t.doff || !t.dir) return fail(SWX_ENOMEM, "device pool exhausted (graph traceback)");
  }
  if (!g.tb_by_pairs) {
    FixedTb &t = g.tb[5];
    const int64_t capW = (B + kTbwSlots - 1) / kTbwSlots;
    t.cap_tasks = capW;
    t.tasks = A.get<TbwTask>(capW);
    t.dsz = A.get<int64_t>(capW + 1); t.doff = A.get<int64_t>(capW + 1);
    t.bsz = A.get<int64_t>(capW + 1); t.boff = A.get<int64_t>(capW + 1);
    // a safe band is at most m + w + 1 diagonals wide; the union over a task's
    // pairs at most 2 (m + w) + 1; a strip of width W holds (W + 4) / 2 code
    // dwords per lane
    const int64_t W = 16 + 2 * (g.QM + g.RM) + 2;
    const int64_t nstrips = (g.QM + 15) / 16;
    t.dir = A.get<uint32_t>(capW * nstrips * ((W + 4) / 2) * 64);
    t.bnd = A.get<int32_t>(capW * 2 * (g.RM + 1) * kTbwSlots);
    if (!t.tasks || !t.dsz || !t.doff || !t.bsz || !t.boff || !t.dir || !t.bnd)
      return fail(SWX_ENOMEM, "device pool exhausted (graph traceback)");
  }
  size_t sb = 0;
  HIP_TRY(sort_keys(B, g.tk0, g.tk1, g.tv0, g.tv1, nullptr, &sb, &g.tb_sorted, nullptr, kTbKeyBits,
                    true));
  g.tb_sort_bytes = sb;
  g.tb_sort_tmp = A.alloc(sb);
  // scan scratch: the largest scan is over B + 1 elements
  size_t sc1 = 0;
  HIP_TRY(launch_exclusive_scan(g.f64, g.pos, B + 1, nullptr, &sc1, nullptr));
  g.scan_bytes = sc1 + 4096;
  g.scan_tmp = A.alloc(g.scan_bytes);
  if (!g.qcat || !g.rcat || !g.qoff || !g.roff || !g.pair_q || !g.pair_r || !g.recs || !g.cigar ||
      !g.cscr || !g.bad || !g.status || !g.f64 || !g.pos || !g.ids || !g.tk0 || !g.tk1 ||
      !g.coff || !g.counts || !g.ranges || !g.len64 || !g.cig_off_final ||
      !g.tb_sort_tmp || !g.scan_tmp)
    return fail(SWX_ENOMEM, "device pool exhausted (graph)");
  return SWX_OK;
}

int internal_fail(int code, const char *msg) { return fail(code, msg); }
hipStream_t internal_stream(swx_ctx *ctx) { return ctx->stream; }
int internal_device(const swx_ctx *ctx) { return ctx->device; }
void internal_route_as(swx_ctx *ctx, int64_t n) {
  std::lock_guard<std::mutex> g(ctx->mu);
  ctx->route_pairs = n;
}

}  // namespace swx

using namespace swx;

// ============================================================================
// C ABI
// ============================================================================
extern "C" {

const char *swx_strerror(int status) {
  switch (status) {
    case SWX_OK: return "ok";
    case SWX_EINVAL: return "invalid argument";
    case SWX_ENOMEM: return "out of memory";
    case SWX_EDEVICE: return "device error";
    case SWX_EBUSY: return "busy";
    case SWX_EOVERFLOW: return "score range overflow";
    case SWX_ERANGE: return "output arena too small";
    case SWX_EINTERNAL: return "internal consistency check failed";
    default: return "unknown status";
  }
}

const char *swx_last_error(void) { return g_last_error.c_str(); }

int swx_get_tuning(const swx_ctx *ctx, swx_tuning *out) {
  if (!ctx || !out) return fail(SWX_EINVAL, "null argument");
  swx_tuning t{};
  t.long_cells = ctx->long_cells;
  t.long_rlen = ctx->long_rlen;
  t.intra_jobs = ctx->intra_jobs;
  t.fill_rows = ctx->fill_rows;
  t.side_streams = ctx->side_streams ? 1 : 0;
  t.fill_sched = ctx->fill_sched;
  t.fill_coop = ctx->fill_coop;
  t.intra_bits = ctx->intra_bits;
  *out = t;
  return SWX_OK;
}

int swx_set_tuning(swx_ctx *ctx, const swx_tuning *t) {
  if (!ctx || !t) return fail(SWX_EINVAL, "null argument");
  if (t->long_cells < -1 || t->long_rlen < 0 || t->intra_jobs < 1 ||
      (t->side_streams != 0 && t->side_streams != 1) || t->fill_sched < 0 || t->fill_sched > 2 ||
      t->fill_coop < 0 || t->fill_coop > 2 || (t->intra_bits != 0 && t->intra_bits != 16 && t->intra_bits != 32) ||
      t->pad_ != 0 ||
      (t->fill_rows != 16 && t->fill_rows != 24 && t->fill_rows != 32))
    return fail(SWX_EINVAL, "tuning value out of range");
  std::lock_guard<std::mutex> g(ctx->mu);
  ctx->long_cells = t->long_cells;
  ctx->long_rlen = t->long_rlen;
  ctx->intra_jobs = t->intra_jobs;
  ctx->fill_rows = t->fill_rows;
  ctx->side_streams = t->side_streams != 0;
  ctx->fill_sched = t->fill_sched;
  ctx->fill_coop = t->fill_coop;
  ctx->intra_bits = t->intra_bits;
  return SWX_OK;
}

// frees whatever a context holds (also one that was only partly created)
static void release_ctx(swx_ctx *ctx) {
  (void)hipSetDevice(ctx->device);
  ctx->arena.release();
  if (ctx->queue) (void)hipFree(ctx->queue);
  if (ctx->pinned) (void)hipHostFree(ctx->pinned);
  if (ctx->pair_in) (void)hipHostFree(ctx->pair_in);
  if (ctx->pair_out) (void)hipHostFree(ctx->pair_out);
  if (ctx->stage_in) (void)hipHostFree(ctx->stage_in);
  if (ctx->stage_out) (void)hipHostFree(ctx->stage_out);
  for (auto &e : ctx->ev)
    if (e) (void)hipEventDestroy(e);
  for (int k = 0; k < swx_ctx::kAux; ++k) {
    if (ctx->aux[k]) (void)hipStreamDestroy(ctx->aux[k]);
    if (ctx->join_ev[k]) (void)hipEventDestroy(ctx->join_ev[k]);
  }
  if (ctx->fork_ev) (void)hipEventDestroy(ctx->fork_ev);
  if (ctx->own) (void)hipStreamDestroy(ctx->own);
  delete ctx;
}

int swx_ctx_create(int device, swx_ctx **out) {
  if (!out) return fail(SWX_EINVAL, "out is null");
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0)
    return fail(SWX_EDEVICE, "no HIP device available");
  if (device < 0 || device >= ndev) return fail(SWX_EINVAL, "device ordinal out of range");
  swx_ctx *c = new (std::nothrow) swx_ctx();
  if (!c) return fail(SWX_ENOMEM, "host allocation failed");
  c->device = device;
  if (hipSetDevice(device) != hipSuccess || hipStreamCreate(&c->own) != hipSuccess) {
    release_ctx(c);
    return fail(SWX_EDEVICE, "could not create a stream");
  }
  c->stream = c->own;
  for (auto &e : c->ev) {
    if (hipEventCreate(&e) != hipSuccess) {
      release_ctx(c);
      return fail(SWX_EDEVICE, "could not create events");
    }
  }
  bool ok = hipEventCreateWithFlags(&c->fork_ev, hipEventDisableTiming) == hipSuccess;
  for (int k = 0; k < swx_ctx::kAux && ok; ++k)
    ok = hipEventCreateWithFlags(&c->join_ev[k], hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    release_ctx(c);
    return fail(SWX_EDEVICE, "could not create side streams");
  }
  if (hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
      c->cus < 1 || hipMalloc(&c->queue, 256) != hipSuccess ||
      hipHostMalloc(&c->pinned, 8 * (swx_ctx::kPinned + 8), hipHostMallocDefault) != hipSuccess) {
    release_ctx(c);
    return fail(SWX_EDEVICE, "could not query the device or allocate the work queue");
  }
  c->pinned_flag = (uint64_t *)(c->pinned + swx_ctx::kPinned);
  *c->pinned_flag = 0;
  c->scratch = scratch_address(device);
  if (!c->scratch) {
    release_ctx(c);
    return fail(SWX_EDEVICE, "could not find the device address of the static scratch");
  }
  *out = c;
  return SWX_OK;
}

int swx_ctx_destroy(swx_ctx *ctx) {
  if (!ctx) return fail(SWX_EINVAL, "ctx is null");
  {
    std::lock_guard<std::mutex> g(ctx->mu);
    (void)hipSetDevice(ctx->device);
    if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
    for (int k = 0; k < swx_ctx::kAux; ++k)
      if (ctx->aux[k]) (void)hipStreamSynchronize(ctx->aux[k]);
  }
  release_ctx(ctx);
  return SWX_OK;
}

int swx_last_stage_ms(const swx_ctx *ctx, double *ms, int cap) {
  if (!ctx || !ms || cap < 0) return fail(SWX_EINVAL, "bad arguments");
  int n = std::min(cap, ctx->nstages);
  for (int k = 0; k < n; ++k) ms[k] = ctx->stage_ms[k];
  return n;
}

int swx_lane_probe(swx_ctx *ctx, int32_t bits, int64_t columns, int64_t blocks, int32_t gap_open,
                   int32_t gap_extend, uint32_t *best, double *ms) {
  if (!ctx || !best || !ms) return fail(SWX_EINVAL, "null argument");
  if ((bits != 8 && bits != 16) || columns < 1 || blocks < 1 || blocks > (int64_t(1) << 20) ||
      gap_open < gap_extend || gap_extend < 0 || gap_open > 60)
    return fail(SWX_EINVAL, "bad probe arguments");
  std::lock_guard<std::mutex> g(ctx->mu);
  if (hipSetDevice(ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  ctx->arena.reset();
  const int64_t npairs = blocks * 256 * (32 / bits);
  uint32_t *d = ctx->arena.get<uint32_t>(npairs);
  if (!d) return fail(SWX_ENOMEM, "device pool exhausted (probe)");
  hipStream_t st = ctx->stream;
  HIP_TRY(hipEventRecord(ctx->ev[0], st));
  HIP_TRY(lane_probe(bits, columns, blocks, gap_open, gap_extend, d, st));
  HIP_TRY(hipEventRecord(ctx->ev[1], st));
  HIP_TRY(hipMemcpyAsync(best, d, sizeof(uint32_t) * (size_t)npairs, hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  float t = 0;
  HIP_TRY(hipEventElapsedTime(&t, ctx->ev[0], ctx->ev[1]));
  *ms = t;
  return SWX_OK;
}

int swx_check_max3(swx_ctx *ctx, uint64_t *mismatches, uint64_t *checked) {
  if (!ctx || !mismatches || !checked) return fail(SWX_EINVAL, "null argument");
  std::lock_guard<std::mutex> g(ctx->mu);
  if (hipSetDevice(ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  ctx->arena.reset();
  unsigned long long *d = ctx->arena.get<unsigned long long>(1);
  if (!d) return fail(SWX_ENOMEM, "device pool exhausted (check)");
  hipStream_t st = ctx->stream;
  HIP_TRY(hipMemsetAsync(d, 0, sizeof(*d), st));
  HIP_TRY(max3_check(d, checked, st));
  unsigned long long h = 0;
  HIP_TRY(hipMemcpyAsync(&h, d, sizeof(h), hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  *mismatches = h;
  return SWX_OK;
}

int swx_profile_create(swx_ctx *ctx, const int8_t *query, int32_t qlen, const int8_t *matrix,
                       int32_t n, int32_t gap_open, int32_t gap_extend, swx_profile **out) {
  if (!out) return fail(SWX_EINVAL, "out is null");
  *out = nullptr;
  if (!query || !matrix) return fail(SWX_EINVAL, "null query or matrix");
  if (qlen < 1) return fail(SWX_EINVAL, "qlen must be >= 1");
  Scoring sc;
  int rc = make_scoring(matrix, n, gap_open, gap_extend, &sc);
  if (rc) return rc;
  for (int32_t i = 0; i < qlen; ++i)
    if (query[i] < 0 || query[i] >= n) return fail(SWX_EINVAL, "query symbol outside [0, n)");
  if (!ctx) return fail(SWX_EINVAL, "ctx is null");
  swx_profile *p = new (std::nothrow) swx_profile();
  if (!p) return fail(SWX_ENOMEM, "host allocation failed");
  p->ctx = ctx;
  p->query.assign(query, query + qlen);
  p->matrix.assign(matrix, matrix + (size_t)n * n);
  p->n = n;
  p->o = gap_open;
  p->e = gap_extend;
  if (!sc.qsel) {
    // the query profile on the device, once: forward strips of 32 and of 16
    // rows and the reversed table (alphabets of at most 4 symbols need none:
    // their fill builds two scores per instruction from a 4-byte table)
    p->qp32 = (int32_t)round_up(qlen, 32);
    p->qp16 = (int32_t)round_up(qlen, 16);
    p->rev_row = qprof_rev_row(qlen, 32);
    const int64_t n1 = n + 1;
    const int64_t f32b = n1 * p->qp32, f16b = n1 * p->qp16, rb = 16 * n1 * p->rev_row;
    const int64_t scratch = qlen + (int64_t)n * n;
    std::lock_guard<std::mutex> g(ctx->mu);
    hipStream_t st = ctx->stream;
    bool ok = hipSetDevice(ctx->device) == hipSuccess &&
              hipMalloc(&p->dev, (size_t)(f32b + f16b + rb + scratch + 64)) == hipSuccess;
    if (ok) {
      p->fwd32 = p->dev;
      p->fwd16 = p->fwd32 + f32b;
      p->rev = p->fwd16 + f16b;
      int8_t *dq = (int8_t *)(p->rev + rb), *dm = dq + qlen;
      ok = hipMemcpyAsync(dq, query, qlen, hipMemcpyHostToDevice, st) == hipSuccess &&
           hipMemcpyAsync(dm, matrix, (size_t)n * n, hipMemcpyHostToDevice, st) == hipSuccess &&
           build_qprof(dq, qlen, dm, n, sc.bias, p->qp32, p->fwd32, p->rev_row, p->rev, st) ==
               hipSuccess &&
           build_qprof(dq, qlen, dm, n, sc.bias, p->qp16, p->fwd16, 0, p->rev, st) == hipSuccess &&
           hipStreamSynchronize(st) == hipSuccess;
    }
    if (!ok) {
      if (p->dev) (void)hipFree(p->dev);
      delete p;
      return fail(SWX_EDEVICE, "could not build the device query profile");
    }
  }
  *out = p;
  return SWX_OK;
}

int swx_profile_destroy(swx_profile *p) {
  if (!p) return fail(SWX_EINVAL, "profile is null");
  if (p->dev) {
    std::lock_guard<std::mutex> g(p->ctx->mu);
    (void)hipSetDevice(p->ctx->device);
    (void)hipStreamSynchronize(p->ctx->stream);
    (void)hipFree(p->dev);
  }
  delete p;
  return SWX_OK;
}

void swx_result_free(swx_result *r) {
  if (!r) return;
  free(r->cigar);
  free(r->sub_cigar);
  r->cigar = nullptr;
  r->sub_cigar = nullptr;
}

int64_t swx_cigar_bound(const swx_batch *b) {
  if (!b || b->in_mem != SWX_MEM_HOST || !b->qoff || !b->roff || !b->pair_q || !b->pair_r)
    return -1;
  int64_t s = 0;
  for (int64_t k = 0; k < b->npairs; ++k) {
    const int64_t qi = b->pair_q[k], ri = b->pair_r[k];
    if (qi < 0 || qi >= b->nq || ri < 0 || ri >= b->nr) return -1;
    s += (b->qoff[qi + 1] - b->qoff[qi]) + (b->roff[ri + 1] - b->roff[ri]) + 1;
  }
  return (b->flags & SWX_SUBOPT) ? 2 * s : s;
}

// dev_ref: the reference codes in device memory of a host-memory batch (whose
// rcat then only has to be non-null)
static int align_batch_locked(swx_ctx *ctx, const swx_batch *b, swx_batch_out *out,
                              const swx_profile *prof = nullptr, const int8_t *dev_ref = nullptr) {
  Scoring sc;
  int rc = make_scoring(b->matrix, b->n, b->gap_open, b->gap_extend, &sc);
  if (rc) return rc;
  if (b->npairs < 0 || b->nq < 0 || b->nr < 0 || b->qcat_len < 0 || b->rcat_len < 0)
    return fail(SWX_EINVAL, "negative count");
  if (!b->qoff || !b->roff || (b->npairs && (!b->pair_q || !b->pair_r)))
    return fail(SWX_EINVAL, "null offsets or pair arrays");
  if ((b->qcat_len && !b->qcat) || (b->rcat_len && !b->rcat))
    return fail(SWX_EINVAL, "null code arrays");
  if (!out || (b->npairs && !out->recs)) return fail(SWX_EINVAL, "null output");
  if (b->in_mem > 1 || out->out_mem > 1) return fail(SWX_EINVAL, "bad memory-space flag");
  if (b->flags & ~(SWX_ALL | SWX_SUBOPT)) return fail(SWX_EINVAL, "unknown flag bits");
  if ((b->flags & SWX_SUBOPT) && b->npairs && !out->sub_recs)
    return fail(SWX_EINVAL, "SWX_SUBOPT needs sub_recs");
  if (hipSetDevice(ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  ctx->arena.reset();
  DevArena &A = ctx->arena;
  hipStream_t st = ctx->stream;
  int8_t *dmat = A.get<int8_t>((int64_t)sc.n * sc.n);
  if (!dmat) return fail(SWX_ENOMEM, "device pool exhausted");
  sc.dmat = dmat;
  HostIn in[7];
  int nin = 0;
  in[nin++] = {dmat, b->matrix, (int64_t)sc.n * sc.n};
  ctx->out_used = 0;
  ctx->out_copies.clear();
  DeviceBatch db{};
  db.qcat_len = b->qcat_len; db.rcat_len = b->rcat_len; db.nq = b->nq; db.nr = b->nr;
  db.npairs = b->npairs;
  if (b->in_mem == SWX_MEM_DEVICE) {
    db.qcat = b->qcat; db.rcat = b->rcat; db.qoff = b->qoff; db.roff = b->roff;
    db.pair_q = b->pair_q; db.pair_r = b->pair_r;
  } else {
    int8_t *qc = A.get<int8_t>(b->qcat_len), *rc8 = dev_ref ? nullptr : A.get<int8_t>(b->rcat_len);
    int64_t *qo = A.get<int64_t>(b->nq + 1), *ro = A.get<int64_t>(b->nr + 1);
    int64_t *pq = A.get<int64_t>(b->npairs), *pr = A.get<int64_t>(b->npairs);
    if (!qc || (!rc8 && !dev_ref) || !qo || !ro || !pq || !pr) return fail(SWX_ENOMEM, "device pool exhausted");
    in[nin++] = {qc, b->qcat, b->qcat_len};
    if (!dev_ref) in[nin++] = {rc8, b->rcat, b->rcat_len};
    in[nin++] = {qo, b->qoff, 8 * (b->nq + 1)};
    in[nin++] = {ro, b->roff, 8 * (b->nr + 1)};
    in[nin++] = {pq, b->pair_q, 8 * b->npairs};
    in[nin++] = {pr, b->pair_r, 8 * b->npairs};
    db.qcat = qc; db.rcat = dev_ref ? dev_ref : rc8; db.qoff = qo; db.roff = ro; db.pair_q = pq; db.pair_r = pr;
  }
  if (b->npairs == 0) {
    out->cigar_used = 0;
    return SWX_OK;
  }
  rc = upload(ctx, in, nin);
  if (rc == SWX_OK) rc = run_pipeline(ctx, sc, db, b->flags, b->mask_len, out, prof);
  // a call that failed on its way leaves nothing running on the pinned buffers
  if (rc != SWX_OK && (ctx->stage_busy || !ctx->out_copies.empty())) {
    (void)hipStreamSynchronize(st);
    ctx->stage_busy = false;
    ctx->out_copies.clear();
  }
  return rc;
}

int swx_align_batch(swx_ctx *ctx, const swx_batch *b, swx_batch_out *out, void *hip_stream) {
  if (!ctx || !b || !out) return fail(SWX_EINVAL, "null argument");
  std::lock_guard<std::mutex> g(ctx->mu);
  StreamScope ss(ctx, hip_stream);
  return align_batch_locked(ctx, b, out);
}

int swx_align_batch_noalloc(swx_ctx *ctx, const swx_batch *b, swx_batch_out *out,
                            void *hip_stream) {
  if (!ctx || !b || !out) return fail(SWX_EINVAL, "null argument");
  if (b->npairs > SWX_NOALLOC_MAX_PAIRS)
    return fail(SWX_EINVAL, "batch above SWX_NOALLOC_MAX_PAIRS pairs");
  // host-memory inputs are staged in the scratch too
  if (b->in_mem == SWX_MEM_HOST) {
    const int64_t staged = b->qcat_len + b->rcat_len + 8 * (b->nq + b->nr + 2 + 2 * b->npairs);
    if (staged < 0 || staged > (int64_t)SWX_NOALLOC_SCRATCH_BYTES / 2)
      return fail(SWX_EINVAL, "inputs above half of the static scratch (SWX_NOALLOC_SCRATCH_BYTES)");
  }
  if (!ctx->scratch || ctx->device < 0 || ctx->device >= kMaxDevices)
    return fail(SWX_EDEVICE, "no static scratch on this device");
  std::lock_guard<std::mutex> dev(g_scratch_use[ctx->device]);
  std::lock_guard<std::mutex> g(ctx->mu);
  StreamScope ss(ctx, hip_stream);
  struct Restore {   // pool mode and side streams as they were, whatever happens
    swx_ctx *c;
    bool side;
    ~Restore() {
      c->arena.use_pool();
      c->side_streams = side;
    }
  } restore{ctx, ctx->side_streams};
  ctx->arena.use_fixed(ctx->scratch, SWX_NOALLOC_SCRATCH_BYTES);
  ctx->side_streams = false;   // making side streams would allocate
  int rc = align_batch_locked(ctx, b, out);
  const bool short_of_scratch = ctx->arena.fixed_exhausted();
  // the scratch is free for the next call only once this call's work is done
  if (wait_stream(ctx->stream) != hipSuccess && rc == SWX_OK)
    rc = fail(SWX_EDEVICE, "stream wait failed");
  if (rc == SWX_ENOMEM && short_of_scratch)
    rc = fail(SWX_ENOMEM, "the batch needs more device scratch than the static "
                          "SWX_NOALLOC_SCRATCH_BYTES; split it or use swx_align_batch");
  return rc;
}

// The one-pair call of short queries (kPairMaxQ x kPairMaxR) in three kernels.
// ref: host memory, or device memory with ref_dev.  Callers hold ctx->mu and a
// StreamScope.  1: memory for it could not be had (nothing has run).
static int align_pair_short(const swx_profile *p, const int8_t *ref, bool ref_dev, int64_t rlen,
                            uint32_t flags, int32_t mask_len, swx_result *out) {
  swx_ctx *ctx = p->ctx;
  if (hipSetDevice(ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  const int64_t Lq = (int64_t)p->query.size();
  Scoring sc;
  int rc = make_scoring(p->matrix.data(), p->n, p->o, p->e, &sc);
  if (rc) return rc;
  constexpr int64_t kInR = kPairMaxQ, kInM = kInR + kPairMaxR;   // offsets of the staged inputs
  if (!ctx->pair_in &&
      hipHostMalloc(&ctx->pair_in, kInM + 32 * 32, hipHostMallocDefault) != hipSuccess) {
    ctx->pair_in = nullptr;
    return 1;
  }
  if (!ctx->pair_out &&
      hipHostMalloc(&ctx->pair_out, sizeof(PairOut) + 4 * (kPairMaxQ + kPairMaxR + 2),
                    hipHostMallocDefault) != hipSuccess) {
    ctx->pair_out = nullptr;
    return 1;
  }
  if (ctx->pairs == 0) ctx->pair_out->done = 0;
  if (flags & (SWX_CIGAR | SWX_SCORE2)) flags |= SWX_BEGIN;
  PairArgs a{};
  a.Lq = (int32_t)Lq;
  a.Lr = rlen;
  a.n = sc.n; a.o = sc.o; a.e = sc.e; a.bias = sc.bias; a.smax = sc.smax;
  a.strips = (int32_t)((Lq + 64 * kPairRows - 1) / (64 * kPairRows));
  a.kb = code_bits((int64_t)a.strips * 64 * kPairRows);
  a.flags = flags;
  a.mask_len = mask_len;
  // column chunks, each on a workgroup of its own: as many as shorten the
  // longest sweep (a chunk and its warm-up, the widest positive-scoring span; by
  // less than 1/32 they are not worth their repeated columns), with at most 64 MiB
  // of several strips' words (2,048 x 65,536 DNA takes 48; 128 chunks of it took
  // 180 at scores of 11 with an extension of 1, and 459 at 30, where the warm-up
  // spans 97% of the reference)
  a.warm = intra_warmup(sc, Lq, rlen);
  a.chunk = std::max<int64_t>(rlen, 1);
  if (a.warm < rlen) {
    int64_t most = a.strips == 1 ? 256 : 128;
    if (a.strips > 1)
      most = std::min(most, std::max<int64_t>(((int64_t(8) << 20) / (a.strips - 1) - rlen) / a.warm, 1));
    const int64_t c = std::max<int64_t>(64, (rlen + most - 1) / most);
    if (32 * (c + a.warm) <= 31 * rlen) a.chunk = c;
  }
  ctx->arena.reset();
  DevArena &A = ctx->arena;
  a.rcount = (a.strips - 1) * rlen;
  a.q = A.get<int8_t>(Lq);
  a.r = A.get<int8_t>(rlen);
  a.m = A.get<int8_t>((int64_t)sc.n * sc.n);
  a.maxcol = A.get<uint32_t>(rlen);
  a.rwords = A.get<uint64_t>(a.rcount);
  a.state = A.get<PairState>(1);
  uint32_t *cig = A.get<uint32_t>(Lq + rlen + 2);
  bool have = a.q && a.r && a.m && a.maxcol && a.rwords && a.state && cig;
  if (flags & SWX_CIGAR) {
    // an alignment of positive score spans at most the warm-up's columns
    const int64_t w = std::min(rlen, a.warm);
    a.dir = A.get<uint8_t>(tb_wave_dir_bytes(Lq, w, kPairRows));
    a.bnd = A.get<int32_t>(2 * (w + 1) * (a.strips + 1));
    have = have && a.dir && a.bnd;
  }
  for (;;) {   // (one chunk where device memory is short)
    a.nchunks = (int32_t)((rlen + a.chunk - 1) / a.chunk);
    a.fstride = (a.strips - 1) * std::min(rlen, a.chunk + a.warm);
    a.fwords = A.get<uint64_t>(a.fstride * a.nchunks);
    if (a.fwords || a.nchunks == 1) break;
    a.chunk = rlen;
  }
  if (!have || !a.fwords) return 1;
  PairState *y = a.state;
  TbArgs &t = a.tb;
  t.score = &y->score; t.qbeg = &y->qbeg; t.qend = &y->qend; t.rbeg = &y->rbeg; t.rend = &y->rend;
  t.qstart = &y->qstart; t.rstart = &y->rstart; t.qlen = &y->qlen; t.rlen = &y->rlen;
  t.qcat = a.q; t.rcat = a.r; t.matrix = a.m;
  t.n = sc.n; t.o = sc.o; t.e = sc.e; t.smax = sc.smax;
  t.cig = cig; t.cig_off = &y->cig_off; t.cig_len = &y->cig_len; t.err = &y->err;
  memcpy(ctx->pair_in, p->query.data(), (size_t)Lq);
  if (!ref_dev) memcpy(ctx->pair_in + kInR, ref, (size_t)rlen);
  memcpy(ctx->pair_in + kInM, p->matrix.data(), (size_t)sc.n * sc.n);
  a.src_q = ctx->pair_in;
  a.src_r = ref_dev ? ref : ctx->pair_in + kInR;
  a.src_m = ctx->pair_in + kInM;
  a.out = ctx->pair_out;
  a.out->bad = a.out->err = 0;
  a.seq = ++ctx->pairs;   // (the word before the first call is 0)
  hipError_t he = pair_stage(a, ctx->stream);
  if (he == hipSuccess) he = pair_forward(a, ctx->stream);
  if (he == hipSuccess) he = pair_rest(a, ctx->stream);
  // (the pinned buffers are the next call's too)
  const hipError_t hw = he == hipSuccess ? wait_word(ctx->stream, &a.out->done, a.seq) : wait_stream(ctx->stream);
  if (he == hipSuccess) he = hw;
  if (he != hipSuccess) return fail(SWX_EDEVICE, std::string("one-pair call: ") + hipGetErrorString(he));
  if (a.out->bad) return fail(SWX_EINVAL, "symbol code outside [0, n)");
  if (a.out->err) return fail(SWX_EINTERNAL, "internal consistency check failed");
  memcpy(&out->rec, &a.out->rec, sizeof(swx_rec));
  if (out->rec.cigar_len > 0) {
    const size_t bytes = sizeof(uint32_t) * (size_t)out->rec.cigar_len;
    out->cigar = (uint32_t *)malloc(bytes);
    if (!out->cigar) {
      memset(out, 0, sizeof(*out));
      return fail(SWX_ENOMEM, "host allocation failed");
    }
    memcpy(out->cigar, a.out + 1, bytes);
  }
  return SWX_OK;
}

// Pairs of at most this size are always aligned on 32-bit long-pair lanes
// (the record's lane_bits), whatever the context's routing.
static constexpr int64_t kPair32MaxQ = 4096;

int swx_align(const swx_profile *p, const int8_t *ref, int64_t rlen, uint32_t flags,
              int32_t mask_len, void *hip_stream, swx_result *out) {
  if (!p || !out || (rlen > 0 && !ref)) return fail(SWX_EINVAL, "null argument");
  if (rlen < 0) return fail(SWX_EINVAL, "rlen must be >= 0");
  if (flags & ~(SWX_ALL | SWX_SUBOPT | SWX_REF_DEVICE)) return fail(SWX_EINVAL, "unknown flag bits");
  swx_ctx *ctx = p->ctx;
  memset(out, 0, sizeof(*out));
  const bool subopt = (flags & SWX_SUBOPT) != 0;
  if (subopt) flags |= SWX_ALL;
  bool ref_dev = (flags & SWX_REF_DEVICE) != 0 && rlen > 0;
  const int64_t Lq = (int64_t)p->query.size();
  std::lock_guard<std::mutex> g(ctx->mu);
  std::vector<int8_t> href;
  if (ref_dev) {
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
    // device memory of this GPU is read in place (a 5,000,000-column reference
    // took 1 ms to the host and back); anything else goes through a copy,
    // which also reports what cannot be read
    hipPointerAttribute_t at{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    const bool here = hipPointerGetAttributes(&at, ref) == hipSuccess &&
                      at.type == hipMemoryTypeDevice && at.device == ctx->device && !at.isManaged &&
                      hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)ref) == hipSuccess &&
                      (const int8_t *)base + size >= ref + rlen;
    if (!here) (void)hipGetLastError();
    // ordered after the caller's work: on its stream, or (none given) on the
    // default stream, where a copy of one byte waits as one of all would
    const size_t bytes = here ? 1 : (size_t)rlen;
    href.resize(bytes);
    if (!hip_stream) {
      if (hipMemcpy(href.data(), ref, bytes, hipMemcpyDeviceToHost) != hipSuccess)
        return fail(SWX_EDEVICE, "could not read the device reference");
    } else if (!here) {
      if (hipMemcpyAsync(href.data(), ref, bytes, hipMemcpyDeviceToHost, (hipStream_t)hip_stream) !=
              hipSuccess ||
          wait_stream((hipStream_t)hip_stream) != hipSuccess)
        return fail(SWX_EDEVICE, "could not read the device reference");
    }
    if (!here) {
      ref = href.data();
      ref_dev = false;
    }
  }
  StreamScope ss(ctx, hip_stream);
  const bool plain = !subopt && Lq <= kPair32MaxQ && rlen <= kPairMaxR;
  if (plain && Lq <= kPairMaxQ && rlen > 0) {
    const int rc = align_pair_short(p, ref, ref_dev, rlen, flags & SWX_ALL, mask_len, out);
    if (rc <= 0) return rc;
  }
  struct Routing {   // plain pairs: the 32-bit long-pair lanes
    swx_ctx *c;
    int64_t cells, len;
    int32_t bits;
    Routing(swx_ctx *c_, bool on) : c(c_), cells(c_->long_cells), len(c_->long_rlen), bits(c_->intra_bits) {
      if (on) {
        c->long_cells = 0;
        c->intra_bits = 32;
      }
    }
    ~Routing() {
      c->long_cells = cells;
      c->long_rlen = len;
      c->intra_bits = bits;
    }
  } routing(ctx, plain);
  const int64_t qoff[2] = {0, Lq};
  const int64_t roff[2] = {0, rlen};
  const int64_t pq = 0, pr = 0;
  swx_batch b{};
  b.matrix = p->matrix.data(); b.n = p->n; b.gap_open = p->o; b.gap_extend = p->e;
  b.qcat = p->query.data(); b.qcat_len = Lq; b.qoff = qoff; b.nq = 1;
  b.rcat = ref; b.rcat_len = rlen; b.roff = roff; b.nr = 1;
  b.pair_q = &pq; b.pair_r = &pr; b.npairs = 1;
  b.flags = flags & (SWX_ALL | SWX_SUBOPT); b.mask_len = mask_len; b.in_mem = SWX_MEM_HOST;
  swx_rec rec{}, sub{};
  Scoring sc;
  int rc = make_scoring(p->matrix.data(), p->n, p->o, p->e, &sc);
  if (rc) return rc;
  // an alignment spans at most the widest positive-scoring path's columns; the
  // suboptimal alignment's CIGAR goes to the same arena
  const int64_t cap = (subopt ? 2 : 1) * (Lq + std::min(rlen, intra_warmup(sc, Lq, rlen)) + 2);
  std::unique_ptr<uint32_t[]> cig(new (std::nothrow) uint32_t[(size_t)cap]);
  if (!cig) return fail(SWX_ENOMEM, "host allocation failed");
  swx_batch_out bo{&rec, cig.get(), cap, 0, SWX_MEM_HOST, 0, subopt ? &sub : nullptr};
  rc = align_batch_locked(ctx, &b, &bo, p, ref_dev ? ref : nullptr);
  if (rc) return rc;
  if (plain && rlen == 0) rec.lane_bits = 32;
  auto copy_out = [&](const swx_rec &r, swx_rec &dst, uint32_t *&dcig) {
    dst = r;
    dcig = nullptr;
    if (r.cigar_len > 0) {
      dcig = (uint32_t *)malloc(sizeof(uint32_t) * r.cigar_len);
      if (!dcig) return false;
      memcpy(dcig, cig.get() + r.cigar_off, sizeof(uint32_t) * r.cigar_len);
    }
    dst.cigar_off = 0;
    return true;
  };
  if (!copy_out(rec, out->rec, out->cigar) || (subopt && !copy_out(sub, out->sub, out->sub_cigar))) {
    swx_result_free(out);
    return fail(SWX_ENOMEM, "host allocation failed");
  }
  return SWX_OK;
}

}  // extern "C"

// ---- graph mode ---------------------------------------------------------------
struct swx_graph {
  swx_ctx *ctx = nullptr;
  swx::GraphState g;
};

extern "C" {

int swx_graph_create(swx_ctx *ctx, const swx_graph_cfg *cfg, swx_graph **out, swx_graph_io *io) {
  if (!ctx || !cfg || !out || !io) return fail(SWX_EINVAL, "null argument");
  *out = nullptr;
  if (cfg->max_pairs < 1 || cfg->max_qlen < 1 || cfg->max_rlen < 0 || cfg->qcat_cap < 0 ||
      cfg->rcat_cap < 0 || cfg->nq_cap < 1 || cfg->nr_cap < 1 || (cfg->flags & ~SWX_ALL))
    return fail(SWX_EINVAL, "bad graph capacities or flags");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (hipSetDevice(ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  swx_graph *gr = new (std::nothrow) swx_graph();
  if (!gr) return fail(SWX_ENOMEM, "host allocation failed");
  gr->ctx = ctx;
  GraphState &g = gr->g;
  g.cfg = *cfg;
  g.matrix.assign(cfg->matrix, cfg->matrix + (size_t)cfg->n * cfg->n);
  g.cfg.matrix = g.matrix.data();
  int rc = make_scoring(g.matrix.data(), cfg->n, cfg->gap_open, cfg->gap_extend, &g.sc);
  if (rc) { delete gr; return rc; }
  g.B = cfg->max_pairs;
  g.QM = cfg->max_qlen;
  g.RM = cfg->max_rlen;
  const int64_t bound = (int64_t)std::max(g.sc.smax, 0) * std::min<int64_t>(g.QM, g.RM);
  if (bound >= (1 << 26) - 1) { delete gr; return fail(SWX_EOVERFLOW, "scores could exceed the lane range"); }
  g.clamp = bound > kInter16Limit - 1;
  g.pair3 = bound <= kInter16PairLimit;
  g.need32 = bound >= kInter16Limit;
  g.intra = cfg->route == SWX_ROUTE_INTRA;
  g.fill_sched = ctx->fill_sched;
  g.fill_coop = ctx->fill_coop;
  g.cus = ctx->cus;
  int8_t *dmat = g.A.get<int8_t>((int64_t)g.sc.n * g.sc.n);
  if (!dmat) { delete gr; return fail(SWX_ENOMEM, "device pool exhausted"); }
  if (hipMemcpy(dmat, g.matrix.data(), (size_t)g.sc.n * g.sc.n, hipMemcpyHostToDevice) != hipSuccess) {
    delete gr;
    return fail(SWX_EDEVICE, "could not upload the matrix");
  }
  g.sc.dmat = dmat;
  if ((rc = graph_alloc(g))) { delete gr; return rc; }
  // valid empty contents: every code 0, every offset 0, every pair (0, 0); and no
  // results, for a read before the first run
  hipStream_t st = ctx->stream;
  bool ok = fill_u8(g.cfg.qcat_cap, (uint8_t *)g.qcat, 0, st) == hipSuccess &&
            fill_u8(g.cfg.rcat_cap, (uint8_t *)g.rcat, 0, st) == hipSuccess &&
            fill_i64(g.cfg.nq_cap + 1, g.qoff, 0, st) == hipSuccess &&
            fill_i64(g.cfg.nr_cap + 1, g.roff, 0, st) == hipSuccess &&
            fill_i64(g.B, g.pair_q, 0, st) == hipSuccess && fill_i64(g.B, g.pair_r, 0, st) == hipSuccess &&
            fill_u8(sizeof(swx_rec) * g.B, (uint8_t *)g.recs, 0, st) == hipSuccess &&
            fill_i64(g.B + 1, g.cig_off_final, 0, st) == hipSuccess &&
            hipStreamSynchronize(st) == hipSuccess;
  if (!ok) { delete gr; return fail(SWX_EDEVICE, "could not clear the graph buffers"); }
  // capture the whole chain once
  if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    delete gr;
    return fail(SWX_EDEVICE, "could not begin stream capture");
  }
  rc = fixed_issue(g, st);
  hipGraph_t graph = nullptr;
  const hipError_t ce = hipStreamEndCapture(st, &graph);
  if (rc != SWX_OK || ce != hipSuccess || !graph) {
    if (graph) hipGraphDestroy(graph);
    delete gr;
    return rc != SWX_OK ? rc : fail(SWX_EDEVICE, "stream capture failed");
  }
  g.graph = graph;
  if (hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0) != hipSuccess) {
    hipGraphDestroy(graph);
    delete gr;
    return fail(SWX_EDEVICE, "could not instantiate the graph");
  }
  io->qcat = g.qcat; io->qoff = g.qoff; io->rcat = g.rcat; io->roff = g.roff;
  io->pair_q = g.pair_q; io->pair_r = g.pair_r;
  io->recs = (swx_rec *)g.recs;
  io->cigar = g.cigar;
  io->cigar_cap = g.cigar_cap;
  *out = gr;
  return SWX_OK;
}

// waits for the stream and reads the run's flags; the caller holds ctx->mu
static int graph_check(swx_graph *gr) {
  GraphState &g = gr->g;
  swx_ctx *ctx = gr->ctx;
  int64_t h[2];
  if (read_two(ctx, (const int64_t *)g.bad, 1, g.status, 1, h) != SWX_OK)
    return fail(SWX_EDEVICE, "could not read the graph status");
  const uint32_t bad = (uint32_t)h[0];
  const int64_t nerr = h[1];
  if (bad & 1u) return fail(SWX_EINVAL, "offsets must be non-decreasing and within the code arrays");
  if (bad & 2u) return fail(SWX_EINVAL, "pair index out of range");
  if (bad & 12u) return fail(SWX_EINVAL, "symbol code outside [0, n)");
  if (nerr) return fail(SWX_EINTERNAL, "internal consistency check failed");
  return SWX_OK;
}

static int graph_run_on(swx_graph *gr, void *hip_stream) {
  std::lock_guard<std::mutex> lk(gr->ctx->mu);
  StreamScope ss(gr->ctx, hip_stream);
  if (hipSetDevice(gr->ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  HIP_TRY(hipGraphLaunch(gr->g.exec, gr->ctx->stream));
  return graph_check(gr);
}

int swx_graph_run(swx_graph *gr, void *hip_stream) {
  if (!gr) return fail(SWX_EINVAL, "null argument");
  return graph_run_on(gr, hip_stream);
}

int swx_graph_run_eager(swx_graph *gr, void *hip_stream) {
  if (!gr) return fail(SWX_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(gr->ctx->mu);
  StreamScope ss(gr->ctx, hip_stream);
  if (hipSetDevice(gr->ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  int rc = fixed_issue(gr->g, gr->ctx->stream);
  if (rc) return rc;
  return graph_check(gr);
}

int swx_graph_load(swx_graph *gr, const swx_batch *b) {
  if (!gr || !b) return fail(SWX_EINVAL, "null argument");
  GraphState &g = gr->g;
  if (b->in_mem != SWX_MEM_HOST) return fail(SWX_EINVAL, "swx_graph_load takes host memory");
  if (b->npairs < 0 || b->npairs > g.B || b->nq < 1 || b->nq > g.cfg.nq_cap ||
      b->nr < 0 || b->nr + 1 > g.cfg.nr_cap || b->qcat_len > g.cfg.qcat_cap ||
      b->rcat_len > g.cfg.rcat_cap || !b->qoff || !b->roff ||
      (b->npairs && (!b->pair_q || !b->pair_r)) || (b->qcat_len && !b->qcat) ||
      (b->rcat_len && !b->rcat))
    return fail(SWX_EINVAL, "batch does not fit the graph's capacities");
  // the host holds the whole batch here: offsets, pair indices and lengths
  // are checked before anything reaches the device
  for (int64_t k = 0; k < b->nq; ++k)
    if (b->qoff[k] < 0 || b->qoff[k] > b->qoff[k + 1] || b->qoff[k + 1] > b->qcat_len)
      return fail(SWX_EINVAL, "offsets must be non-decreasing and within the code arrays");
  for (int64_t k = 0; k < b->nr; ++k)
    if (b->roff[k] < 0 || b->roff[k] > b->roff[k + 1] || b->roff[k + 1] > b->rcat_len)
      return fail(SWX_EINVAL, "offsets must be non-decreasing and within the code arrays");
  for (int64_t k = 0; k < b->npairs; ++k) {
    const int64_t qi = b->pair_q[k], ri = b->pair_r[k];
    if (qi < 0 || qi >= b->nq || ri < 0 || ri >= b->nr)
      return fail(SWX_EINVAL, "pair index out of range");
    if (b->qoff[qi + 1] - b->qoff[qi] > g.QM || b->roff[ri + 1] - b->roff[ri] > g.RM)
      return fail(SWX_EINVAL, "a pair exceeds the graph's length capacities");
  }
  // symbols too: a rejected code must never reach the device buffers, where
  // it would outlive this load past the next, shorter one (every run checks
  // the whole code arrays)
  // (whole arrays without a branch per symbol: 275 KB of a 500-read batch
  // took 0.1 ms with one)
  auto symbols_ok = [&](const int8_t *s, int64_t len) {
    const unsigned n = (unsigned)g.sc.n;
    unsigned bad = 0;
    for (int64_t k = 0; k < len; ++k) bad |= (unsigned)((uint8_t)s[k] >= n);
    return bad == 0;
  };
  if (!symbols_ok(b->qcat, b->qcat_len) || !symbols_ok(b->rcat, b->rcat_len))
    return fail(SWX_EINVAL, "symbol code outside [0, n)");
  // offsets padded with their last value; pair slots past npairs take the
  // empty reference nr (roff[nr] == roff[nr + 1])
  std::vector<int64_t> qo(g.cfg.nq_cap + 1), ro(g.cfg.nr_cap + 1), pq(g.B, 0), pr(g.B, b->nr);
  for (int64_t k = 0; k <= g.cfg.nq_cap; ++k) qo[k] = b->qoff[std::min(k, b->nq)];
  for (int64_t k = 0; k <= g.cfg.nr_cap; ++k) ro[k] = b->roff[std::min(k, b->nr)];
  for (int64_t k = 0; k < b->npairs; ++k) { pq[k] = b->pair_q[k]; pr[k] = b->pair_r[k]; }
  std::lock_guard<std::mutex> lk(gr->ctx->mu);
  const HostIn in[6] = {{g.qcat, b->qcat, b->qcat_len},
                        {g.rcat, b->rcat, b->rcat_len},
                        {g.qoff, qo.data(), 8 * (int64_t)qo.size()},
                        {g.roff, ro.data(), 8 * (int64_t)ro.size()},
                        {g.pair_q, pq.data(), 8 * (int64_t)pq.size()},
                        {g.pair_r, pr.data(), 8 * (int64_t)pr.size()}};
  int rc;
  if (hipSetDevice(gr->ctx->device) != hipSuccess) return fail(SWX_EDEVICE, "hipSetDevice failed");
  if ((rc = upload(gr->ctx, in, 6))) return rc;
  // the host vectors must outlive the copies, and a run may be on another stream
  HIP_TRY(wait_stream(gr->ctx->stream));
  gr->ctx->stage_busy = false;
  return SWX_OK;
}

int swx_graph_read(swx_graph *gr, int64_t npairs, swx_batch_out *out) {
  if (!gr || !out || npairs < 0 || npairs > gr->g.B || (npairs && !out->recs))
    return fail(SWX_EINVAL, "bad arguments");
  GraphState &g = gr->g;
  std::lock_guard<std::mutex> lk(gr->ctx->mu);
  if (npairs == 0) { out->cigar_used = 0; return SWX_OK; }
  swx_ctx *ctx = gr->ctx;
  // small results in one kernel, through pinned memory: the records, then the
  // CIGAR words as far as there is room
  const int64_t head = round_up((int64_t)sizeof(swx_rec) * npairs, 256) + 256;
  const bool cigars = (g.cfg.flags & SWX_CIGAR) != 0;
  if (head < swx_ctx::kStage / 2 &&
      (ctx->stage_out || hipHostMalloc(&ctx->stage_out, swx_ctx::kStage, hipHostMallocDefault) == hipSuccess)) {
    int64_t *total = (int64_t *)ctx->stage_out;
    swx_rec_dev *hrecs = (swx_rec_dev *)(ctx->stage_out + 256);
    uint32_t *hcig = (uint32_t *)(ctx->stage_out + head);
    const int64_t room = std::min<int64_t>((swx_ctx::kStage - head) / 4, g.cigar_cap);
    HIP_TRY(hipSetDevice(ctx->device));
    HIP_TRY(graph_out(npairs, g.recs, g.cigar, cigars ? g.cig_off_final : nullptr, room, hrecs, hcig,
                      total, ctx->stream));
    HIP_TRY(wait_stream(ctx->stream));
    memcpy(out->recs, hrecs, sizeof(swx_rec) * (size_t)npairs);
    const int64_t used = *total;
    out->cigar_used = used;
    if (used > out->cigar_cap || (used && !out->cigar)) return fail(SWX_ERANGE, "CIGAR arena too small");
    if (used > room) HIP_TRY(hipMemcpy(out->cigar, g.cigar, sizeof(uint32_t) * used, hipMemcpyDeviceToHost));
    else if (used) memcpy(out->cigar, hcig, sizeof(uint32_t) * (size_t)used);
    return SWX_OK;
  }
  if (head < swx_ctx::kStage / 2) ctx->stage_out = nullptr;   // (no pinned memory to be had)
  HIP_TRY(hipMemcpy(out->recs, g.recs, sizeof(swx_rec) * npairs, hipMemcpyDeviceToHost));
  int64_t used = 0;
  for (int64_t k = 0; k < npairs; ++k)
    used = std::max<int64_t>(used, out->recs[k].cigar_off + out->recs[k].cigar_len);
  out->cigar_used = used;
  if (used > out->cigar_cap || (used && !out->cigar)) return fail(SWX_ERANGE, "CIGAR arena too small");
  if (used) HIP_TRY(hipMemcpy(out->cigar, g.cigar, sizeof(uint32_t) * used, hipMemcpyDeviceToHost));
  return SWX_OK;
}

int swx_graph_destroy(swx_graph *gr) {
  if (!gr) return fail(SWX_EINVAL, "null argument");
  {
    std::lock_guard<std::mutex> lk(gr->ctx->mu);
    (void)hipSetDevice(gr->ctx->device);
    (void)hipStreamSynchronize(gr->ctx->stream);
    if (gr->g.exec) (void)hipGraphExecDestroy(gr->g.exec);
    if (gr->g.graph) (void)hipGraphDestroy(gr->g.graph);
    gr->g.A.release();
  }
  delete gr;
  return SWX_OK;
}

}  // extern "C"
