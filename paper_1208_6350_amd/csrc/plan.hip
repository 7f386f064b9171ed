// plan.hip -- device-side batching: length-bucketed task formation.
//
// Pairs of one pass are sorted by a key (band class, padded query height,
// reference length) with a device radix sort and cut into tasks of `slots`
// consecutive pairs, so that the pairs sharing a wave have nearly the same
// dimensions and little padding.  Task sizes and buffer offsets are derived on
// the device; the host only reads back the totals it must allocate.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <rocprim/device/device_radix_sort.hpp>

#include "swx_internal.h"
#include "swx_kernels.h"

namespace swx {

// The key's fields from the lowest: reference length, half-strip count of the
// query, band class.  Their widths cover the batch's longest sequences and no
// more: a pass of the sort per 8 bits is 40 us for 2,000,000 pairs, and two
// clears with their launches (44 and 64 bits as fixed fields: 14 passes for
// both fills of 70 x 70 overlaps, now 5).
struct PlanBits { int r, q, b; };
static int bits_of(int64_t v) {
  int k = 1;
  while (k < 62 && (int64_t(1) << k) <= v) ++k;
  return k;
}
// max_q, max_r: no pair of the pass is longer (0: not known)
static PlanBits plan_bits(int64_t max_q, int64_t max_r, int32_t R, bool band) {
  PlanBits w{28, 16, band ? 20 : 0};
  if (max_q > 0 || max_r > 0) {
    w.r = std::min(w.r, bits_of(max_r));
    w.q = std::min(w.q, bits_of((std::max<int64_t>(max_q, 1) + R / 2 - 1) / (R / 2)));
    if (band) w.b = std::min(w.b, bits_of(max_r / 2 + 3));   // (a banded class is below rlen / 2)
  }
  return w;
}

// n_dev (may be null): the number of valid ids, read on the device; entries
// beyond it get the largest key (they sort last and form empty tasks)
__global__ void k_plan_keys(int64_t n, const int64_t *n_dev, const int64_t *ids, const int32_t *qlen,
                            const int64_t *rlen, const int32_t *band, int32_t R, PlanBits w,
                            uint64_t *keys, int64_t *vals) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  if (n_dev && k >= *n_dev) {
    keys[k] = ~0ull;
    vals[k] = -1;
    return;
  }
  const int64_t p = ids ? ids[k] : k;
  int64_t q = qlen[p];
  if (q < 1) q = 1;
  const uint64_t qc = (uint64_t)((q + R / 2 - 1) / (R / 2));   // half-strip buckets
  auto top = [](int k) { return (uint64_t(1) << k) - 1; };
  uint64_t r = (uint64_t)rlen[p];
  if (r > top(w.r)) r = top(w.r);
  // band class: the band half-width, except that pairs whose band spans
  // nearly the whole reference (2 * band + R >= rlen: a strip's window then
  // leaves out few columns) are grouped by size alone, after the banded ones,
  // and unbanded pairs come last
  uint64_t b = 0;
  if (band) {
    if (band[p] < 0) b = top(w.b);
    else if (2 * (int64_t)band[p] + R >= (int64_t)rlen[p]) b = top(w.b) - 1;
    else b = (uint64_t)band[p] > top(w.b) - 2 ? top(w.b) - 2 : (uint64_t)band[p];
  }
  keys[k] = (b << (w.q + w.r)) | ((qc > top(w.q) ? top(w.q) : qc) << w.r) | r;
  vals[k] = p;
}

__device__ __forceinline__ int64_t wave_max_i64(int64_t v) {
  for (int off = 32; off >= 1; off >>= 1) {
    const int64_t o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return v;
}

// one wave per task: the lanes take the task's slots in turn, and the
// maxima are reduced across the wave
__global__ void k_plan_tasks(int64_t n, const int64_t *n_dev, int64_t ntasks, int32_t slots,
                             int32_t R, int64_t qdata_per_row, const int64_t *sorted,
                             const int32_t *qlen, const int64_t *rlen, const int32_t *band,
                             const int32_t *band_q, InterTask *tasks, int64_t *bnd_size,
                             int64_t *qdata_size) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (t >= ntasks) return;
  if (n_dev) n = *n_dev;
  const int64_t s0 = t * slots;
  int64_t s1 = (s0 + slots < n) ? s0 + slots : n;
  if (s1 < s0) s1 = s0;   // a task past the valid ids is empty
  // mb, mbq: a negative band (none) counts as the largest
  int64_t mq = 1, mr = 1, mb = 0, mbq = 0;
  for (int64_t k = s0 + lane; k < s1; k += 64) {
    const int64_t p = sorted[k];
    if (qlen[p] > mq) mq = qlen[p];
    if (rlen[p] > mr) mr = rlen[p];
    if (band) {
      const int64_t b = band[p] < 0 ? INT64_MAX : band[p];
      mb = b > mb ? b : mb;
      const int64_t bq = band_q ? (band_q[p] < 0 ? INT64_MAX : band_q[p]) : b;
      mbq = bq > mbq ? bq : mbq;
    }
  }
  mq = wave_max_i64(mq);
  mr = wave_max_i64(mr);
  mb = wave_max_i64(mb);
  mbq = wave_max_i64(mbq);
  if (lane != 0) return;
  if (t == 0) {   // the totals' slots of the two scans
    bnd_size[ntasks] = 0;
    qdata_size[ntasks] = 0;
  }
  InterTask tk{};
  tk.nslots = (int32_t)(s1 - s0);
  // without a query profile the last strip may be half high: rows are
  // padded to a multiple of R / 2 (an odd multiple leaves a half strip last)
  const int64_t unit = qdata_per_row == 0 ? R / 2 : R;
  tk.qp = (int32_t)((mq + unit - 1) / unit * unit);
  tk.rp = (int32_t)((mr + 7) / 8 * 8);
  tk.band = band ? (mb == INT64_MAX ? -1 : (int32_t)mb) : -1;
  tk.band_q = (band && mbq != INT64_MAX && tk.band >= 0) ? (int32_t)mbq : tk.band;
  tk.slot_base = s0;
  tasks[t] = tk;
  bnd_size[t] = 3 * (int64_t)tk.rp * 64;
  // qdata_per_row < 0: a profile shared by every task (whole strips, no bytes per task)
  qdata_size[t] = qdata_per_row > 0 ? ((int64_t)tk.qp * qdata_per_row + 15) / 16 * 16 : 0;
}

__global__ void k_plan_offsets(int64_t ntasks, InterTask *tasks, const int64_t *bnd_off,
                               const int64_t *qdata_off) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ntasks) return;
  tasks[t].bnd_off = bnd_off[t];
  tasks[t].qdata_off = qdata_off[t];
}

// flagged compaction: out[k] = the k-th pair with flag != 0 (in pair order)
// f64[0 .. n) = flags as 0/1 and f64[n] = 0 (the total's slot of the scan)
__global__ void k_flag_to_i64(int64_t n, const uint8_t *flag, int64_t *f64) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) f64[p] = flag[p] ? 1 : 0;
  else if (p == n) f64[n] = 0;
}

__global__ void k_compact(int64_t n, const uint8_t *flag, const int64_t *pos, int64_t *out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n && flag[p]) out[pos[p]] = p;
}

// The reversed pass's setup: the band per pair (rev_band), its views (prefixes q[0..qend] and r[0..rend],
// read backwards by the fill), its target, its score preset to none and flags
// by lane width (f16, f32: may be null).
__global__ void k_rev_setup(int64_t n, PairView v, const int32_t *score, const int32_t *qend,
                            const int64_t *rend, const uint8_t *lanebits, int32_t smax, int32_t o,
                            int32_t e, RevSetup s, uint8_t *err) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  bool ok = score[p] > 0;
  const int64_t rows = (int64_t)qend[p] + 1, cols = rend[p] + 1;
  int32_t b = 0, bq = 0;
  if (ok) rev_band(score[p], rows, cols, smax, o, e, b, bq);
  s.band[p] = b;
  s.band_q[p] = bq;
  if (s.f16) {
    s.f16[p] = (ok && lanebits[p] == 16) ? 1 : 0;
    s.f32[p] = (ok && lanebits[p] == 32) ? 1 : 0;
  }
  if (ok && (rows < 1 || rows > v.qlen[p] || cols < 1 || cols > v.rlen[p])) {
    err[p] = 1;   // an end outside the pair: never read past the sequences
    ok = false;
  }
  s.qstart[p] = v.qstart[p];
  s.rstart[p] = v.rstart[p];
  s.qlen[p] = ok ? (int32_t)rows : 0;
  s.rlen[p] = ok ? cols : 0;
  s.target[p] = ok ? score[p] : 0;
  s.score[p] = 0;
}

static inline unsigned nb(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// Eager sorts go by digit passes (onesweep) at every size: rocprim's default
// sorts up to 2^20 items by block sorts and about ten merge passes instead,
// which took ~0.2 ms per sort of 10^6 pairs (two kernels per merge pass).
// Both are stable, so the order is the same.  Sorts recorded into a graph
// take the merge form at every size: onesweep clears its lookback states with
// a memset, which must not become a graph node.
using OnesweepConfig = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                                  rocprim::default_config, 0>;
using MergeConfig = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                               rocprim::default_config, SIZE_MAX>;

template <class K, class V>
static hipError_t radix_pairs(bool graph, void *tmp, size_t &bytes, rocprim::double_buffer<K> &kb,
                              rocprim::double_buffer<V> &vb, size_t n, unsigned end_bit,
                              hipStream_t st) {
  if (graph) return rocprim::radix_sort_pairs<MergeConfig>(tmp, bytes, kb, vb, n, 0u, end_bit, st);
  return rocprim::radix_sort_pairs<OnesweepConfig>(tmp, bytes, kb, vb, n, 0u, end_bit, st);
}

hipError_t sort_keys(int64_t n, uint64_t *keys, uint64_t *keys_alt, int64_t *vals,
                     int64_t *vals_alt, void *tmp, size_t *tmp_bytes, int64_t **sorted_out,
                     hipStream_t st, int end_bit, bool graph) {
  rocprim::double_buffer<uint64_t> kb(keys, keys_alt);
  rocprim::double_buffer<int64_t> vb(vals, vals_alt);
  hipError_t e = radix_pairs(graph, tmp, *tmp_bytes, kb, vb, (size_t)n, (unsigned)end_bit, st);
  if (tmp) *sorted_out = vb.current();
  return e;
}

hipError_t rev_setup(int64_t npairs, const PairView &v, const int32_t *score, const int32_t *qend,
                     const int64_t *rend, const uint8_t *lanebits, int32_t smax, int32_t o, int32_t e,
                     const RevSetup &s, uint8_t *err, hipStream_t st) {
  if (!npairs) return hipSuccess;
  hipLaunchKernelGGL(k_rev_setup, dim3(nb(npairs, 256)), dim3(256), 0, st, npairs, v, score, qend, rend,
                     lanebits, smax, o, e, s, err);
  return hipGetLastError();
}

hipError_t plan_sort(int64_t n, const int64_t *n_dev, const int64_t *ids, const int32_t *qlen,
                     const int64_t *rlen, const int32_t *band, int32_t R, int64_t max_q, int64_t max_r,
                     uint64_t *keys, uint64_t *keys_alt, int64_t *vals, int64_t *vals_alt, void *tmp,
                     size_t *tmp_bytes, int64_t **sorted_out, hipStream_t st, bool graph) {
  const PlanBits w = n_dev ? plan_bits(0, 0, R, band != nullptr) : plan_bits(max_q, max_r, R, band != nullptr);
  const int end_bit = w.r + w.q + w.b;
  if (tmp == nullptr) {
    rocprim::double_buffer<uint64_t> kb(keys, keys_alt);
    rocprim::double_buffer<int64_t> vb(vals, vals_alt);
    // (a graph's one buffer serves its passes with and without bands)
    size_t own = 0, b44 = 0, b64 = 0;
    hipError_t e = radix_pairs(graph, nullptr, own, kb, vb, (size_t)n, (unsigned)end_bit, st);
    if (graph && e == hipSuccess) e = radix_pairs(graph, nullptr, b44, kb, vb, (size_t)n, 44u, st);
    if (graph && e == hipSuccess) e = radix_pairs(graph, nullptr, b64, kb, vb, (size_t)n, 64u, st);
    *tmp_bytes = std::max(own, std::max(b44, b64));
    return e;
  }
  if (n == 0) { *sorted_out = vals; return hipSuccess; }
  hipLaunchKernelGGL(k_plan_keys, dim3(nb(n, 256)), dim3(256), 0, st, n, n_dev, ids, qlen, rlen,
                     band, R, w, keys, vals);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  rocprim::double_buffer<uint64_t> kb(keys, keys_alt);
  rocprim::double_buffer<int64_t> vb(vals, vals_alt);
  e = radix_pairs(graph, tmp, *tmp_bytes, kb, vb, (size_t)n, (unsigned)end_bit, st);
  *sorted_out = vb.current();
  return e;
}

hipError_t plan_tasks_dev(int64_t n, const int64_t *n_dev, int64_t ntasks, int32_t slots, int32_t R,
                          int64_t qdata_per_row, const int64_t *sorted, const int32_t *qlen,
                          const int64_t *rlen, const int32_t *band, const int32_t *band_q,
                          InterTask *tasks, int64_t *bnd_size, int64_t *qdata_size,
                          hipStream_t st) {
  if (ntasks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_plan_tasks, dim3(nb(ntasks, 4)), dim3(256), 0, st, n, n_dev, ntasks,
                     slots, R, qdata_per_row, sorted, qlen, rlen, band, band_q, tasks, bnd_size,
                     qdata_size);
  return hipGetLastError();
}

hipError_t plan_offsets_dev(int64_t ntasks, InterTask *tasks, const int64_t *bnd_off,
                            const int64_t *qdata_off, hipStream_t st) {
  if (ntasks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_plan_offsets, dim3(nb(ntasks, 128)), dim3(128), 0, st, ntasks, tasks,
                     bnd_off, qdata_off);
  return hipGetLastError();
}

hipError_t flags_to_i64(int64_t n, const uint8_t *flag, int64_t *f64, hipStream_t st) {
  hipLaunchKernelGGL(k_flag_to_i64, dim3(nb(n + 1, 256)), dim3(256), 0, st, n, flag, f64);
  return hipGetLastError();
}

hipError_t compact_flags(int64_t n, const uint8_t *flag, const int64_t *pos, int64_t *out,
                         hipStream_t st) {
  if (!n) return hipSuccess;
  hipLaunchKernelGGL(k_compact, dim3(nb(n, 256)), dim3(256), 0, st, n, flag, pos, out);
  return hipGetLastError();
}

// ---- plain fills (graph-capturable in place of memset nodes) ------------------
__global__ void k_fill_u8(int64_t n, uint8_t *p, uint8_t v) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = v;
}

__global__ void k_fill_i64(int64_t n, int64_t *p, int64_t v) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = v;
}

hipError_t fill_u8(int64_t n, uint8_t *p, uint8_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u8, dim3(nb(n, 256)), dim3(256), 0, st, n, p, v);
  return hipGetLastError();
}

hipError_t fill_i64(int64_t n, int64_t *p, int64_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i64, dim3(nb(n, 256)), dim3(256), 0, st, n, p, v);
  return hipGetLastError();
}

// ranges[2c], ranges[2c+1]: positions of class c in the class-sorted list
__global__ void k_class_ranges(const int64_t *counts, int64_t *ranges) {
  if (threadIdx.x != 0) return;
  int64_t pos = 0;
  for (int c = 0; c < 8; ++c) {
    ranges[2 * c] = pos;
    pos += counts[c];
    ranges[2 * c + 1] = pos;
  }
}

hipError_t class_ranges(const int64_t *counts, int64_t *ranges, hipStream_t st) {
  hipLaunchKernelGGL(k_class_ranges, dim3(1), dim3(64), 0, st, counts, ranges);
  return hipGetLastError();
}

}  // namespace swx
