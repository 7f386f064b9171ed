// swx_kernels.h -- launchers of the HIP kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>

#include "swx_internal.h"

namespace swx {

// device copy of the public swx_rec (same layout)
struct swx_rec_dev {
  int32_t score1, score2;
  int32_t read_begin1, read_end1;
  int64_t ref_begin1, ref_end1, ref_end2;
  int64_t cigar_off;
  int32_t cigar_len;
  int32_t lane_bits;
};

struct PackArgs {            // QGEN profile construction
  const InterTask *tasks;
  int64_t ntasks;
  const int64_t *slot_pair;
  PairView view;
  uint8_t *prof;
  uint2 *rsym;            // packed reference symbols (k_inter_rsym)
  const int8_t *matrix;   // n x n, [query symbol][reference symbol], device
  int32_t n, bias, halves, strip_rows, rev;
};

struct Score2InterArgs {
  const InterTask *tasks;
  int64_t ntasks;
  const int64_t *slot_pair;
  const int64_t *rlen;
  const int32_t *qlen;
  const uint32_t *bnd;
  const int32_t *score1;
  const int64_t *rbeg, *rend;
  int32_t mask_len;       // < 0: per pair max(qlen/2, 15)
  int32_t halves;
  int32_t *score2;
  int64_t *rend2;
};

struct ValidateArgs {
  const int8_t *qcat; int64_t qcat_len; const int64_t *qoff; int64_t nq;
  const int8_t *rcat; int64_t rcat_len; const int64_t *roff; int64_t nr;
  const int64_t *pair_q, *pair_r; int64_t npairs;
  int32_t n;
  uint32_t *bad;          // bit flags: 1 offsets, 2 pair index, 4 query symbol, 8 reference symbol
};

// banded traceback
struct TbTask {
  int32_t nslots, rows, bw, pad_;
  int64_t slot_base;
  int64_t dir_off;     // dwords
};

constexpr int kTbwSlots = 16;   // pairs per wide-band traceback task (four lanes each)
constexpr int kTbKeyBits = 23;  // traceback sort key: class (3 bits) above 20 bits of rows
constexpr int kTbFlat = 7;      // class of pairs whose alignment is their main diagonal (m M)

struct TbwTask {        // wide-band traceback task (kTbwSlots pairs)
  int32_t nslots, pad_;
  int64_t rows, wmax, dlo, width;
  int64_t slot_base;
  int64_t dir_off;      // dwords
  int64_t bnd_off;      // ints
};

// Safe band of the banded pass (method section: the band is set by the
// begin and the end).  m x w rectangle, score s1: every path of score s1 has
// at most G = floor((smax*(m+w) - 2o + 2e - 2*s1) / (smax + 2e)) gap symbols,
// so it stays on diagonals j - i in [min(0,D) - hw, max(0,D) + hw] with
// D = w - m and hw = floor((G - |D|) / 2).  Returns the lowest diagonal and
// the number of diagonals.
__host__ __device__ inline int64_t floor_div64(int64_t a, int64_t b) {
  int64_t q = a / b;
  if ((a % b != 0) && ((a < 0) != (b < 0))) --q;
  return q;
}

__host__ __device__ inline void safe_band(int64_t m, int64_t w, int64_t s1, int32_t smax, int32_t o,
                                          int32_t e, int64_t *dlo, int64_t *bw) {
  const int64_t D = w - m;
  const int64_t num = (int64_t)smax * (m + w) - 2 * o + 2 * e - 2 * s1;
  const int64_t den = (int64_t)smax + 2 * e;
  const int64_t G = den > 0 ? floor_div64(num, den) : (m + w);
  const int64_t aD = D < 0 ? -D : D;
  const int64_t hw = (G - aD) >= 0 ? (G - aD) / 2 : 0;
  *dlo = (D < 0 ? D : 0) - hw;
  *bw = ((D > 0 ? D : 0) + hw) - *dlo + 1;
}

// Pairs with more band cells than this take the wave-parallel traceback (one
// pair per workgroup) instead of one pair per lane; in a batch of at most
// kTbFewPairs pairs (less than one wave of lanes) the lower kWaveTbCellsFew.
constexpr int64_t kWaveTbCells = int64_t(1) << 18;
constexpr int64_t kWaveTbCellsFew = int64_t(1) << 14;
constexpr int64_t kTbFewPairs = 64;

// Wave-parallel traceback of one pair: rows in strips of 64 * RL (RL = 4, 8
// or 16 rows per lane), columns swept as a wavefront; choice codes stored per
// (strip, step, lane) as RL nibbles (2, 4 or 8 bytes).
struct TbWaveJob {
  int64_t pair;
  int64_t m, w;          // rectangle: query rows qbeg..qend, reference columns rbeg..rend
  int64_t dlo, bw;       // safe band (diagonals j - i, 1-based coordinates)
  int64_t dir_off;       // bytes: the pair's choice codes start there
  int64_t bnd_off;       // ints of the hand-over rows: per strip boundary (and the
                         // virtual top row) H then F, w + 1 each
};
__host__ __device__ inline int tb_code_bytes(int RL) { return RL / 2; }

// column window [clo, chi) of strip s (rows s*SH+1 .. (s+1)*SH, 1-based;
// column 0 is the virtual column left of the rectangle)
__host__ __device__ inline void tbw_window(int64_t s, int64_t SH, int64_t dlo, int64_t bw,
                                           int64_t w, int64_t *clo, int64_t *chi) {
  int64_t lo = s * SH + 1 + dlo;
  if (lo < 0) lo = 0;
  int64_t hi = (s + 1) * SH + dlo + bw;
  if (hi > w + 1) hi = w + 1;
  *clo = lo;
  *chi = hi > lo ? hi : lo;
}

// Scratch of a pair on k_tb_pairs: hand-over rows, then choice codes.
constexpr int kTbPairRows = 4;   // rows per lane
__host__ __device__ inline int64_t tb_pair_bnd_bytes(int64_t m, int64_t w) {
  const int64_t nstrips = (m + 64 * kTbPairRows - 1) / (64 * kTbPairRows);
  return (8 * (w + 1) * (nstrips + 1) + 255) / 256 * 256;
}
__host__ __device__ inline int64_t tb_pair_bytes(int64_t m, int64_t w, int64_t dlo, int64_t bw) {
  constexpr int64_t SH = 64 * kTbPairRows;
  int64_t steps = 0;
  for (int64_t s = 0; s * SH < m; ++s) {
    int64_t lo, hi;
    tbw_window(s, SH, dlo, bw, w, &lo, &hi);
    steps += hi - lo + 63;
  }
  return tb_pair_bnd_bytes(m, w) + (steps * 64 * tb_code_bytes(kTbPairRows) + 255) / 256 * 256;
}

struct TbArgs {
  const int32_t *score;
  const int32_t *qbeg, *qend;
  const int64_t *rbeg, *rend;
  const int64_t *qstart, *rstart;
  const int32_t *qlen;
  const int64_t *rlen;
  const int8_t *qcat, *rcat;
  const int8_t *matrix;
  int32_t n, o, e, smax;
  uint32_t *dir;
  uint32_t *cig;
  const int64_t *cig_off;   // null: pair p's run at p * cig_stride
  int64_t cig_stride;
  int32_t *cig_len;
  uint8_t *err;
  int64_t wave_cells;    // wide bands with more cells go to the wave-parallel kernel
};

// counts[c] (cleared by the caller) += pairs of class c, and with bytes (may be
// null) bytes[c] += their scratch on the wave kernel (k_tb_pairs).  coff[p]:
// pair p's place among the *words CIGAR scratch words (cleared by the caller);
// cig_len is preset (1 for flat pairs, else 0).
hipError_t tb_classify(const TbArgs &a, int64_t npairs, uint8_t *cls, uint64_t *key, int64_t *vals,
                       int64_t *coff, int64_t *counts, int64_t *words, int64_t *bytes, hipStream_t st);
// Wave traceback planned on the device, a workgroup per pair: pairs
// sorted[lo[x] .. lo[x] + cnt[x]) of each range, or (sorted null) every pair
// by its class, or (cls null too) every pair by its own look at it: no class
// pass ran, flat pairs are traced here and every cig_len is set.  Scratch:
// stride bytes per block, or taken from cap bytes through *used.
struct TbPairs {
  const int64_t *sorted;
  const uint8_t *cls;
  int64_t lo[4], cnt[4];
  int32_t ranges, pad_;
  int64_t stride, cap;
  unsigned long long *used;
  uint8_t *scratch;
};
hipError_t tb_pairs(const TbArgs &a, const TbPairs &t, int64_t blocks, int64_t max_rows,
                    hipStream_t st);
hipError_t tb_tasks(int64_t n0, int64_t n1, const int64_t *sorted, const TbArgs &a, int32_t bw,
                    TbTask *tasks, int64_t *dir_words, hipStream_t st);
hipError_t tb_offsets(int64_t ntasks, TbTask *tasks, const int64_t *off, hipStream_t st);
hipError_t tb_tasks_range(const int64_t *range, int64_t ntasks_cap, const int64_t *sorted,
                          const TbArgs &a, int32_t bw, TbTask *tasks, int64_t *dir_words,
                          hipStream_t st);
hipError_t tbw_tasks_range(const int64_t *range, int64_t ntasks_cap, const int64_t *sorted,
                           const TbArgs &a, TbwTask *tasks, int64_t *dir_words, int64_t *bnd_words,
                           hipStream_t st);
hipError_t tb_band(const TbArgs &a, const TbTask *tasks, int64_t ntasks, const int64_t *sorted,
                   int32_t bw, hipStream_t st);
hipError_t tbw_tasks(int64_t n0, int64_t n1, const int64_t *sorted, const TbArgs &a,
                     TbwTask *tasks, int64_t *dir_words, int64_t *bnd_words, hipStream_t st);
hipError_t tbw_offsets(int64_t ntasks, TbwTask *tasks, const int64_t *doff, const int64_t *boff,
                       hipStream_t st);
hipError_t tb_strip(const TbArgs &a, const TbwTask *tasks, int64_t ntasks, const int64_t *sorted,
                    int32_t *bndbuf, hipStream_t st);
// upper bound of the code bytes of a pair of at most m rows and w columns
int64_t tb_wave_dir_bytes(int64_t m, int64_t w, int RL);
// segs > 1: each pair's strips spread over that many workgroups (sync: one
// record per pair), then a walk kernel; else the fill and the walk in one
hipError_t tb_wave(const TbArgs &a, const TbWaveJob *jobs, int64_t njobs, int RL, int waves,
                   int segs, IntraSync *sync, uint8_t *dirw, int32_t *bnd, hipStream_t st);
int tb_wave_waves(int64_t m, int n, int RL);   // waves per workgroup for a pair of m rows
int tb_wave_max_strips();
hipError_t fill_u8(int64_t n, uint8_t *p, uint8_t v, hipStream_t st);
hipError_t fill_i64(int64_t n, int64_t *p, int64_t v, hipStream_t st);
// lane-width probe: blocks x 256 threads, each 32/bits synthetic pairs of 16
// rows x cols columns; best[pair] = the pair's best score
// adds to *bad the results of VT<u16x2>::max3 that differ from the unsigned
// maximum over the check's operand set; *checked: the number of lane results
hipError_t max3_check(unsigned long long *bad, uint64_t *checked, hipStream_t st);
hipError_t lane_probe(int bits, int64_t cols, int64_t blocks, int32_t o, int32_t e, uint32_t *best,
                      hipStream_t st);
hipError_t class_ranges(const int64_t *counts, int64_t *ranges, hipStream_t st);
// graph: the sort is recorded into a HIP graph (a form that issues no memset)
hipError_t sort_keys(int64_t n, uint64_t *keys, uint64_t *keys_alt, int64_t *vals,
                     int64_t *vals_alt, void *tmp, size_t *tmp_bytes, int64_t **sorted_out,
                     hipStream_t st, int end_bit = 64, bool graph = false);
// Drift band of the reversed pass over `rows` rows and `cols` columns.
// Every alignment of score score1 in the reversed region starts at the
// reversed corner (T1 leaves no other cell of that value there).  A path
// that drifts d diagonals off the corner's diagonal holds at least d gap
// symbols, so score1 <= smax*min(qend+1, rend+1) - o - (d-1)e: d <= G'.
// When the drift is towards the query (i - j = d) those d symbols are
// insertions, which also leave at most qend+1-d rows for matches:
// score1 <= smax*(qend+1-d) - o - (d-1)e, so d <= Gq =
// (smax*(qend+1) - o + e - score1) / (smax + e); towards the reference
// likewise with rend+1 (Gr).  band = max(min(G', Gq), min(G', Gr)) bounds
// both sides, band_q = min(G', Gq) the query side (e > 0; with e == 0 no band
// is used).
__device__ __forceinline__ int64_t rev_drift(int64_t num, int64_t den) {
  const int64_t g = num / den;
  return g < 0 ? 0 : (g > (1 << 30) ? (1 << 30) : g);
}

__device__ __forceinline__ void rev_band(int32_t score, int64_t rows, int64_t cols, int32_t smax,
                                         int32_t o, int32_t e, int32_t &band, int32_t &band_q) {
  band = band_q = -1;
  if (e <= 0) return;
  const int64_t base = -(int64_t)o + e - score;
  const int64_t g = rev_drift((int64_t)smax * (rows < cols ? rows : cols) + base, e);
  int64_t gq = rev_drift((int64_t)smax * rows + base, (int64_t)smax + e);
  int64_t gr = rev_drift((int64_t)smax * cols + base, (int64_t)smax + e);
  gq = gq < g ? gq : g;
  gr = gr < g ? gr : g;
  band = (int32_t)(gq > gr ? gq : gr);
  band_q = (int32_t)gq;
}

// what the reversed pass takes of each pair, and its score's preset (k_rev_setup)
struct RevSetup {
  int64_t *qstart, *rstart, *rlen;
  int32_t *qlen, *target, *band, *band_q, *score;
  uint8_t *f16, *f32;
};
hipError_t rev_setup(int64_t npairs, const PairView &v, const int32_t *score, const int32_t *qend,
                     const int64_t *rend, const uint8_t *lanebits, int32_t smax, int32_t o, int32_t e,
                     const RevSetup &s, uint8_t *err, hipStream_t st);

hipError_t inter_fill(const InterArgs &a, int lane_bits, int R, hipStream_t st);
// keys[t] = padded rows x swept columns of task t (a banded task's window of R +
// band_q + band columns per strip) / 256, vals[t] = t (for InterArgs::order; sorted on
// 24 key bits)
hipError_t inter_area_keys(const InterTask *tasks, int64_t ntasks, int32_t R, uint64_t *keys,
                           int64_t *vals, hipStream_t st);

// intra-sequence path (long pairs)
struct IntraPair {         // one long pair's forward max array
  int64_t pair;
  int64_t mc_off;          // words at maxcol + mc_off, [rlen]
  int32_t kbits;           // row-code bits
  int32_t sh;              // strip height of its forward jobs (padding rows = roundup(qlen, sh) - qlen)
};
struct IntraPairArgs {
  const IntraPair *pairs;  // null: pair ids[k] (ids null: k) as AloneArgs lays it out
  const int64_t *ids;
  int64_t stride;
  const uint32_t *maxcol;
  const int32_t *qlen;
  const int64_t *rlen;
  int32_t *score;          // score1 (written by the end kernel, read by score2)
  int32_t *qend;
  int64_t *rend;
  uint8_t *overflow;
  const int64_t *rbeg;     // score2: begin of the primary alignment
  int32_t mask_len;
  int32_t *score2;
  int64_t *rend2;
  int32_t *part_v;         // per (pair, slice) partial bests: intra_slices() per pair
  int64_t *part_j;
  int64_t max_rlen;        // longest reference of the launch (its shape)
  int64_t first;           // (launches of part of the list) its first pair
};

// Long-path pairs of short queries, a wave per pair (or two pairs on 16-bit
// lanes), whole references: no job tables.  ids (null: every pair in turn) and
// the max array words of the k-th at maxcol + k * stride, row-code bits
// kAloneBits, rows coded in kAloneMaxQ padded rows.
constexpr int32_t kAloneMaxQ = 512;
constexpr int32_t kAloneBits = 16;
struct AloneArgs {
  const int64_t *ids;
  int64_t count;
  PairView view;
  const int8_t *matrix;
  int32_t n, o, e, bias;
  int32_t max_q;             // longest query of the launch (its shape)
  uint32_t *maxcol;
  int64_t stride;
  uint8_t *lanebits;         // forward: 32 is written (32-bit lanes; may be null)
  const uint8_t *is_long;    // 16-bit forward (may be null): ... for other pairs that reach the
                             // limit of the batched pass's 16-bit lanes, which rerun there
  const int32_t *target, *band;   // reversed pass (band may be null)
  // what follows the forward pass in one go (alone_pass, alone_begin): begins
  // and, with score2, the best outside the mask
  int32_t smax, mask_len;
  int32_t *qbeg, *score2;    // (score2 may be null)
  int64_t *rbeg, *rend2;
  uint8_t *err;
  uint32_t anchor;           // ... of paths from the corner alone (queries shorter than max_q then), else 0
  FillOut out;
};
// above every score of a pair whose words have room for the anchor and a score
constexpr uint32_t kAloneAnchor = 1u << 15;
hipError_t alone_forward(const AloneArgs &a, hipStream_t st);
hipError_t alone_pass(const AloneArgs &a, hipStream_t st);    // forward, 32-bit lanes, and all that follows it
hipError_t alone_begin(const AloneArgs &a, hipStream_t st);   // what follows it alone
hipError_t alone_last(const AloneArgs &a, hipStream_t st);   // best of the last column only; empty references skipped
hipError_t alone_forward16(const AloneArgs &a, bool m3, hipStream_t st);
hipError_t alone_reverse(const AloneArgs &a, hipStream_t st);

// The one-pair call (swx_align) of short queries, in three kernels: the inputs
// staged and checked, the forward pass on a workgroup per column chunk, and
// everything after it on one workgroup.
constexpr int kPairRows = 4;          // rows per lane
constexpr int kPairWaves = 8;         // most waves of a workgroup, and most strips of a query
constexpr int32_t kPairMaxQ = 64 * kPairRows * kPairWaves;
constexpr int64_t kPairMaxR = int64_t(1) << 16;
struct PairOut {         // in pinned host memory, the CIGAR's words after it
  swx_rec_dev rec;
  int32_t bad;           // a symbol code outside [0, n)
  int32_t err;           // an internal check failed
  uint64_t done;         // the call's number, written last
};
struct PairState {       // the pair's arrays of one element each (TbArgs)
  int64_t qstart, rstart, rbeg, rend, rlen, cig_off;
  int32_t score, qbeg, qend, qlen, cig_len;
  uint8_t err;
};
struct PairArgs {
  const int8_t *src_q, *src_r, *src_m;   // pinned host memory, or the caller's device reference
  int8_t *q, *r, *m;                     // device copies, every code inside [0, n)
  int32_t Lq, kb;
  int64_t Lr;
  int32_t n, o, e, bias, smax;
  int64_t chunk, warm;                   // columns per chunk, warm-up before it
  int32_t nchunks, strips;
  uint32_t *maxcol;                      // [Lr]
  uint64_t *fwords, *rwords;             // hand-over words of several strips, cleared by the staging
  int64_t fstride, rcount;               // words per chunk; words of the reversed pass
  uint32_t flags;
  int32_t mask_len;
  TbArgs tb;
  PairState *state;
  uint8_t *dir;
  int32_t *bnd;
  PairOut *out;
  uint64_t seq;            // this call's number
};
int pair_waves(int strips, int n);
hipError_t pair_stage(const PairArgs &a, hipStream_t st);
hipError_t pair_forward(const PairArgs &a, hipStream_t st);
hipError_t pair_rest(const PairArgs &a, hipStream_t st);

size_t intra_lds_bytes(int n, int RL);
int intra_slices();
hipError_t intra_fill(const IntraArgs &a, int RL, int waves, bool rev, hipStream_t st);
// sets the progress records of a spread launch's jobs (before each launch)
hipError_t intra_sync_init(IntraSync *sync, int64_t njobs, hipStream_t st);
// forward pass on packed 16-bit lanes: jobs[2b] and jobs[2b + 1] (same padded
// height; pair -1: none) share workgroup b; a.njobs even
// m3: every pair's score bound plus bias is below 0x7C00 (one packed
// three-way maximum per row instead of two maxima)
hipError_t intra_fill16(const IntraArgs &a, int RL, int waves, bool m3, hipStream_t st);
size_t intra_lds_bytes16(int n, int RL);
int intra_max_strips();
int intra_max_waves();
hipError_t intra_jobs_chunked(int64_t B, int32_t nc, int64_t cw, const int32_t *qlen,
                              const int64_t *rlen, int32_t smax, int32_t o, int32_t e,
                              int32_t kbits, int32_t sh, int64_t mc_stride, int64_t bnd_stride,
                              IntraJob *jobs, IntraPair *pairs, hipStream_t st);
hipError_t intra_rev_jobs_fixed(int64_t B, const int32_t *score, const int64_t *rend,
                                const int32_t *band, int32_t kbits, int64_t bnd_stride,
                                IntraJob *jobs, hipStream_t st);
size_t intra_static_lds();
hipError_t intra_end(const IntraPairArgs &a, int64_t npairs, hipStream_t st);
hipError_t intra_score2(const IntraPairArgs &a, int64_t npairs, hipStream_t st);
hipError_t split_long(int64_t n, const int32_t *qlen, const int64_t *rlen, int64_t cells_thr,
                      int64_t mult, int64_t rlen_thr, const int64_t *stats, uint8_t *is_long,
                      uint8_t *is_short, int64_t *count, hipStream_t st);
hipError_t gather_pairs(int64_t n, const int64_t *ids, const int32_t *qlen, const int64_t *rlen,
                        const int32_t *score, const int32_t *qend, const int64_t *rend,
                        const int32_t *band, int64_t *out, hipStream_t st);
hipError_t clear_flags(int64_t n, const int64_t *ids, uint8_t *f1, uint8_t *f2, hipStream_t st);
hipError_t inter_pack(const PackArgs &a, hipStream_t st);
hipError_t inter_pack_ref(const PackArgs &a, hipStream_t st);

hipError_t launch_validate(const ValidateArgs &a, hipStream_t st);
// the shared query profile of a pass whose pairs all use one query (k_build_qprof)
hipError_t build_qprof(const int8_t *q, int32_t qlen, const int8_t *matrix, int32_t n, int32_t bias,
                       int32_t qp, uint8_t *fwd, int64_t rev_row, uint8_t *rev, hipStream_t st);
// bytes of a reversed row of the shared profile for strips of R rows
inline int64_t qprof_rev_row(int64_t qlen, int R) { return (2 * qlen + 2 * R + 16 + 15) / 16 * 16; }
hipError_t lens_to_i64(int64_t n, const int32_t *len, int64_t *out, hipStream_t st);
// off[0 .. n] = exclusive prefix sums of len and their total, in one launch of
// one block (n up to kScanLensMax)
constexpr int64_t kScanLensMax = 65536;
hipError_t scan_lens(int64_t n, const int32_t *len, int64_t *off, hipStream_t st);
hipError_t mark_lanes(int64_t n, const int64_t *ids, uint8_t *lanebits, int v, hipStream_t st);
hipError_t mark_lanes_dev(int64_t cap, const int64_t *n_dev, const int64_t *ids, uint8_t *lanebits,
                          int v, hipStream_t st);
// bounds the views are clamped into (see k_views)
struct ViewCaps {
  int64_t nq, nr, qcat_len, rcat_len;
  int32_t max_qlen, pad_;
  int64_t max_rlen;
};
hipError_t launch_views(int64_t npairs, const int64_t *qoff, const int64_t *roff,
                        const int64_t *pair_q, const int64_t *pair_r, const ViewCaps &caps,
                        int64_t *qstart, int32_t *qlen, int64_t *rstart, int64_t *rlen,
                        int64_t *stats, hipStream_t st);
// one launch for many clears: entry k sets n[k] elements of size[k] bytes
// (1, 4 or 8) at p[k] to v[k]
constexpr int kFillSetMax = 12;
struct FillSet {
  void *p[kFillSetMax];
  int64_t n[kFillSetMax];
  int64_t v[kFillSetMax];
  int32_t size[kFillSetMax];
  int32_t count;
  void add(void *ptr, int64_t count_, int32_t bytes, int64_t value) {
    p[count] = ptr; n[count] = count_; size[count] = bytes; v[count] = value; ++count;
  }
};
hipError_t fill_set(const FillSet &f, hipStream_t st);
// Copies by a kernel between device memory and pinned host memory.
constexpr int kCopySetMax = 8;
struct CopySet {         // every pointer 16-byte aligned
  const void *src[kCopySetMax];
  void *dst[kCopySetMax];
  int64_t bytes[kCopySetMax];
  int32_t count;
  void add(const void *s, void *d, int64_t n) {
    src[count] = s; dst[count] = d; bytes[count] = n; ++count;
  }
};
hipError_t copy_set(const CopySet &c, hipStream_t st);
// values of up to two device arrays to pinned host memory, one after the other,
// then *flag = seq
hipError_t publish(const int64_t *a, int64_t na, const int64_t *b, int64_t nb, int64_t *dst,
                   uint64_t *flag, uint64_t seq, hipStream_t st);
// npairs records and, with CIGARs, their words [0, off[npairs]) up to cap, to
// pinned host memory; *total = off[npairs]
hipError_t graph_out(int64_t npairs, const swx_rec_dev *recs, const uint32_t *cigar, const int64_t *off,
                     int64_t cap, swx_rec_dev *hrecs, uint32_t *hcigar, int64_t *total, hipStream_t st);
// CIGAR words to their final offsets
// cls: the traceback classes (pairs of class kTbFlat hold no scratch words:
// their one word is made from qbeg and qend)
// (src_off null: runs at p * stride; cls may be null; nothing is copied when
// the words, dst_off[npairs], are more than cap)
hipError_t launch_cigar_compact(int64_t npairs, const uint32_t *src, const int64_t *src_off,
                                const int32_t *len, const int64_t *dst_off, const uint8_t *cls,
                                const int32_t *qbeg, const int32_t *qend, uint32_t *dst,
                                int64_t stride, int64_t cap, hipStream_t st);
hipError_t launch_score2_inter(const Score2InterArgs &a, hipStream_t st);
// err (may be null): *nerr += the pairs whose flag is set; CIGARs of more than
// cap words in all (cig_off[npairs]) are left out of the records
hipError_t launch_records(int64_t npairs, const int32_t *score1, const int32_t *score2,
                          const int32_t *qbeg, const int32_t *qend, const int64_t *rbeg,
                          const int64_t *rend, const int64_t *rend2, const int64_t *cig_off,
                          const int32_t *cig_len, const uint8_t *lane_bits, uint32_t flags,
                          swx_rec_dev *recs, const uint8_t *err, int64_t *nerr, int64_t cap,
                          hipStream_t st);
// the suboptimal alignment: window views, anchored reversed views, begins,
// and CIGAR offsets of records counted from the arena's start
hipError_t launch_sub_window(int64_t npairs, const int64_t *rstart, const int32_t *qlen,
                             const int32_t *score2, const int64_t *rend2, int32_t smax, int32_t o,
                             int32_t e, int64_t *wrstart, int64_t *wrlen, uint8_t *flag,
                             hipStream_t st);
hipError_t launch_sub_rev_views(int64_t npairs, const int64_t *qstart, const int64_t *rstart,
                                const int32_t *qlen, const int32_t *score2, const int64_t *rend2,
                                const int32_t *wscore, const int32_t *wqend, uint32_t anchor,
                                int64_t *rqstart, int32_t *rqlen, int64_t *rrstart, int64_t *rrlen,
                                int32_t *target, uint8_t *flag, uint8_t *err, hipStream_t st);
hipError_t launch_sub_begins(int64_t npairs, const int32_t *score2, const int64_t *rend2,
                             const int32_t *wqend, const uint8_t *flag, const int32_t *target,
                             const int32_t *rscore, const int32_t *rqend, const int64_t *rrend,
                             int32_t *sscore, int32_t *sqbeg, int32_t *sqend, int64_t *srbeg,
                             int64_t *srend, uint8_t *err, hipStream_t st);
hipError_t shift_cigar_offsets(int64_t npairs, int64_t base, swx_rec_dev *recs, hipStream_t st);
hipError_t launch_begins(int64_t npairs, const int32_t *score1, const int32_t *qend,
                         const int64_t *rend, const int32_t *rscore, const int32_t *rqend,
                         const int64_t *rrend, int32_t *qbeg, int64_t *rbeg, uint8_t *err,
                         hipStream_t st);
// max_q, max_r: no pair is longer (0: not known; not used with n_dev)
hipError_t plan_sort(int64_t n, const int64_t *n_dev, const int64_t *ids, const int32_t *qlen, const int64_t *rlen,
                     const int32_t *band, int32_t R, int64_t max_q, int64_t max_r, uint64_t *keys, uint64_t *keys_alt,
                     int64_t *vals, int64_t *vals_alt, void *tmp, size_t *tmp_bytes,
                     int64_t **sorted_out, hipStream_t st, bool graph = false);
hipError_t plan_tasks_dev(int64_t n, const int64_t *n_dev, int64_t ntasks, int32_t slots, int32_t R,
                          int64_t qdata_per_row, const int64_t *sorted, const int32_t *qlen,
                          const int64_t *rlen, const int32_t *band, const int32_t *band_q,
                          InterTask *tasks, int64_t *bnd_size, int64_t *qdata_size,
                          hipStream_t st);
hipError_t plan_offsets_dev(int64_t ntasks, InterTask *tasks, const int64_t *bnd_off,
                            const int64_t *qdata_off, hipStream_t st);
// f64[0 .. n) = flag != 0, f64[n] = 0 (n + 1 values, ready for an exclusive scan)
hipError_t flags_to_i64(int64_t n, const uint8_t *flag, int64_t *f64, hipStream_t st);
hipError_t compact_flags(int64_t n, const uint8_t *flag, const int64_t *pos, int64_t *out,
                         hipStream_t st);
hipError_t launch_exclusive_scan(const int64_t *in, int64_t *out, int64_t n, void *tmp,
                                 size_t *tmp_bytes, hipStream_t st);

}  // namespace swx
