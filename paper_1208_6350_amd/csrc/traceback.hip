// traceback.hip -- the banded pass that produces the detailed alignment.
//
// Method section: "the banded SW (whose band is defined by the beginning and
// ending positions) generates the detailed alignment".  For each pair the
// global 3-state DP on q[qbeg..qend] x r[rbeg..rend] is filled inside the
// safe band (every path of score score1 has at most G gap symbols, so it stays
// within a fixed set of diagonals; inside any superset of that set the DP
// values on those paths are exact), a 4-bit choice code is stored per cell,
// and the path is traced back from the end cell with rule T3 (M, then D, then
// I; inside a gap "open" before "extend").
//
// Layout: one lane per pair, 64 pairs of similar band width per wave.  The
// band of a lane is BW diagonals starting at its own lowest diagonal; BW is
// the task's width class (8, 16, 32 or 64), a superset of the lane's band.
// The previous row of H and F lives in registers; cells left of column 0 hold
// -inf and cells right of the last column only feed cells right of it, so no
// per-cell masking is needed.  Choice codes of one row are packed 8 per dword
// (the first cell in the top nibble) and stored lane-interleaved (coalesced).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "intra_strips.h"
#include "swx_internal.h"
#include "swx_kernels.h"

namespace swx {

constexpr int32_t kNeg = -(1 << 29);
constexpr int64_t kTbMaxStripsDecl = 256;   // strips of one wave-traceback pair (kTbMaxStrips)

// Choice code of a cell: bit 3 "H does not come from the diagonal"
// (diag < H), bit 2 "F rather than E" (E < F), bit 1 "E extends" (the
// opening H - o < the extension E - e), bit 0 "F extends".  Each bit is the
// sign of a difference (every value here lies in [-2^30, 2^26]), shifted into
// the accumulator from the right, so a word fills from its top nibble down.
// Ties give M before E before F and "open" before "extend" (rule T3).
constexpr uint32_t kCodeNotM = 8u, kCodeF = 4u, kCodeEExt = 2u, kCodeFExt = 1u;
__device__ __forceinline__ uint32_t push_code(uint32_t acc, int32_t diag, int32_t h, int32_t eij,
                                              int32_t fij, int32_t eo, int32_t ex, int32_t fo,
                                              int32_t fx) {
  acc = __builtin_amdgcn_alignbit(acc, (uint32_t)(diag - h), 31);
  acc = __builtin_amdgcn_alignbit(acc, (uint32_t)(eij - fij), 31);
  acc = __builtin_amdgcn_alignbit(acc, (uint32_t)(eo - ex), 31);
  return __builtin_amdgcn_alignbit(acc, (uint32_t)(fo - fx), 31);
}
// the source of H named by a code: 0 diagonal, 1 E, 2 F
__device__ __forceinline__ uint32_t code_src(uint32_t c) {
  return (c & kCodeNotM) ? ((c & kCodeF) ? 2u : 1u) : 0u;
}
// The walk's moves (rule T3) by state (0 H, 1 E, 2 F) and choice code:
// nibble c of walk_moves(state) = next state << 2 | row up << 1 | column
// left.  In H the code names H's source: the diagonal (M, up and left) or a
// gap state; in E a D move left, staying in E while E extends; in F an I move
// up, staying in F while F extends.
constexpr uint64_t walk_moves(int state) {
  uint64_t t = 0;
  for (uint32_t c = 0; c < 16; ++c) {
    uint32_t v = 0;
    if (state == 0) {
      const uint32_t src = (c & kCodeNotM) ? ((c & kCodeF) ? 2u : 1u) : 0u;
      v = src == 0 ? 3u : (src << 2);
    } else if (state == 1) {
      v = ((c & kCodeEExt) ? 1u : 0u) << 2 | 1u;
    } else {
      v = ((c & kCodeFExt) ? 2u : 0u) << 2 | 2u;
    }
    t |= (uint64_t)v << (4 * c);
  }
  return t;
}
constexpr uint64_t kMovesH = walk_moves(0), kMovesE = walk_moves(1), kMovesF = walk_moves(2);

// row 0 of the global DP: reached from the left by one deletion run
__device__ __forceinline__ uint32_t row0_code(int64_t j, int32_t o, int32_t e) {
  return (j == 0) ? 0u : (kCodeNotM | ((j == 1 || o <= e) ? 0u : kCodeEExt));
}

// where pair p's runs go
__device__ __forceinline__ uint32_t *tb_cig(const TbArgs &a, int64_t p) {
  return a.cig + (a.cig_off ? a.cig_off[p] : p * a.cig_stride);
}

__device__ __forceinline__ bool tb_coords_ok(const TbArgs &a, int64_t p) {
  return a.qbeg[p] >= 0 && a.qbeg[p] <= a.qend[p] && a.qend[p] < a.qlen[p] && a.rbeg[p] >= 0 &&
         a.rbeg[p] <= a.rend[p] && a.rend[p] < a.rlen[p];
}

// per pair: band class (0: none, 1..4: BW 8/16/32/64, 5: wider, 6: wave kernel,
// kTbFlat: no band pass), rows, key; counts[c] += pairs of class c.
//
// kTbFlat: a square rectangle whose main diagonal alone scores score1.  No
// path scores more (score1 is the optimum of the rectangle), so on the
// diagonal H(k, k) equals the diagonal's prefix sum at every k (a larger
// value, completed along the diagonal, would beat score1): the diagonal
// candidate always equals H, and rule T3, which prefers M, walks it
// end to end.  The CIGAR is m M, with no choice codes needed.  A thread sums
// its pair's diagonal in 16-byte words (about 2 bytes read per row, against
// ~20 instructions per band cell and a serial walk).  On reads with 0.5%
// indels about 40% of the pairs end here (1,000,000 reads: band kernels'
// tasks 900k -> 507k pairs, the sums 0.08 ms, the whole call 19.1 -> 18.6 ms).
__device__ __forceinline__ int32_t diagonal_sum(const int8_t *q, const int8_t *r, int32_t m,
                                                const int8_t *s_mat) {
  // 32 x 32 scores, zero past n x n: any code stays inside the table
  auto cell = [&](uint32_t qc, uint32_t rc) { return (int32_t)s_mat[(qc & 31u) * 32u + (rc & 31u)]; };
  int32_t sum = 0;
  if (m < 16) {
    for (int32_t x = 0; x < m; ++x) sum += cell((uint8_t)q[x], (uint8_t)r[x]);
    return sum;
  }
  for (int32_t x = 0; x < m; x += 16) {
    // whole words at any alignment; the last one ends with the diagonal and
    // skips the bytes it shares with the one before
    const int32_t x0 = x + 16 <= m ? x : m - 16;
    const int32_t skip = x - x0;
    uint32_t qw[4], rw[4];
    __builtin_memcpy(qw, q + x0, 16);
    __builtin_memcpy(rw, r + x0, 16);
#pragma unroll
    for (int b = 0; b < 16; ++b) {
      const int32_t v = cell(__builtin_amdgcn_ubfe(qw[b >> 2], 8 * (b & 3), 8),
                             __builtin_amdgcn_ubfe(rw[b >> 2], 8 * (b & 3), 8));
      sum += b >= skip ? v : 0;
    }
  }
  return sum;
}

__global__ __launch_bounds__(256) void k_tb_classify(TbArgs a, int64_t npairs, uint8_t *cls,
                                                     uint64_t *key, int64_t *vals, int64_t *coff,
                                                     int64_t *counts, int64_t *words, int64_t *bytes) {
  __shared__ int8_t s_mat[32 * 32];
  __shared__ unsigned long long s_cnt[8], s_bytes[8];
  __shared__ int64_t s_words[5];   // CIGAR scratch words of the waves, and where the block's begin
  for (int k = threadIdx.x; k < 32 * 32; k += blockDim.x) {
    const int qc = k / 32, rc = k % 32;
    s_mat[k] = qc < a.n && rc < a.n ? a.matrix[qc * a.n + rc] : (int8_t)0;
  }
  if (threadIdx.x < 8) s_cnt[threadIdx.x] = s_bytes[threadIdx.x] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x; p0 < npairs; p0 += stride) {
    const int64_t p = p0 + threadIdx.x;
    uint8_t c = 0;
    int64_t m = 0, w = 0, bw = 0, dlo = 0;
    const int32_t s1 = p < npairs ? a.score[p] : 0;
    if (s1 > 0) {
      if (tb_coords_ok(a, p)) {
        m = a.qend[p] - a.qbeg[p] + 1;
        w = a.rend[p] - a.rbeg[p] + 1;
        safe_band(m, w, s1, a.smax, a.o, a.e, &dlo, &bw);
        // bands wider than 32 go to the strip kernel (a 64-wide band in one
        // lane's registers spills and leaves too few waves); pairs of more
        // than wave_cells band cells to the wave-parallel kernel
        const bool wave_fits = m <= int64_t(64) * 16 * kTbMaxStripsDecl;   // the wave kernel's strip limit
        c = (m * bw > a.wave_cells && wave_fits) ? 6 : bw <= 8 ? 1 : bw <= 16 ? 2 : bw <= 32 ? 3 : 5;
        // flat pairs with k mismatches have bands of about 2k diagonals: the
        // test is left out where the band is wide, i.e. for the weak
        // alignments of unrelated sequences, which hold gaps nearly always
        // (all-vs-all reads: 92 us of diagonal sums for nothing).  (2^24
        // scores of at most 127 fit 32 bits.)
        if (m == w && bw <= 16 && m < (1 << 24) &&
            diagonal_sum(a.qcat + a.qstart[p] + a.qbeg[p], a.rcat + a.rstart[p] + a.rbeg[p],
                         (int32_t)m, s_mat) == s1)
          c = kTbFlat;
      } else {
        a.err[p] = 1;
      }
    }
    // the scratch words of the block's pairs: one place in the buffer for all
    // of them (no prefix sum over the batch, which took three launches)
    const int64_t need = (c != 0 && c != kTbFlat) ? (m + w + 2) : 0;
    int64_t before = need;   // inclusive sum over the wave's lanes
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t u = __shfl_up(before, off, 64);
      if ((int)(threadIdx.x & 63) >= off) before += u;
    }
    const int wv = (int)(threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 63) s_words[wv] = before;
    __syncthreads();
    if (threadIdx.x == 0) {
      const int64_t all = s_words[0] + s_words[1] + s_words[2] + s_words[3];
      s_words[4] = all ? (int64_t)atomicAdd((unsigned long long *)words, (unsigned long long)all) : 0;
    }
    __syncthreads();
    int64_t at = s_words[4] + before - need;
    for (int k = 0; k < wv; ++k) at += s_words[k];
    __syncthreads();   // (before the next round's sums)
    if (p >= npairs) continue;
    cls[p] = c;
    coff[p] = at;
    // class, then rows (clamped: only the grouping of similar heights matters);
    // wide bands (16 pairs share a task's column window, the union of their
    // bands) by rows in steps of 16, then lowest and highest diagonal, so that
    // a task's pairs have similar bands
    uint64_t sub = (uint64_t)(m > 0xFFFFF ? 0xFFFFF : m);
    if (c == 5) {
      const int64_t mq = m / 16 > 63 ? 63 : m / 16;
      const int64_t lo = -dlo < 0 ? 0 : (-dlo > 127 ? 127 : -dlo);
      const int64_t hi = dlo + bw - 1 + 32;
      sub = (uint64_t)(mq << 14) | (uint64_t)(lo << 7) | (uint64_t)(hi < 0 ? 0 : (hi > 127 ? 127 : hi));
    }
    key[p] = ((uint64_t)c << (kTbKeyBits - 3)) | sub;
    vals[p] = p;
    a.cig_len[p] = c == kTbFlat ? 1 : 0;
    if (bytes && c >= 1 && c <= 5) {   // too tall for the wave kernel's strips: more than any scratch
      const bool fits = (m + 64 * kTbPairRows - 1) / (64 * kTbPairRows) <= kTbMaxStripsDecl;
      atomicAdd(&s_bytes[c], (unsigned long long)(fits ? tb_pair_bytes(m, w, dlo, bw) : int64_t(1) << 40));
    }
    // class counts: one LDS atomic per class present in the wave
    for (int k = 0; k < 8; ++k) {
      const unsigned long long in = __ballot(c == k);
      if (in && (int)(threadIdx.x & 63) == __builtin_ctzll(in)) atomicAdd(&s_cnt[k], (unsigned long long)__popcll(in));
    }
  }
  __syncthreads();
  if (threadIdx.x < 8 && s_cnt[threadIdx.x])
    atomicAdd((unsigned long long *)&counts[threadIdx.x], s_cnt[threadIdx.x]);
  if (threadIdx.x < 8 && s_bytes[threadIdx.x])
    atomicAdd((unsigned long long *)&bytes[threadIdx.x], s_bytes[threadIdx.x]);
}

__device__ __forceinline__ int64_t wave_max_i64(int64_t v) {
  for (int off = 32; off >= 1; off >>= 1) {
    const int64_t o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return v;
}

// tasks over sorted[n0 .. n1); with range (device) the bounds are read there
// and every task slot up to ntasks_cap is written (empty past the range).
// One wave per task, one lane per slot.
__global__ void k_tb_tasks(int64_t n0, int64_t n1, const int64_t *range, int64_t ntasks_cap,
                           const int64_t *sorted, const TbArgs a, int32_t bw, TbTask *tasks,
                           int64_t *dir_words) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (range) { n0 = range[0]; n1 = range[1]; }
  const int64_t ntasks = (n1 - n0 + 63) / 64;
  if (t >= (range ? ntasks_cap : ntasks)) return;
  if (t >= ntasks) {
    if (lane == 0) {
      tasks[t] = TbTask{};
      dir_words[t] = 0;
    }
    return;
  }
  const int64_t s0 = n0 + t * 64;
  const int64_t s1 = (s0 + 64 < n1) ? s0 + 64 : n1;
  int64_t rows = 1;
  if (s0 + lane < s1) {
    const int64_t p = sorted[s0 + lane];
    rows = a.qend[p] - a.qbeg[p] + 1;
  }
  rows = wave_max_i64(rows);
  if (lane != 0) return;
  TbTask tk{};
  tk.nslots = (int32_t)(s1 - s0);
  tk.rows = (int32_t)rows;
  tk.bw = bw;
  tk.slot_base = s0;
  tasks[t] = tk;
  dir_words[t] = (rows + 1) * (bw / 8) * 64;
}

__global__ void k_tb_offsets(int64_t ntasks, TbTask *tasks, const int64_t *off) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < ntasks) tasks[t].dir_off = off[t];
}

template <int BW, bool LUT4>
__global__ __launch_bounds__(256) void k_tb_band(TbArgs a, const TbTask *tasks, int64_t ntasks,
                                                 const int64_t *sorted) {
  __shared__ int8_t s_mat[32 * 32];
  __shared__ uint32_t s_lut4[32];   // LUT4: scores of query symbol x against reference 0..3
  constexpr int kRunSlots = 16;     // CIGAR runs per thread kept in LDS during the walk
  __shared__ uint32_t s_runs[(kRunSlots + 1) * 256];
  for (int k = threadIdx.x; k < a.n * a.n; k += blockDim.x) s_mat[k] = a.matrix[k];
  if (LUT4 && (int)threadIdx.x < a.n) {
    uint32_t l = 0;
    for (int b = 0; b < a.n; ++b) l |= (uint32_t)(uint8_t)a.matrix[threadIdx.x * a.n + b] << (8 * b);
    s_lut4[threadIdx.x] = l;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  // tasks are sorted by rows, ascending: the largest go first, so that the
  // launch does not end on its longest tasks
  const int64_t k_ = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (k_ >= ntasks) return;
  const int64_t tid = ntasks - 1 - k_;
  const TbTask tk = tasks[tid];
  if (tk.nslots == 0) return;
  const bool live = lane < tk.nslots;
  const int64_t p = live ? sorted[tk.slot_base + lane] : -1;
  int64_t m = 1, w = 1, dlo = 0, bwl = 1;
  int32_t s1 = 0;
  const int8_t *q = a.qcat, *r = a.rcat;
  if (live) {
    s1 = a.score[p];
    m = a.qend[p] - a.qbeg[p] + 1;
    w = a.rend[p] - a.rbeg[p] + 1;
    safe_band(m, w, s1, a.smax, a.o, a.e, &dlo, &bwl);
    q = a.qcat + a.qstart[p] + a.qbeg[p];
    r = a.rcat + a.rstart[p] + a.rbeg[p];
  }
  const int32_t o = a.o, e = a.e;
  uint32_t *dir = a.dir + tk.dir_off;
  constexpr int ND = BW / 8;        // direction dwords per row
  constexpr int NW = BW / 4 + 2;    // reference window dwords

  const int8_t *qq = live ? q : (const int8_t *)a.matrix;   // readable bytes for empty lanes
  const int8_t *rr = live ? r : (const int8_t *)a.matrix;
  const int64_t mq = live ? m : 1, wr = live ? w : 1;
  // reference window: byte k of the window = symbol at local column
  // base + k (1-based columns j use symbol r[j-1]); row i covers j = i+dlo+k.
  // Its bytes are loaded all at once (indices clamped into the sequence) and
  // masked afterwards.
  uint32_t win[NW];
  {
    const int64_t j0 = 1 + dlo;   // row 1, k = 0
    int32_t raw[4 * NW];
#pragma unroll
    for (int x = 0; x < 4 * NW; ++x) {
      int64_t y = j0 + x - 1;
      y = y < 0 ? 0 : (y > wr - 1 ? wr - 1 : y);
      raw[x] = rr[y];
    }
#pragma unroll
    for (int d = 0; d < NW; ++d) {
      uint32_t v = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int64_t j = j0 + 4 * d + b;
        const int32_t c = (live && j >= 1 && j <= w) ? raw[4 * d + b] : 0;
        const uint32_t sy = (c >= 0 && c < a.n) ? (uint32_t)c : 0u;   // a bad code never indexes a table
        v |= (LUT4 ? sy * 8u : sy) << (8 * b);
      }
      win[d] = v;
    }
  }
  int32_t H[BW], F[BW];
  // row 0: H(0,0) = 0, H(0,j) = E(0,j) = -(o + (j-1)e); F(0,.) = -inf
  {
    uint32_t dw[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) dw[d] = 0;
#pragma unroll
    for (int k = 0; k < BW; ++k) {
      const int64_t j = dlo + k;
      int32_t h = kNeg;
      uint32_t c = 0;
      if (j == 0) h = 0;
      else if (j > 0) {
        h = -(o + (int32_t)(j - 1) * e);
        c = row0_code(j, o, e);
      }
      H[k] = h;
      F[k] = kNeg;
      dw[k >> 3] |= c << (4 * (7 - (k & 7)));
    }
#pragma unroll
    for (int d = 0; d < ND; ++d) dir[(int64_t)d * 64 + lane] = dw[d];
  }
  int32_t hend = kNeg;
  const int64_t kend = w - m - dlo;
  // Rows go in blocks of UB: the query symbols and the window's next
  // reference bytes of block b+1 are requested while block b is computed.
  // The loads are unconditional (indices clamped into the sequences), so
  // they land straight in their registers; values outside the pair are
  // masked when decoded.
  constexpr int UB = BW <= 16 ? 8 : (BW <= 32 ? 4 : 2);
  // row and column arithmetic in 32 bits (pairs of this path are far
  // shorter than 2^31), so that clamps are single instructions
  const int32_t mq32 = (int32_t)mq, wr32 = (int32_t)wr, dlo32 = (int32_t)dlo;
  const int32_t m32 = (int32_t)m, w32 = (int32_t)w, rows32 = (int32_t)tk.rows;
  auto load_block = [&](int32_t i0, int32_t (&qo)[UB], int32_t (&no)[UB]) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      int32_t x = i0 + u - 1;                       // query index of row i0 + u
      x = x < 0 ? 0 : (x > mq32 - 1 ? mq32 - 1 : x);
      qo[u] = qq[x];
      int32_t y = i0 + u + dlo32 + 4 * NW - 1;   // reference index of the window's new column
      y = y < 0 ? 0 : (y > wr32 - 1 ? wr32 - 1 : y);
      no[u] = rr[y];
    }
  };
  int32_t qraw[UB], nraw[UB];
  load_block(1, qraw, nraw);
  for (int32_t i0 = 1; i0 <= rows32; i0 += UB) {
    uint32_t qb[UB], nbb[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int32_t i = i0 + u;
      const int32_t c = (live && i <= m32) ? qraw[u] : -1;
      qb[u] = (c >= 0 && c < a.n) ? (uint32_t)c : 0xFFu;
      const int32_t j = i + 1 + dlo32 + 4 * NW - 1;   // 1-based column entering the window
      const int32_t cr = (live && j >= 1 && j <= w32) ? nraw[u] : 0;
      const uint32_t v = (cr >= 0 && cr < a.n) ? (uint32_t)cr : 0u;   // a bad code never indexes a table
      nbb[u] = LUT4 ? v * 8u : v;
    }
    load_block(i0 + UB, qraw, nraw);
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int32_t i = i0 + u;
      if (i > rows32) break;
      int32_t lut = 0, qrow = 0;
      if (qb[u] != 0xFFu) {
        if (LUT4) lut = (int32_t)s_lut4[qb[u]];
        else qrow = (int32_t)qb[u] * a.n;
      }
      uint32_t dw[ND];
#pragma unroll
      for (int d = 0; d < ND; ++d) dw[d] = 0;
      int32_t ev = kNeg, hleft = kNeg;
#pragma unroll
      for (int k = 0; k < BW; ++k) {
        const uint32_t sym = __builtin_amdgcn_ubfe(win[k >> 2], 8 * (k & 3), 8);
        const int32_t sc = LUT4 ? __builtin_amdgcn_sbfe(lut, sym, 8) : (int32_t)s_mat[qrow + sym];
        const int32_t hup = (k + 1 < BW) ? H[k + 1] : kNeg;
        const int32_t fup = (k + 1 < BW) ? F[k + 1] : kNeg;
        const int32_t diag = H[k] + sc;
        const int32_t fo = hup - o, fx = fup - e;
        const int32_t fij = fo > fx ? fo : fx;
        const int32_t eo = hleft - o, ex = ev - e;
        const int32_t eij = eo > ex ? eo : ex;
        int32_t h = diag > eij ? diag : eij;
        h = h > fij ? h : fij;
        dw[k >> 3] = push_code(dw[k >> 3], diag, h, eij, fij, eo, ex, fo, fx);
        H[k] = h;
        F[k] = fij;
        ev = eij;
        hleft = h;
      }
#pragma unroll
      for (int d = 0; d < ND; ++d) dir[(i * ND + d) * 64 + lane] = dw[d];
      if (live && i == m32) {
#pragma unroll
        for (int k = 0; k < BW; ++k)
          if (k == kend) hend = H[k];
      }
      // slide the reference window one column to the right
#pragma unroll
      for (int d = 0; d < NW - 1; ++d) win[d] = __builtin_amdgcn_alignbyte(win[d + 1], win[d], 1);
      win[NW - 1] = (win[NW - 1] >> 8) | (nbb[u] << 24);
    }
  }
  if (!live) return;
  if (s1 <= 0) { a.cig_len[p] = 0; return; }
  if (hend != s1 || kend < 0 || kend >= BW) a.err[p] = 1;
  // Walk from (m, w) in state H.  D moves stay in their row and every other
  // move goes up exactly one row, so a lane handles row m - t at its t-th row
  // step: the lanes step through rows together, and each lane's row codes
  // stream in kWP rows ahead, loaded at the same point of every step.  The
  // walk itself issues no global store (a store between a load and its use
  // would make the wait for that load a wait for everything): runs go to
  // this thread's LDS slots, and are written out, in CIGAR order, after the
  // walk.  A lane whose runs outgrow its slots finishes on a plain walk.
  uint32_t *out = a.cig + a.cig_off[p];
  int32_t nruns = 0;
  int32_t i = m32, j = w32;   // 32-bit walk state
  int state = 0;
  uint32_t cur_op = 3, cur_len = 0;   // 3: no run yet
  // flags as 0/1 integers: lane booleans that live across the walk loop
  // would be kept as lane masks, merged with scalar instructions per move
  uint32_t walking = 1, bad = 0, full = 0;
  uint32_t pend = 0;
  // (a masked OR rather than a select chain, which the compiler would turn
  // into an indexed load from a private copy of the ring)
  auto code_at = [&](const uint32_t (&rc)[ND], int32_t k) -> uint32_t {
    const uint32_t idx = (uint32_t)(k >> 3);
    uint32_t word = 0;
#pragma unroll
    for (int d = 0; d < ND; ++d) word |= rc[d] & (0u - (uint32_t)(idx == (uint32_t)d));
    return (word >> (4 * (7 - (k & 7)))) & 0xFu;
  };
  // one move of the state machine from code c; returns the op (0xFF: none)
  auto move = [&](uint32_t c, bool &up) -> uint32_t {
    uint32_t op = 0xFF;
    up = false;
    if (state == 0) {
      const uint32_t src = code_src(c);
      if (src == 0 && i > 0 && j > 0) { op = 0; --i; --j; up = true; }
      else if (src == 1) state = 1;
      else state = 2;
    } else if (state == 1) {
      op = 2;
      state = (c & kCodeEExt) ? 1 : 0;
      --j;
    } else {
      op = 1;
      state = (c & kCodeFExt) ? 2 : 0;
      --i;
      up = true;
    }
    return op;
  };
  constexpr int kWP = 8;
  uint32_t ring[kWP][ND];
  // rows above row 0 are never walked: their slots load row 0, so that every
  // load lands straight in its ring registers
  auto load_row = [&](int32_t row, uint32_t (&dst)[ND]) {
    const int32_t rr = row >= 0 ? row : 0;
#pragma unroll
    for (int d = 0; d < ND; ++d) dst[d] = dir[(rr * ND + d) * 64 + lane];
  };
#pragma unroll
  for (int u = 0; u < kWP; ++u) load_row(m - u, ring[u]);
  for (int32_t t0 = 0; t0 <= m32 && walking; t0 += kWP) {
#pragma unroll
    for (int u = 0; u < kWP; ++u) {   // no early exit: every step issues the same loads
      const int32_t row = m32 - (t0 + u);
      // the moves inside this row: D moves, then one M or I out of it.  One
      // move per iteration, in lane arithmetic rather than branches (the lanes
      // of a wave sit in different states): the move comes from walk_moves, the
      // run bookkeeping from 0/1 integers, and the finished run is stored
      // unconditionally into the next free slot (slot kRunSlots takes the
      // stores that end no run).
      for (int g = 0; g < 2 * BW + 4 && row >= 0 && walking; ++g) {
        const int32_t k = j - i - dlo32;
        const uint32_t ok = (uint32_t)(((k | (BW - 1 - k)) >= 0) & (i == row));
        const uint32_t c = code_at(ring[u], k);   // k out of range matches no word
        const uint64_t moves = state == 0 ? kMovesH : (state == 1 ? kMovesE : kMovesF);
        const uint32_t r = (uint32_t)(moves >> (4 * c)) & 15u;
        const uint32_t step = (r & 3u) * ok;          // 2 * (row up) + (column left)
        const uint32_t op = 3u - step;                // M 0, I 1, D 2; 3: no move
        const uint32_t moved = step != 0u;
        const uint32_t same = op == cur_op;
        const uint32_t ends = moved & (same ^ 1u) & (cur_len != 0u);
        const uint32_t run = (cur_len << 4) | cur_op;
        s_runs[nruns * 256 + threadIdx.x] = run;
        const uint32_t room = nruns < kRunSlots;
        nruns += ends & room;
        const uint32_t spill = ends & (room ^ 1u);   // no slot left: finish on the plain walk
        pend = spill ? run : pend;
        full |= spill;
        cur_len = moved ? (same ? cur_len + 1 : 1u) : cur_len;
        cur_op = moved ? op : cur_op;
        i -= (int32_t)(step >> 1);
        j -= (int32_t)(step & 1u);
        state = ok ? (int)(r >> 2) : state;
        bad |= ok ^ 1u;
        const uint32_t stop = (ok ^ 1u) | (uint32_t)((i | j) == 0) | full;
        walking &= stop ^ 1u;
        if (stop | (step >> 1)) break;   // the move went up a row
      }
      load_row(row - kWP, ring[u]);   // the slot is free again: kWP rows up
    }
  }
  if (full) {
    // the runs so far, the one that found no slot, then the rest of the walk
    for (int32_t x = 0; x < nruns; ++x) out[x] = s_runs[x * 256 + threadIdx.x];
    out[nruns++] = pend;
    int64_t guard = 2 * (m + w) + 4;
    while ((i > 0 || j > 0) && guard-- > 0) {
      const int32_t k = j - i - dlo32;
      if (k < 0 || k >= BW) { bad = true; break; }
      const uint32_t word = dir[(i * ND + (k >> 3)) * 64 + lane];
      bool up;
      const uint32_t op = move((word >> (4 * (7 - (k & 7)))) & 0xFu, up);
      if (op != 0xFF) {
        if (op == cur_op) ++cur_len;
        else {
          if (cur_len) out[nruns++] = (cur_len << 4) | cur_op;
          cur_op = op;
          cur_len = 1;
        }
      }
    }
  }
  if (bad || i != 0 || j != 0) a.err[p] = 1;
  if (full) {
    if (cur_len) out[nruns++] = (cur_len << 4) | cur_op;
    for (int32_t x = 0, y = nruns - 1; x < y; ++x, --y) {
      const uint32_t t = out[x]; out[x] = out[y]; out[y] = t;
    }
  } else {
    // runs were found end -> begin: write them reversed
    const int32_t total = nruns + (cur_len ? 1 : 0);
    if (cur_len) out[0] = (cur_len << 4) | cur_op;
    for (int32_t x = 0; x < nruns; ++x) out[total - 1 - x] = s_runs[x * 256 + threadIdx.x];
    nruns = total;
  }
  a.cig_len[p] = nruns;
}

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

hipError_t tb_classify(const TbArgs &a, int64_t npairs, uint8_t *cls, uint64_t *key, int64_t *vals,
                       int64_t *coff, int64_t *counts, int64_t *words, int64_t *bytes, hipStream_t st) {
  if (!npairs) return hipSuccess;
  // at most 8 blocks per compute unit: each adds its class counts once
  hipLaunchKernelGGL(k_tb_classify, dim3(std::min(nblk(npairs, 256), 2048u)), dim3(256), 0, st, a, npairs, cls, key,
                     vals, coff, counts, words, bytes);
  return hipGetLastError();
}

hipError_t tb_tasks(int64_t n0, int64_t n1, const int64_t *sorted, const TbArgs &a, int32_t bw,
                    TbTask *tasks, int64_t *dir_words, hipStream_t st) {
  const int64_t nt = (n1 - n0 + 63) / 64;
  if (nt <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tb_tasks, dim3(nblk(nt, 4)), dim3(256), 0, st, n0, n1,
                     (const int64_t *)nullptr, (int64_t)0, sorted, a, bw, tasks, dir_words);
  return hipGetLastError();
}

hipError_t tb_tasks_range(const int64_t *range, int64_t ntasks_cap, const int64_t *sorted,
                          const TbArgs &a, int32_t bw, TbTask *tasks, int64_t *dir_words,
                          hipStream_t st) {
  if (ntasks_cap <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tb_tasks, dim3(nblk(ntasks_cap, 4)), dim3(256), 0, st, (int64_t)0,
                     (int64_t)0, range, ntasks_cap, sorted, a, bw, tasks, dir_words);
  return hipGetLastError();
}

hipError_t tb_offsets(int64_t ntasks, TbTask *tasks, const int64_t *off, hipStream_t st) {
  if (!ntasks) return hipSuccess;
  hipLaunchKernelGGL(k_tb_offsets, dim3(nblk(ntasks, 128)), dim3(128), 0, st, ntasks, tasks, off);
  return hipGetLastError();
}

template <int BW>
static hipError_t launch_band(const TbArgs &a, const TbTask *tasks, int64_t ntasks,
                              const int64_t *sorted, bool lut4, hipStream_t st) {
  const unsigned blocks = nblk(ntasks, 4);
  if (lut4)
    hipLaunchKernelGGL((k_tb_band<BW, true>), dim3(blocks), dim3(256), 0, st, a, tasks, ntasks, sorted);
  else
    hipLaunchKernelGGL((k_tb_band<BW, false>), dim3(blocks), dim3(256), 0, st, a, tasks, ntasks, sorted);
  return hipGetLastError();
}

hipError_t tb_band(const TbArgs &a, const TbTask *tasks, int64_t ntasks, const int64_t *sorted,
                   int32_t bw, hipStream_t st) {
  if (!ntasks) return hipSuccess;
  const bool lut4 = a.n <= 4;
  switch (bw) {
    case 8: return launch_band<8>(a, tasks, ntasks, sorted, lut4, st);
    case 16: return launch_band<16>(a, tasks, ntasks, sorted, lut4, st);
    case 32: return launch_band<32>(a, tasks, ntasks, sorted, lut4, st);
    default: return hipErrorInvalidValue;
  }
}


// ---- wide bands: row strips over four lanes, columns swept left to right ---
// A task holds kTbwSlots pairs; four consecutive lanes share one pair.  The
// task's strip s covers rows sR+1 .. sR+R (R = 16, 1-based, row 0 is the
// virtual row before the begin) and columns [clo(s), chi(s)): the unclipped
// window starts at c0(s) = sR + 1 + dlo_min and is W = R + (width of the union
// of the task's bands) columns wide, clipped to [0, wmax], so every pair
// computes a superset of its own safe band.  Lane g of a pair holds rows
// sR+4g+1 .. sR+4g+4 and at step t computes column clo + t - g: the H and F of
// its last row reach lane g+1 through a one-lane DPP shift, one step later,
// as the row above.  H and F of a strip's last row are handed to the next
// strip through global memory.  Lane g's four choice codes of step t (16 bits)
// are stored as half t & 1 of dword [s][t >> 1][g][slot], so that each store
// covers the whole wave with one 256-byte write.
namespace {
constexpr int kStripR = 16;                     // rows per strip
constexpr int kStripLP = 4;                     // lanes per pair
constexpr int kStripRL = kStripR / kStripLP;    // rows per lane
static_assert(kTbwSlots * kStripLP == 64, "one task per wave");

// columns of strip s and the code dwords a strip holds per (lane, slot)
__device__ __forceinline__ void strip_window(int64_t s, const TbwTask &tk, int64_t *clo,
                                             int64_t *chi) {
  const int64_t cstart = s * kStripR + 1 + tk.dlo;
  int64_t lo = cstart > 0 ? cstart : 0;
  int64_t hi = cstart + tk.width;
  if (hi > tk.wmax + 1) hi = tk.wmax + 1;
  *clo = lo;
  *chi = hi > lo ? hi : lo;
}
// lane k of each quad of lanes, to the whole quad (k a constant after unrolling)
__device__ __forceinline__ int32_t quad_bcast(int32_t x, int k) {
  switch (k) {
    // every source lane exists: no old value to keep
    case 0: return __builtin_amdgcn_mov_dpp(x, 0x00, 0xF, 0xF, true);
    case 1: return __builtin_amdgcn_mov_dpp(x, 0x55, 0xF, 0xF, true);
    case 2: return __builtin_amdgcn_mov_dpp(x, 0xAA, 0xF, 0xF, true);
    default: return __builtin_amdgcn_mov_dpp(x, 0xFF, 0xF, 0xF, true);
  }
}
__host__ __device__ __forceinline__ int64_t strip_dwords(int64_t width) {
  return (width + kStripLP) / 2;   // steps: at most width + kStripLP - 1
}
}  // namespace

__global__ void k_tbw_tasks(int64_t n0, int64_t n1, const int64_t *range, int64_t ntasks_cap,
                            const int64_t *sorted, const TbArgs a, TbwTask *tasks,
                            int64_t *dir_words, int64_t *bnd_words) {
  // one wave per task, one lane per slot
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (range) { n0 = range[0]; n1 = range[1]; }
  const int64_t ntasks = (n1 - n0 + kTbwSlots - 1) / kTbwSlots;
  if (t >= (range ? ntasks_cap : ntasks)) return;
  if (t >= ntasks) {
    if (lane == 0) {
      tasks[t] = TbwTask{};
      dir_words[t] = 0;
      bnd_words[t] = 0;
    }
    return;
  }
  const int64_t s0 = n0 + t * kTbwSlots;
  const int64_t s1 = (s0 + kTbwSlots < n1) ? s0 + kTbwSlots : n1;
  int64_t rows = 1, wmax = 1, ndlo_max = 0, dhi_max = 0;   // ndlo: -dlo, so all four are maxima
  if (lane < kTbwSlots && s0 + lane < s1) {
    const int64_t p = sorted[s0 + lane];
    const int64_t m = a.qend[p] - a.qbeg[p] + 1, w = a.rend[p] - a.rbeg[p] + 1;
    int64_t dlo, bw;
    safe_band(m, w, a.score[p], a.smax, a.o, a.e, &dlo, &bw);
    rows = m > rows ? m : rows;
    wmax = w > wmax ? w : wmax;
    ndlo_max = -dlo > ndlo_max ? -dlo : ndlo_max;
    dhi_max = (dlo + bw - 1) > dhi_max ? (dlo + bw - 1) : dhi_max;
  }
  rows = wave_max_i64(rows);
  wmax = wave_max_i64(wmax);
  const int64_t dlo_min = -wave_max_i64(ndlo_max);
  dhi_max = wave_max_i64(dhi_max);
  if (lane != 0) return;
  TbwTask tk{};
  tk.nslots = (int32_t)(s1 - s0);
  tk.rows = rows;
  tk.wmax = wmax;
  tk.dlo = dlo_min;
  tk.width = kStripR + (dhi_max - dlo_min + 1);
  tk.slot_base = s0;
  tasks[t] = tk;
  const int64_t nstrips = (rows + kStripR - 1) / kStripR;
  dir_words[t] = nstrips * strip_dwords(tk.width) * 64;
  bnd_words[t] = 2 * (wmax + 1) * kTbwSlots;
}

__global__ void k_tbw_offsets(int64_t ntasks, TbwTask *tasks, const int64_t *doff,
                              const int64_t *boff) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < ntasks) { tasks[t].dir_off = doff[t]; tasks[t].bnd_off = boff[t]; }
}

template <bool LUT4>
__global__ __launch_bounds__(256) void k_tb_strip(TbArgs a, const TbwTask *tasks, int64_t ntasks,
                                                  const int64_t *sorted, int32_t *bndbuf) {
  constexpr int LP = kStripLP, RL = kStripRL, NS = kTbwSlots;
  constexpr int kCU = 16;   // walk cache: code dwords (32 steps) per lane
  __shared__ int8_t s_mat[32 * 32];
  __shared__ uint32_t s_walk[4 * 64 * kCU];
  for (int k = threadIdx.x; k < a.n * a.n; k += blockDim.x) s_mat[k] = a.matrix[k];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int g = lane & (LP - 1);        // row group of this lane
  const int slot = lane / LP;           // pair slot of the task
  // tasks are sorted by rows and band, ascending: the largest go first
  const int64_t k_ = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (k_ >= ntasks) return;
  const int64_t tid = ntasks - 1 - k_;
  const TbwTask tk = tasks[tid];
  if (tk.nslots == 0) return;
  const bool live = slot < tk.nslots;
  const int64_t p = live ? sorted[tk.slot_base + slot] : -1;
  int64_t m = 1, w = 1, dlo = 0, bwl = 1;
  int32_t s1 = 0;
  const int8_t *q = a.qcat, *r = a.rcat;
  if (live) {
    s1 = a.score[p];
    m = a.qend[p] - a.qbeg[p] + 1;
    w = a.rend[p] - a.rbeg[p] + 1;
    safe_band(m, w, s1, a.smax, a.o, a.e, &dlo, &bwl);
    q = a.qcat + a.qstart[p] + a.qbeg[p];
    r = a.rcat + a.rstart[p] + a.rbeg[p];
  }
  const int32_t o = a.o, e = a.e;
  uint32_t *dir = a.dir + tk.dir_off;
  int32_t *bH = bndbuf + tk.bnd_off;
  int32_t *bF = bH + (tk.wmax + 1) * NS;
  const int64_t SW = strip_dwords(tk.width);
  // row 0 (virtual): H(0,0) = 0, H(0,j) = -(o + (j-1)e), F = -inf; the walk
  // decodes row 0 itself, so it has no stored codes
  for (int64_t j = g; j <= tk.wmax; j += LP) {
    bH[j * NS + slot] = (j == 0) ? 0 : -(o + (int32_t)(j - 1) * e);
    bF[j * NS + slot] = kNeg;
  }
  const int64_t nstrips = (tk.rows + kStripR - 1) / kStripR;
  int32_t plo = 0, phi = (int32_t)tk.wmax + 1;   // columns of row sR that hold valid values
  const int8_t *rr = live ? r : (const int8_t *)a.matrix;   // readable bytes for empty slots
  const int8_t *qq = live ? q : (const int8_t *)a.matrix;
  const int64_t mq = live ? m : 1;
  for (int64_t s = 0; s < nstrips; ++s) {
    const int64_t sR = s * kStripR;
    int64_t clo64, chi64;
    strip_window(s, tk, &clo64, &chi64);
    // 32-bit column and step arithmetic (a strip task spans well under 2^31
    // code dwords), so that the block's addresses stay in few registers
    const int32_t clo = (int32_t)clo64, chi = (int32_t)chi64;
    const int32_t ncol = chi - clo;
    const int32_t nsteps = ncol + LP - 1;
    const int32_t wmax = (int32_t)tk.wmax, wl = (int32_t)w;
    uint32_t *sdir = dir + s * SW * 64;
    // this lane's rows: score tables
    int32_t lut[RL], qn[RL], qraw[RL];
#pragma unroll
    for (int k = 0; k < RL; ++k) {   // all loads first (clamped), then decode
      int64_t x = sR + g * RL + k;
      x = x > mq - 1 ? mq - 1 : x;
      qraw[k] = qq[x];
    }
#pragma unroll
    for (int k = 0; k < RL; ++k) {
      const int64_t i = sR + g * RL + 1 + k;
      lut[k] = 0;
      qn[k] = 0;
      const int32_t qs = (live && i <= m) ? qraw[k] : -1;
      if (qs >= 0 && qs < a.n) {   // a bad code never indexes a table
        if (LUT4) {
          uint32_t l = 0;
          for (int b = 0; b < a.n; ++b) l |= (uint32_t)(uint8_t)s_mat[qs * a.n + b] << (8 * b);
          lut[k] = (int32_t)l;
        } else {
          qn[k] = qs * a.n;
        }
      }
    }
    int32_t H[RL], E[RL], HO[RL];   // HO = H - o: the E opening of the next column
#pragma unroll
    for (int k = 0; k < RL; ++k) { H[k] = kNeg; E[k] = kNeg; HO[k] = kNeg - o; }
    // H of the row above at the previous column (lane 0: row sR at clo - 1)
    int32_t hdiag0 = kNeg;
    if (g == 0 && clo >= 1 && clo - 1 >= plo && clo - 1 < phi) hdiag0 = bH[(clo - 1) * NS + slot];
    int32_t xh = kNeg, xf = kNeg;   // last row's H, F of the previous step
    uint32_t xs = 0;                // reference symbol of the previous step
    // Steps go in blocks of kPB.  Lane 0 of a pair consumes the row above and
    // the reference symbol of its column; the pair's four lanes load them, a
    // quarter each, and hand them over by a DPP broadcast inside the lane
    // quad (the other lanes take theirs from the lane before).  The strip's
    // last row goes the other way: lane 3 broadcasts it and the lanes keep
    // a quarter each for the boundary stores.  At the top of a block the wave
    // waits for the block's operands (requested one block earlier), then
    // stores the previous block's codes and boundary values and requests the
    // next block's operands, and only then computes.
    constexpr int kPB = 4;   // (8 leaves three waves per SIMD, 4 leaves four)
    constexpr int kPV = kPB / LP;   // columns per lane and block
    int32_t n_h[kPV], n_f[kPV], n_c[kPV];
    // lane g loads columns clo + t0 + g + LP * v of the block
    auto fetch_block = [&](int32_t t0) {
#pragma unroll
      for (int v = 0; v < kPV; ++v) {
        int32_t j = clo + t0 + g + LP * v;
        j = j < 0 ? 0 : (j > wmax ? wmax : j);
        n_h[v] = bH[j * NS + slot];
        n_f[v] = bF[j * NS + slot];
        int32_t x = clo + t0 + g + LP * v - 1;
        x = x < 0 ? 0 : (x > wl - 1 ? wl - 1 : x);
        n_c[v] = (int32_t)rr[x];
      }
    };
    uint32_t p_code[kPB / 2];
    int32_t p_h[kPV], p_f[kPV];   // last row of step g + LP * v of the pending block
    int32_t p_t0 = -1;   // first step of the pending block (-1: none)
    auto flush = [&]() {
      if (p_t0 < 0) return;
#pragma unroll
      for (int u = 0; u < kPB / 2; ++u)
        if (p_t0 + 2 * u < nsteps) sdir[((p_t0 >> 1) + u) * 64 + lane] = p_code[u];
#pragma unroll
      for (int v = 0; v < kPV; ++v) {
        const int32_t t = p_t0 + g + LP * v, j = clo + t - (LP - 1);
        if (t >= LP - 1 && t < nsteps) {
          bH[j * NS + slot] = p_h[v];
          bF[j * NS + slot] = p_f[v];
        }
      }
    };
    fetch_block(0);
    for (int32_t t0 = 0; t0 < nsteps; t0 += kPB) {
      int32_t c_h[kPV], c_f[kPV];
      int32_t c_sy[kPV];
#pragma unroll
      for (int v = 0; v < kPV; ++v) {
        const int32_t j = clo + t0 + g + LP * v;
        const bool inprev = j >= plo && j < phi;
        c_h[v] = inprev ? n_h[v] : kNeg;
        c_f[v] = inprev ? n_f[v] : kNeg;
        const int32_t c = (live && j >= 1 && j <= wl) ? n_c[v] : -1;
        c_sy[v] = (c >= 0 && c < a.n) ? c : 0;
      }
      // the operands are consumed (waited for) before any store is issued
      __builtin_amdgcn_sched_barrier(0);
      flush();
      fetch_block(t0 + kPB);   // past the window too: clamped, and never used
      uint32_t acc = 0;
#pragma unroll
      for (int u = 0; u < kPB; ++u) {
        const int32_t t = t0 + u;
        // lane 0's operands: from lane u % 4 of the quad
        const int32_t bh = quad_bcast(c_h[u / LP], u & (LP - 1));
        const int32_t bf = quad_bcast(c_f[u / LP], u & (LP - 1));
        const int32_t bs = quad_bcast(c_sy[u / LP], u & (LP - 1));
        // the other lanes': from the lane before (its last row, one step earlier)
        // (lane 0 of each row of 16 has no source and reads 0; it is a
        // pair's lane 0, which takes the loaded operands instead)
        const int32_t dh = __builtin_amdgcn_mov_dpp(xh, 0x111, 0xF, 0xF, true);
        const int32_t df = __builtin_amdgcn_mov_dpp(xf, 0x111, 0xF, 0xF, true);
        const int32_t ds = __builtin_amdgcn_mov_dpp((int32_t)xs, 0x111, 0xF, 0xF, true);
        const int32_t hup0 = g == 0 ? bh : dh;
        const int32_t fup0 = g == 0 ? bf : df;
        const uint32_t sym = (uint32_t)(g == 0 ? bs : ds);
        uint32_t code = 0;
        if (t >= g && t < g + ncol) {
          const uint32_t sym8 = LUT4 ? sym * 8u : sym;
          int32_t hdiag = hdiag0;
          hdiag0 = hup0;
          int32_t hupo = hup0 - o, fup = fup0;   // hupo: H of the row above, minus o
#pragma unroll
          for (int k = 0; k < RL; ++k) {
            const int32_t sc = LUT4 ? __builtin_amdgcn_sbfe(lut[k], sym8, 8) : (int32_t)s_mat[qn[k] + sym];
            const int32_t diag = hdiag + sc;
            const int32_t fo = hupo, fx = fup - e;
            const int32_t fij = fo > fx ? fo : fx;
            const int32_t eo = HO[k], ex = E[k] - e;      // row k at column j-1
            const int32_t eij = eo > ex ? eo : ex;
            int32_t h = diag > eij ? diag : eij;
            h = h > fij ? h : fij;
            code = push_code(code, diag, h, eij, fij, eo, ex, fo, fx);   // row k: bits 4(RL-1-k)
            hdiag = H[k];
            H[k] = h;
            E[k] = eij;
            hupo = h - o;
            HO[k] = hupo;
            fup = fij;
          }
          const int32_t hup = H[RL - 1];
          xh = hup;
          xf = fup;
        }
        xs = sym;
        // lane 3's last row, kept by lane u % 4
        const int32_t lh = quad_bcast(xh, LP - 1);
        const int32_t lf = quad_bcast(xf, LP - 1);
        if (g == (u & (LP - 1))) {
          p_h[u / LP] = lh;
          p_f[u / LP] = lf;
        }
        acc |= code << (16 * (u & 1));
        if (u & 1) {
          p_code[u >> 1] = acc;
          acc = 0;
        }
      }
      p_t0 = t0;
    }
    flush();   // the strip's last block, before the next strip reads it
    plo = clo;
    phi = chi;
  }
  if (!live) return;
  if (s1 <= 0) {
    if (g == 0) a.cig_len[p] = 0;
    return;
  }
  // Traceback from (m, w) in state H.  The four lanes of a pair walk it
  // together.  Each lane keeps kCU code dwords of its own row group of the
  // current strip in the pair's LDS slots (a window of columns ending at the
  // column where it was filled; the walk only moves up and left).  On entering
  // a strip the lanes also request the strip above, ending at the current
  // column, into registers: when the walk gets there, the window is written
  // to LDS from those registers without waiting for memory.  Only a walk
  // that leaves a window sideways waits for a load.
  uint32_t *out = a.cig + a.cig_off[p];
  int32_t nruns = 0;
  // (32-bit walk state: a strip task spans well under 2^31 code dwords)
  int32_t i = (int32_t)m, j = (int32_t)w;
  int state = 0;
  uint32_t cur_op = 3, cur_len = 0;   // 3: no run yet
  int64_t guard = 2 * (m + w) + 4;
  uint32_t *cache = s_walk + ((threadIdx.x >> 6) * 64 + slot * LP) * kCU;   // [g][kCU]
  int32_t cache_s = -1, cache_j = -1;
  uint32_t pfx[kCU];              // the strip above, in flight
  int32_t pf_s = -1, pf_j = -1;
  const int32_t SW32 = (int32_t)SW, dlo32 = (int32_t)tk.dlo, width32 = (int32_t)tk.width;
  const int32_t wmax32 = (int32_t)tk.wmax;
  auto window32 = [&](int32_t s, int32_t &clo, int32_t &chi) {   // strip_window in 32 bits
    const int32_t cstart = s * kStripR + 1 + dlo32;
    clo = cstart > 0 ? cstart : 0;
    int32_t hi = cstart + width32;
    hi = hi > wmax32 + 1 ? wmax32 + 1 : hi;
    chi = hi > clo ? hi : clo;
  };
  auto fetch_window = [&](int32_t s, int32_t jj, uint32_t (&dst)[kCU]) {
    int32_t clo, chi;
    window32(s, clo, chi);
    const int32_t mytop = (jj - clo + g) >> 1;
#pragma unroll
    for (int x = 0; x < kCU; ++x) {
      int32_t uu = mytop - x;
      uu = uu < 0 ? 0 : (uu > SW32 - 1 ? SW32 - 1 : uu);   // clamped: never read outside the strip
      dst[x] = dir[(s * SW32 + uu) * 64 + slot * LP + g];
    }
  };
  bool bad = false;
  while ((i > 0 || j > 0) && guard-- > 0) {
    uint32_t c;
    if (i == 0) {
      c = row0_code(j, o, e);
    } else {
      const int32_t s = (i - 1) / kStripR, k = (i - 1) % kStripR;
      const int32_t gk = k / RL;
      int32_t clo, chi;
      window32(s, clo, chi);
      if (j < clo || j >= chi) { bad = true; break; }
      const int32_t t = j - clo + gk;
      // cached: dwords (cache_j - clo + g) / 2 - kCU + 1 .. (cache_j - clo + g) / 2 of row group g
      const int32_t top = (cache_j - clo + gk) >> 1;
      if (s != cache_s || (t >> 1) > top || (t >> 1) <= top - kCU) {
        const int32_t ptop = (pf_j - clo + gk) >> 1;
        const bool use_pf = s == pf_s && (t >> 1) <= ptop && (t >> 1) > ptop - kCU;
        if (use_pf) {
#pragma unroll
          for (int x = 0; x < kCU; ++x) cache[g * kCU + x] = pfx[x];
          cache_j = pf_j;
        } else {
          uint32_t now[kCU];
          fetch_window(s, j, now);
#pragma unroll
          for (int x = 0; x < kCU; ++x) cache[g * kCU + x] = now[x];
          cache_j = j;
        }
        if (s != cache_s && s > 0) {   // a new strip: request the one above
          fetch_window(s - 1, j, pfx);
          pf_s = s - 1;
          pf_j = j;
        }
        cache_s = s;
      }
      const int32_t top2 = (cache_j - clo + gk) >> 1;
      const uint32_t dwv = cache[gk * kCU + (top2 - (t >> 1))];
      c = (dwv >> (16 * (t & 1) + 4 * (RL - 1 - k % RL))) & 0xFu;
    }
    // the move from the per-state table (M 0, I 1, D 2; 3: a change of state)
    const uint64_t moves = state == 0 ? kMovesH : (state == 1 ? kMovesE : kMovesF);
    const uint32_t r = (uint32_t)(moves >> (4 * c)) & 15u;
    const uint32_t step = r & 3u, op = 3u - step;
    i -= (int32_t)(step >> 1);
    j -= (int32_t)(step & 1u);
    state = (int)(r >> 2);
    if (step) {
      if (op == cur_op) ++cur_len;
      else {
        if (cur_len && g == 0) out[nruns] = (cur_len << 4) | cur_op;
        if (cur_len) ++nruns;
        cur_op = op;
        cur_len = 1;
      }
    }
  }
  if (g != 0) return;
  if (bad || i != 0 || j != 0) a.err[p] = 1;
  if (cur_len) out[nruns++] = (cur_len << 4) | cur_op;
  for (int32_t x = 0, y = nruns - 1; x < y; ++x, --y) {
    const uint32_t t = out[x]; out[x] = out[y]; out[y] = t;
  }
  a.cig_len[p] = nruns;
}

// ---- wave-parallel traceback (long pairs with wide bands) -------------------
// One pair per workgroup.  Lane k holds rows [k*RL+1, (k+1)*RL] of a strip of
// 64*RL rows and computes column c - k at step c; the H and F leaving a lane's
// last row move one lane down per step through a DPP shift, as in the
// intra-sequence fill.  Each step stores the lane's RL choice codes (same
// 4-bit code as the per-lane kernels, RL/2 bytes) at [step][lane], so a
// strip's codes are written with coalesced stores.  The walk then runs on the
// whole wave with uniform state, copying the codes of up to 32 KiB of steps
// at a time (a contiguous range: steps [t - TS + 1, t] of the current strip)
// into LDS with 16-byte loads: the walk only moves to smaller steps and lanes
// inside a strip, so each copy serves many moves.  RL is chosen per pair on
// the host: short lanes shorten the chain of strips and the work per step,
// tall ones hold longer queries within the strip limit.
__device__ __forceinline__ int32_t tb_from_above(int32_t src, int32_t top) {
  return __builtin_amdgcn_update_dpp(top, src, 0x138, 0xF, 0xF, false);   // wave_shr:1
}

// vec moved one lane down with lane 63 taking its own v
__device__ __forceinline__ int32_t tb_shift_in(int32_t vec, int32_t v) {
  return __builtin_amdgcn_update_dpp(v, vec, 0x130, 0xF, 0xF, false);   // wave_shl:1
}

constexpr int kTbMaxStrips = (int)kTbMaxStripsDecl;
constexpr int kTbMaxWaves = 8;
constexpr int64_t kTbSpinLimit = int64_t(1) << 26;
constexpr int kTbTileBytes = 32768;

// RL score bytes of the LDS profile in words
constexpr int tb_prof_words(int RL) { return RL >= 4 ? RL / 4 : 1; }
template <int RL>
__device__ __forceinline__ void tb_prof_load(const int8_t *src, uint32_t (&w)[tb_prof_words(RL)]) {
  if constexpr (RL == 16) {
    const uint4 v = *reinterpret_cast<const uint4 *>(src);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else if constexpr (RL == 8) {
    const uint2 v = *reinterpret_cast<const uint2 *>(src);
    w[0] = v.x; w[1] = v.y;
  } else if constexpr (RL == 4) {
    w[0] = *reinterpret_cast<const uint32_t *>(src);
  } else {
    w[0] = *reinterpret_cast<const uint16_t *>(src);
  }
}

// The walk back along the path (rule T3) over one pair's stored codes, by
// one wave (uniform state), TILE bytes of codes at a time; defined below.
template <int RL, int TILE>
__device__ void tb_wave_walk(const TbArgs &a, const TbWaveJob &jb, const uint8_t *dir,
                             uint4 *s_tile, int lane);

// The choice codes of one pair, its strips on the waves of one workgroup.
// s_profs: the workgroup's profiles, [(n+1)][64][RL] score bytes per wave;
// s_mat: room for the matrix; s_prog, s_done: progress per strip.
template <int RL>
__device__ __forceinline__ void tb_wave_fill(const TbArgs &a, const TbWaveJob &jb, int32_t *s_prog,
                                             int32_t *s_done, int8_t *s_mat, int8_t *s_profs,
                                             uint8_t *dir, int32_t *bnd0) {
  constexpr int64_t SH = 64 * RL;
  constexpr int WB = RL / 2;                      // code bytes per lane and step
  constexpr int SCOPE = __HIP_MEMORY_SCOPE_WORKGROUP;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int NW = blockDim.x >> 6;
  const int64_t p = jb.pair, m = jb.m, w = jb.w;
  const int n = a.n;
  const int32_t o = a.o, e = a.e;
  const int64_t nstrips = (m + SH - 1) / SH;
  for (int k = threadIdx.x; k < n * n; k += blockDim.x) s_mat[k] = a.matrix[k];
  for (int k = threadIdx.x; k < nstrips && k < kTbMaxStrips; k += blockDim.x) {
    s_prog[k] = 0;
    s_done[k] = 0;
  }
  const int8_t *q = a.qcat + a.qstart[p] + a.qbeg[p];
  const int8_t *r = a.rcat + a.rstart[p] + a.rbeg[p];
  // hand-over rows: row 0 is the virtual top row H(0,0) = 0,
  // H(0,j) = -(o + (j-1)e), F(0,j) = -inf; row s + 1 is strip s's last row
  for (int64_t j = threadIdx.x; j <= w; j += blockDim.x) {   // strip 0 reads it after the barrier below
    bnd0[j] = (j == 0) ? 0 : -(o + (int32_t)(j - 1) * e);
    bnd0[(w + 1) + j] = kNeg;
  }
  __threadfence_block();
  __syncthreads();
  int8_t *s_prof = s_profs + (size_t)wave * (n + 1) * 64 * RL;
  bool spin_fail = false;

  // choice codes of strip s start this many bytes after those of strip 0
  auto strip_base = [&](int64_t s) {
    int64_t off = 0;
    for (int64_t k = 0; k < s; ++k) {
      int64_t lo, hi;
      tbw_window(k, SH, jb.dlo, jb.bw, w, &lo, &hi);
      off += ((hi - lo) + 63) * 64 * WB;
    }
    return off;
  };

  for (int64_t s = wave; s < nstrips; s += NW) {
    int64_t clo, chi, plo = 0, phi = w + 1;
    tbw_window(s, SH, jb.dlo, jb.bw, w, &clo, &chi);
    if (s > 0) tbw_window(s - 1, SH, jb.dlo, jb.bw, w, &plo, &phi);
    const int32_t *inH = bnd0 + 2 * (w + 1) * s;    // the row above this strip
    const int32_t *inF = inH + (w + 1);
    int32_t *outH = bnd0 + 2 * (w + 1) * (s + 1);   // this strip's last row
    int32_t *outF = outH + (w + 1);
    const bool hand_over = (s + 1 < nstrips);
    uint8_t *dstrip = dir + strip_base(s);
    auto publish = [&](int32_t ncols, bool fin) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0) {
        __hip_atomic_store(&s_prog[s], ncols, __ATOMIC_RELAXED, SCOPE);
        if (fin) __hip_atomic_store(&s_done[s], 1, __ATOMIC_RELAXED, SCOPE);
      }
    };
    int32_t avail = (s == 0) ? (int32_t)(w + 1) : 0;
    auto wait_for = [&](int32_t need) {
      if (s == 0) return;
      int64_t spins = 0;
      for (;;) {
        const int32_t done = __hip_atomic_load(&s_done[s - 1], __ATOMIC_RELAXED, SCOPE);
        avail = __hip_atomic_load(&s_prog[s - 1], __ATOMIC_RELAXED, SCOPE);
        if (done || avail >= need) break;
        if (++spins > kTbSpinLimit) { spin_fail = true; break; }
        __builtin_amdgcn_s_sleep(2);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    auto rd = [](const int32_t *ptr) {   // past the L1: another wave wrote it
      return __hip_atomic_load(ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // profile of this lane's rows (signed scores; padding rows score 0)
    {
      int32_t qv[RL];
#pragma unroll
      for (int k = 0; k < RL; ++k) {
        const int64_t i = s * SH + lane * RL + k + 1;
        qv[k] = (i <= m) ? (int32_t)q[i - 1] : -1;
      }
      for (int sy = 0; sy <= n; ++sy) {
        uint32_t wv[RL / 4];
#pragma unroll
        for (int k = 0; k < RL / 4; ++k) wv[k] = 0u;
#pragma unroll
        for (int k = 0; k < RL; ++k) {
          const uint32_t b = (qv[k] >= 0 && sy < n) ? (uint32_t)(uint8_t)s_mat[qv[k] * n + sy] : 0u;
          wv[k >> 2] |= b << (8 * (k & 3));
        }
        uint32_t *dst = reinterpret_cast<uint32_t *>(s_prof + ((int64_t)sy * 64 + lane) * RL);
#pragma unroll
        for (int k = 0; k < RL / 4; ++k) dst[k] = wv[k];
      }
    }
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    int32_t H[RL], E[RL];
#pragma unroll
    for (int k = 0; k < RL; ++k) { H[k] = kNeg; E[k] = kNeg; }
    int32_t hup_prev = kNeg;
    if (clo >= 1 && clo - 1 >= plo && clo - 1 < phi) {
      wait_for((int32_t)(clo - plo));
      if (lane == 0 && clo - 1 < plo + avail) hup_prev = rd(&inH[clo - 1]);
    }
    int32_t hout = kNeg, fout = kNeg;
    int32_t hbuf = kNeg, fbuf = kNeg;
    int32_t obH = 0, obF = 0;
    // the last strip ends once the lane that holds the last row has swept
    // the window (nothing leaves lane 63)
    const int64_t nsteps = (chi - clo) + (hand_over ? 63 : (m - s * SH + RL - 1) / RL - 1);
    // reference symbols of columns [c0, c0 + 64) at lane c - c0; the profile
    // row of a step is read one step ahead (its symbol is the one the lane
    // above holds now)
    auto symbols = [&](int64_t c0) -> int32_t {
      const int64_t c = c0 + lane;
      return (c < chi && c >= 1) ? (int32_t)(uint8_t)r[c - 1] : n;
    };
    int32_t symbuf = symbols(clo), symnext = symbols(clo + 64);
    uint32_t sym = (uint32_t)tb_from_above(n, __builtin_amdgcn_readlane(symbuf, 0));
    uint32_t X[RL / 4];
    tb_prof_load<RL>(s_prof + ((int64_t)sym * 64 + lane) * RL, X);
    // Steps in blocks of 64: the block's start reads the symbols and the row
    // above for its 64 columns; step t gathers lane 63's H and F of column
    // clo + t - 63 into lane (t - 63) mod 64 (from step 63 on), and step 62
    // of every block after the first completes 64 such columns.
#pragma unroll 1
    for (int64_t t0 = 0; t0 < nsteps; t0 += 64) {
      if (t0 > 0) {
        symbuf = symnext;
        symnext = symbols(clo + t0 + 64);
      }
      {
        const int64_t cend = (clo + t0 + 64 < phi) ? clo + t0 + 64 : phi;
        if (cend > plo) wait_for((int32_t)(cend - plo));
        const int64_t c = clo + t0 + lane;
        const bool prev = c < chi && c >= plo && c < phi && c < plo + avail;
        hbuf = prev ? rd(&inH[c]) : kNeg;
        fbuf = prev ? rd(&inF[c]) : kNeg;
      }
      // step t0 + tm; the next step's symbol is lane `nl` of `nsym`; gather:
      // the step has a column to hand over (t >= 63)
      auto step = [&](int tm, int32_t nsym, int nl, bool gather) {
        const int64_t t = t0 + tm;
        const int32_t hup = tb_from_above(hout, __builtin_amdgcn_readlane(hbuf, tm));
        int32_t fup = tb_from_above(fout, __builtin_amdgcn_readlane(fbuf, tm));
        const uint32_t symn = (uint32_t)tb_from_above((int32_t)sym, __builtin_amdgcn_readlane(nsym, nl));
        uint32_t Xn[RL / 4];
        tb_prof_load<RL>(s_prof + ((int64_t)symn * 64 + lane) * RL, Xn);
        int32_t hdiag = hup_prev;
        int32_t hcur = hup;
        uint32_t dw[(RL + 7) / 8];
#pragma unroll
        for (int k = 0; k < (RL + 7) / 8; ++k) dw[k] = 0u;
#pragma unroll
        for (int k = 0; k < RL; ++k) {
          const int32_t sc = __builtin_amdgcn_sbfe((int32_t)X[k >> 2], 8 * (k & 3), 8);
          const int32_t diag = hdiag + sc;
          const int32_t fo = hcur - o, fx = fup - e;
          const int32_t fij = fo > fx ? fo : fx;
          const int32_t eo = H[k] - o, ex = E[k] - e;
          const int32_t eij = eo > ex ? eo : ex;
          int32_t h = diag > eij ? diag : eij;
          h = h > fij ? h : fij;
          // row k: nibble 7 - k % 8 of dword k / 8 (the first row on top)
          dw[k >> 3] = push_code(dw[k >> 3], diag, h, eij, fij, eo, ex, fo, fx);
          hdiag = H[k];
          H[k] = h;
          E[k] = eij;
          hcur = h;
          fup = fij;
        }
        hup_prev = hup;
        hout = H[RL - 1];
        fout = fup;
        sym = symn;
#pragma unroll
        for (int k = 0; k < RL / 4; ++k) X[k] = Xn[k];
        if constexpr (RL == 16) reinterpret_cast<uint2 *>(dstrip)[t * 64 + lane] = make_uint2(dw[0], dw[1]);
        else if constexpr (RL == 8) reinterpret_cast<uint32_t *>(dstrip)[t * 64 + lane] = dw[0];
        else reinterpret_cast<uint16_t *>(dstrip)[t * 64 + lane] = (uint16_t)dw[0];
        if (hand_over && gather) {
          const int jj = (tm + 1) & 63;   // (t - 63) mod 64
          const int32_t vh = __builtin_amdgcn_readlane(hout, 63);
          const int32_t vf = __builtin_amdgcn_readlane(fout, 63);
          obH = (lane == jj) ? vh : obH;
          obF = (lane == jj) ? vf : obF;
        }
      };
      // columns [cb, cb + jj] are complete: store and publish them
      auto hand = [&](int64_t cb, int jj) {
        if (lane <= jj) { outH[cb + lane] = obH; outF[cb + lane] = obF; }
        publish((int32_t)(cb + jj + 1 - clo), false);
      };
      const bool later = t0 >= 64;
      const int tn = (int)(nsteps - t0 < 64 ? nsteps - t0 : 64);
      const int ta = tn < 62 ? tn : 62;
#pragma unroll 1
      for (int tm = 0; tm < ta; ++tm) step(tm, symbuf, tm + 1, later);
      if (tn > 62) {
        step(62, symbuf, 63, later);
        if (hand_over && later) hand(clo + t0 - 64, 63);
      }
      if (tn > 63) step(63, symnext, 0, true);
      if (hand_over && t0 + tn == nsteps) {   // the strip's last step
        const int64_t t = nsteps - 1;
        const int jj = (int)((t - 63) & 63);
        if (t >= 63 && jj != 63) hand(clo + (t - 63) - jj, jj);
      }
    }
    publish((int32_t)(chi - clo), true);
  }
  if (spin_fail && lane == 0) a.err[p] = 1;   // reported as an internal failure
}

template <int RL>
__global__ __launch_bounds__(64 * kTbMaxWaves) void k_tb_wave(TbArgs a, const TbWaveJob *jobs,
                                                              uint8_t *dirw, int32_t *bndbuf) {
  extern __shared__ uint4 s_dyn[];                // per wave: profile [(n+1)][64][RL] score bytes
  __shared__ uint4 s_tile[kTbTileBytes / 16];
  __shared__ int8_t s_mat[32 * 32];
  __shared__ int32_t s_prog[kTbMaxStrips];   // columns of strip s's last row published
  __shared__ int32_t s_done[kTbMaxStrips];
  const TbWaveJob jb = jobs[blockIdx.x];
  uint8_t *dir = dirw + jb.dir_off;
  tb_wave_fill<RL>(a, jb, s_prog, s_done, s_mat, reinterpret_cast<int8_t *>(s_dyn), dir,
                   bndbuf + jb.bnd_off);
  // the walk reads every wave's codes: the barrier makes the workgroup's
  // stores visible to it (they pass through this compute unit's caches)
  __syncthreads();
  if (threadIdx.x < 64) tb_wave_walk<RL, kTbTileBytes>(a, jb, dir, s_tile, (int)threadIdx.x);
}

// Spread pairs: the pair's strips on the waves of `segs` workgroups (the grid
// fits on the device at once), and the walk left to k_tb_walk.  The hand-over
// is the intra-sequence fill's (k_intra_spread): one 64-bit word per column,
// valid << 63 | (F + 2^30) << 32 | (H + 2^30), its own flag, 16 columns at a
// time, read a block ahead; cleared before the launch.  Bound by the chain of
// strips: a 10,000-row alignment inside its band 3.7 -> 2.5 ms on four rows a
// lane, 2.27 on two (a strip starts its height and 110 steps after the one
// above: 79 of them take 23,000 shorter steps instead of 40 taking 18,600).
constexpr int kTbSpreadBlock = 16;
constexpr int kTbSpreadMaxWaves = 4;
constexpr uint64_t kTbWordValid = 1ull << 63;
__device__ __forceinline__ uint64_t tb_word(int32_t h, int32_t f) {
  constexpr int32_t kMin = -(1 << 30);   // lower values are as good as minus infinity
  h = h < kMin ? kMin : h;
  f = f < kMin ? kMin : f;
  return kTbWordValid | ((uint64_t)(uint32_t)(f - kMin) << 32) | (uint32_t)(h - kMin);
}
__device__ __forceinline__ int32_t tb_word_h(uint64_t w) { return (int32_t)(uint32_t)w - (1 << 30); }
__device__ __forceinline__ int32_t tb_word_f(uint64_t w) {
  return (int32_t)((uint32_t)(w >> 32) & 0x7FFFFFFFu) - (1 << 30);
}

template <int RL>
__global__ __launch_bounds__(64 * kTbSpreadMaxWaves) void k_tb_spread(TbArgs a, const TbWaveJob *jobs,
                                                                      int64_t njobs, int G,
                                                                      IntraSync *sync, uint8_t *dirw,
                                                                      int32_t *bndbuf) {
  constexpr int64_t SH = 64 * RL;
  constexpr int WB = RL / 2;                      // code bytes per lane and step
  constexpr int XW = tb_prof_words(RL);
  constexpr int kUnroll = RL <= 4 ? kTbSpreadBlock : 4;
  constexpr int AGENT = __HIP_MEMORY_SCOPE_AGENT;
  extern __shared__ uint4 s_dyn[];                // per wave: profile [(n+1)][64][RL] score bytes
  __shared__ int8_t s_mat[32 * 32];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int NW = blockDim.x >> 6;
  // block 8 * slot + x (slot = (j / 8) * G + segment) puts the segments of job
  // j on XCD j % 8; blocks past the last job leave at once
  const int64_t slot = blockIdx.x / 8;
  const int64_t jix = (slot / G) * 8 + blockIdx.x % 8;
  const int64_t seg = slot % G;
  if (jix >= njobs) return;
  const TbWaveJob jb = jobs[jix];
  const int32_t *done = sync[jix].done;
  const int64_t p = jb.pair, m = jb.m, w = jb.w;
  const int n = a.n;
  const int32_t o = a.o, e = a.e;
  const int64_t nstrips = (m + SH - 1) / SH;
  for (int k = threadIdx.x; k < n * n; k += blockDim.x) s_mat[k] = a.matrix[k];
  __syncthreads();
  const int8_t *q = a.qcat + a.qstart[p] + a.qbeg[p];
  const int8_t *r = a.rcat + a.rstart[p] + a.rbeg[p];
  uint64_t *rows = reinterpret_cast<uint64_t *>(bndbuf + jb.bnd_off);   // [strip][w + 1]
  int8_t *s_prof = reinterpret_cast<int8_t *>(s_dyn) + (size_t)wave * (n + 1) * 64 * RL;
  bool spin_fail = false;
  // choice codes of strip s start this many bytes after those of strip 0
  int64_t base = 0, base_of = 0;   // ... those of strip base_of at base (strips come in order)

  for (int64_t s = seg * NW + wave; s < nstrips; s += (int64_t)G * NW) {
    for (; base_of < s; ++base_of) {
      int64_t lo, hi;
      tbw_window(base_of, SH, jb.dlo, jb.bw, w, &lo, &hi);
      base += ((hi - lo) + 63) * 64 * WB;
    }
    int64_t clo, chi, plo = 0, phi = w + 1;
    tbw_window(s, SH, jb.dlo, jb.bw, w, &clo, &chi);
    if (s > 0) tbw_window(s - 1, SH, jb.dlo, jb.bw, w, &plo, &phi);
    uint64_t *out = rows + (w + 1) * s;      // this strip's last row
    const uint64_t *in = out - (w + 1);      // the row above it
    const bool hand_over = (s + 1 < nstrips);
    uint8_t *dstrip = dirw + jb.dir_off + base;
    // words of columns c0 .. c0 + cnt - 1 at lanes 0 .. cnt - 1; a column the
    // row above does not hold reads as minus infinity, and the virtual row
    // above strip 0 is H(0,0) = 0, H(0,j) = -(o + (j-1)e), F(0,j) = -inf
    auto fetch = [&](int64_t c0, int cnt) -> uint64_t {
      const int64_t c = c0 + lane;
      const bool have = lane < cnt && c < chi && c >= plo && c < phi;
      if (s == 0) return have ? tb_word(c == 0 ? 0 : -(o + (int32_t)(c - 1) * e), kNeg) : tb_word(kNeg, kNeg);
      return have ? __hip_atomic_load(in + c, __ATOMIC_RELAXED, AGENT) : tb_word(kNeg, kNeg);
    };
    auto ready = [](uint64_t x) { return __ballot((x & kTbWordValid) != 0) == ~0ull; };
    auto settle = [&](uint64_t x, int64_t c0, int cnt) -> uint64_t {
      int64_t spins = 0;
      while (!ready(x)) {
        const int32_t fin = __hip_atomic_load(done + s - 1, __ATOMIC_RELAXED, AGENT);
        if (fin) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        x = fetch(c0, cnt);
        if (fin) break;
        if (++spins > kTbSpinLimit) { spin_fail = true; break; }
        __builtin_amdgcn_s_sleep(1);
      }
      return (x & kTbWordValid) ? x : tb_word(kNeg, kNeg);
    };
    // profile of this lane's rows (signed scores; padding rows score 0)
    {
      int32_t qv[RL];
#pragma unroll
      for (int k = 0; k < RL; ++k) {
        const int64_t i = s * SH + lane * RL + k + 1;
        qv[k] = (i <= m) ? (int32_t)q[i - 1] : -1;
      }
      for (int sy = 0; sy <= n; ++sy) {
        uint32_t wv[XW];
#pragma unroll
        for (int k = 0; k < XW; ++k) wv[k] = 0u;
#pragma unroll
        for (int k = 0; k < RL; ++k) {
          const uint32_t b = (qv[k] >= 0 && sy < n) ? (uint32_t)(uint8_t)s_mat[qv[k] * n + sy] : 0u;
          wv[k >> 2] |= b << (8 * (k & 3));
        }
        int8_t *dst = s_prof + ((int64_t)sy * 64 + lane) * RL;
        if constexpr (RL == 2) {
          *reinterpret_cast<uint16_t *>(dst) = (uint16_t)wv[0];
        } else {
#pragma unroll
          for (int k = 0; k < XW; ++k) reinterpret_cast<uint32_t *>(dst)[k] = wv[k];
        }
      }
    }
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    int32_t H[RL], E[RL];
#pragma unroll
    for (int k = 0; k < RL; ++k) { H[k] = kNeg; E[k] = kNeg; }
    int32_t hup_prev = kNeg;
    if (clo >= 1) {
      const uint64_t x = settle(fetch(clo - 1, 1), clo - 1, 1);
      hup_prev = lane == 0 ? tb_word_h(x) : kNeg;
    }
    int32_t hout = kNeg, fout = kNeg;
    int32_t obH = 0, obF = 0;       // queues of lane 63's outputs, the newest at lane 63
    int64_t newest = clo - 64;      // ... of this column
    auto flush = [&]() {
      const int64_t c = newest - 63 + lane;
      if (hand_over && lane >= 64 - kTbSpreadBlock && c >= clo && c < chi)
        __hip_atomic_store(out + c, tb_word(obH, obF), __ATOMIC_RELAXED, AGENT);
    };
    const int64_t nsteps = (chi - clo) + (hand_over ? 63 : (m - s * SH + RL - 1) / RL - 1);
    // reference symbols of columns [c0, c0 + 16) at lanes 0 .. 15
    auto symbols = [&](int64_t c0) -> int32_t {
      const int64_t c = c0 + lane;
      return (lane < kTbSpreadBlock && c < chi && c >= 1) ? (int32_t)(uint8_t)r[c - 1] : n;
    };
    uint32_t sym = (uint32_t)tb_from_above(n, __builtin_amdgcn_readlane(symbols(clo), 0));
    uint32_t X[XW];
    tb_prof_load<RL>(s_prof + ((int64_t)sym * 64 + lane) * RL, X);
    int32_t symnext = symbols(clo + 1);
    uint64_t wnext = fetch(clo, kTbSpreadBlock);
#pragma unroll 1
    for (int64_t t0 = 0; t0 < nsteps; t0 += kTbSpreadBlock) {
      uint64_t x = wnext;
      const bool here = ready(x);
      const int32_t symbuf = symnext;
      flush();   // the last block's outputs go out before anything waits
      if (!here) x = settle(x, clo + t0, kTbSpreadBlock);
      wnext = fetch(clo + t0 + kTbSpreadBlock, kTbSpreadBlock);
      symnext = symbols(clo + t0 + kTbSpreadBlock + 1);
      const int32_t hbuf = tb_word_h(x), fbuf = tb_word_f(x);
      // codes past the strip's last step are not kept
      const int left = (int)(nsteps - t0 < kTbSpreadBlock ? nsteps - t0 : kTbSpreadBlock);
#pragma unroll kUnroll
      for (int tm = 0; tm < kTbSpreadBlock; ++tm) {
        const int32_t hup = tb_from_above(hout, __builtin_amdgcn_readlane(hbuf, tm));
        int32_t fup = tb_from_above(fout, __builtin_amdgcn_readlane(fbuf, tm));
        const uint32_t symn = (uint32_t)tb_from_above((int32_t)sym, __builtin_amdgcn_readlane(symbuf, tm));
        uint32_t Xn[XW];
        tb_prof_load<RL>(s_prof + ((int64_t)symn * 64 + lane) * RL, Xn);
        int32_t hdiag = hup_prev;
        int32_t hcur = hup;
        uint32_t dw[(RL + 7) / 8];
#pragma unroll
        for (int k = 0; k < (RL + 7) / 8; ++k) dw[k] = 0u;
#pragma unroll
        for (int k = 0; k < RL; ++k) {
          const int32_t sc = __builtin_amdgcn_sbfe((int32_t)X[k >> 2], 8 * (k & 3), 8);
          const int32_t diag = hdiag + sc;
          const int32_t fo = hcur - o, fx = fup - e;
          const int32_t fij = fo > fx ? fo : fx;
          const int32_t eo = H[k] - o, ex = E[k] - e;
          const int32_t eij = eo > ex ? eo : ex;
          int32_t h = diag > eij ? diag : eij;
          h = h > fij ? h : fij;
          // row k: nibble 7 - k % 8 of dword k / 8 (the first row on top)
          dw[k >> 3] = push_code(dw[k >> 3], diag, h, eij, fij, eo, ex, fo, fx);
          hdiag = H[k];
          H[k] = h;
          E[k] = eij;
          hcur = h;
          fup = fij;
        }
        hup_prev = hup;
        hout = H[RL - 1];
        fout = fup;
        sym = symn;
#pragma unroll
        for (int k = 0; k < XW; ++k) X[k] = Xn[k];
        if (tm < left) {
          const int64_t t = t0 + tm;
          if constexpr (RL == 16) reinterpret_cast<uint2 *>(dstrip)[t * 64 + lane] = make_uint2(dw[0], dw[1]);
          else if constexpr (RL == 8) reinterpret_cast<uint32_t *>(dstrip)[t * 64 + lane] = dw[0];
          else if constexpr (RL == 4) reinterpret_cast<uint16_t *>(dstrip)[t * 64 + lane] = (uint16_t)dw[0];
          else dstrip[t * 64 + lane] = (uint8_t)dw[0];
        }
        obH = tb_shift_in(obH, hout);
        obF = tb_shift_in(obF, fout);
      }
      newest = clo + t0 + kTbSpreadBlock - 64;   // step t ends column clo + t - 63
    }
    flush();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane == 0) __hip_atomic_store(&sync[jix].done[s], 1, __ATOMIC_RELAXED, AGENT);
  }
  if (spin_fail && lane == 0) a.err[p] = 1;   // reported as an internal failure
}

// One pair per workgroup, planned by the workgroup itself: the traceback of
// batches (or classes of a batch) too small for the per-lane kernels.  Those
// put 64 or 16 pairs on a wave and take as long as one lane needs for its
// pair, 0.16 (8-wide bands) to 1.0 ms (wide bands) for a read of 150-250 nt
// however few pairs there are, one class after the other in a graph; a
// wavefront over the pair's rows takes about 50 us, and the device runs a few
// thousand such waves at once.  Bound by the wavefront's step chain (few
// pairs), then by VALU issue over all 64 lanes, of which a short read fills
// half: per cell the per-lane kernels are 3-4 times cheaper.  Measured on
// reads (whole traceback stage): 101 pairs 1.14 -> 0.19 ms, 4,000 1.8 ->
// 0.32, 20,000 1.92 -> 0.86; 512 in a graph 1.85 -> 0.1.
constexpr int kTbPairTile = 8192;
constexpr int kTbPairMaxWaves = 4;

__global__ __launch_bounds__(64 * kTbPairMaxWaves) void k_tb_pairs(TbArgs a, TbPairs t) {
  constexpr int RL = kTbPairRows;
  extern __shared__ uint4 s_dyn[];
  __shared__ uint4 s_tile[kTbPairTile / 16];
  __shared__ int8_t s_mat[32 * 32];
  __shared__ int32_t s_prog[kTbMaxStrips], s_done[kTbMaxStrips];
  __shared__ int64_t s_off;
  int64_t p = blockIdx.x;
  if (t.sorted) {
    int64_t k = p;
    int x = 0;
    while (x + 1 < t.ranges && k >= t.cnt[x]) k -= t.cnt[x++];
    p = t.sorted[t.lo[x] + k];
  } else if (t.cls) {
    const uint8_t c = t.cls[p];
    if (c == 0 || c == 6 || c == kTbFlat) return;   // nothing to trace, or another kernel's pair
  }
  TbWaveJob jb{};
  jb.pair = p;
  jb.m = a.qend[p] - a.qbeg[p] + 1;
  jb.w = a.rend[p] - a.rbeg[p] + 1;
  if (!t.sorted && !t.cls) {
    const int32_t s1 = a.score[p];
    const bool ok = s1 > 0 && tb_coords_ok(a, p);
    int32_t sum = 0;   // the main diagonal's, by every wave alike
    if (ok && jb.m == jb.w && jb.m < (1 << 24)) {
      const int8_t *q = a.qcat + a.qstart[p] + a.qbeg[p], *r = a.rcat + a.rstart[p] + a.rbeg[p];
      for (int64_t x = threadIdx.x & 63; x < jb.m; x += 64) {
        const uint32_t qc = (uint8_t)q[x], rc = (uint8_t)r[x];
        sum += qc < (uint32_t)a.n && rc < (uint32_t)a.n ? a.matrix[qc * a.n + rc] : 0;   // (a graph's codes may be bad)
      }
      for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
    }
    const bool flat = ok && jb.m == jb.w && jb.m < (1 << 24) && sum == s1;
    if (!ok || flat) {
      if (threadIdx.x == 0) {
        if (s1 > 0 && !ok) a.err[p] = 1;
        a.cig_len[p] = flat ? 1 : 0;
        if (flat) *tb_cig(a, p) = (uint32_t)jb.m << 4;
      }
      return;
    }
  }
  safe_band(jb.m, jb.w, a.score[p], a.smax, a.o, a.e, &jb.dlo, &jb.bw);
  const int64_t bytes = tb_pair_bytes(jb.m, jb.w, jb.dlo, jb.bw);
  int64_t off = t.stride * (int64_t)blockIdx.x, room = t.stride;
  if (t.used) {
    if (threadIdx.x == 0) s_off = (int64_t)atomicAdd(t.used, (unsigned long long)bytes);
    __syncthreads();
    off = s_off;
    room = t.cap - off;
  }
  if (bytes > room || (jb.m + 64 * RL - 1) / (64 * RL) > kTbMaxStrips) {
    if (threadIdx.x == 0) a.err[p] = 1;   // never expected: the caller sized the scratch
    return;
  }
  int32_t *bnd = reinterpret_cast<int32_t *>(t.scratch + off);
  uint8_t *dir = t.scratch + off + tb_pair_bnd_bytes(jb.m, jb.w);
  tb_wave_fill<RL>(a, jb, s_prog, s_done, s_mat, reinterpret_cast<int8_t *>(s_dyn), dir, bnd);
  __syncthreads();
  if (threadIdx.x < 64) tb_wave_walk<RL, kTbPairTile>(a, jb, dir, s_tile, (int)threadIdx.x);
}

hipError_t tb_pairs(const TbArgs &a, const TbPairs &t, int64_t blocks, int64_t max_rows,
                    hipStream_t st) {
  if (blocks == 0) return hipSuccess;
  if (!t.sorted && !t.cls && t.used) return hipErrorInvalidValue;
  const int64_t per = (int64_t)(a.n + 1) * 64 * kTbPairRows;
  int64_t waves = (max_rows + 64 * kTbPairRows - 1) / (64 * kTbPairRows);
  waves = std::min<int64_t>({waves, (int64_t)kTbPairMaxWaves, (65536 - 16384) / per});
  if (waves < 1) waves = 1;
  hipLaunchKernelGGL(k_tb_pairs, dim3((unsigned)blocks), dim3((unsigned)(64 * waves)),
                     (size_t)(per * waves), st, a, t);
  return hipGetLastError();
}

// The walk of spread pairs, one wave per pair, after their fill kernel.
template <int RL>
__global__ __launch_bounds__(64) void k_tb_walk(TbArgs a, const TbWaveJob *jobs, uint8_t *dirw) {
  __shared__ uint4 s_tile[kTbTileBytes / 16];
  const TbWaveJob jb = jobs[blockIdx.x];
  tb_wave_walk<RL, kTbTileBytes>(a, jb, dirw + jb.dir_off, s_tile, (int)(threadIdx.x & 63));
}

template <int RL, int TILE>
__device__ void tb_wave_walk(const TbArgs &a, const TbWaveJob &jb, const uint8_t *dir,
                             uint4 *s_tile, int lane) {
  constexpr int32_t SH = 64 * RL;
  constexpr int WB = RL / 2;
  constexpr int TS = TILE / (64 * WB);
  static_assert(TILE % (8 * 64 * 16) == 0, "whole rounds of loads");
  const int64_t p = jb.pair;
  // (a column's codes take 128 bytes and more: rows and columns fit 32 bits)
  const int32_t m = (int32_t)jb.m, w = (int32_t)jb.w;
  const int32_t o = a.o, e = a.e;
  const int32_t nstrips = (m + SH - 1) / SH;
  auto strip_base = [&](int32_t s) {
    int64_t off = 0;
    for (int32_t k = 0; k < s; ++k) {
      int64_t lo, hi;
      tbw_window(k, SH, jb.dlo, jb.bw, w, &lo, &hi);
      off += ((hi - lo) + 63) * 64 * WB;
    }
    return off;
  };

  // ---- walk back from (m, w) in state H (rule T3), uniform on the wave ------
  // Each iteration places the walk in a strip and a tile of its codes and
  // follows one run of the path and the gap step after it (below).  Bound by
  // the latency of an iteration's instructions and its one LDS read; with the
  // gap step in an iteration of its own and 64-bit coordinates the walk of
  // 10,000 rows at 10% errors took 1.24 ms; with its tiles loaded eight words a
  // lane at a time and the runs turned round by all lanes besides, 0.43.
  uint32_t *out = tb_cig(a, p);
  int32_t nruns = 0;
  int32_t i = m, j = w;
  int state = 0;
  uint32_t cur_op = 0xFF, cur_len = 0;
  int64_t guard = 2 * ((int64_t)m + w) + 4;
  int32_t ws = nstrips;          // strip whose codes start at wbase
  int64_t wbase = strip_base(nstrips);
  int32_t wclo = 0, wchi = 0;
  int32_t tile_s = -1, tile_lo = 0, tile_hi = -1;
  const uint8_t *tile = reinterpret_cast<const uint8_t *>(s_tile);
  bool bad = false;
  auto emit_run = [&](uint32_t op, uint32_t len) {
    if (op == cur_op) {
      cur_len += len;
    } else {
      if (cur_len && lane == 0) out[nruns] = (cur_len << 4) | cur_op;
      if (cur_len) ++nruns;
      cur_op = op;
      cur_len = len;
    }
  };
  while ((i > 0 || j > 0) && guard > 0) {
    if (i == 0) {   // row 0: reached from the left by one deletion run
      const uint32_t c = row0_code(j, o, e);
      --guard;
      if (state == 0) {
        state = code_src(c) == 1 ? 1 : 2;
      } else if (state == 1) {
        emit_run(2u, 1u);
        state = (c & kCodeEExt) ? 1 : 0;
        --j;
      } else {
        bad = true;   // no cell above row 0
        break;
      }
      continue;
    }
    const int32_t s = (i - 1) / SH;
    while (ws > s) {   // step the strip cursor up (the walk only moves up)
      --ws;
      int64_t lo, hi;
      tbw_window(ws, SH, jb.dlo, jb.bw, w, &lo, &hi);
      wclo = (int32_t)lo;
      wchi = (int32_t)hi;
      wbase -= ((hi - lo) + 63) * 64 * WB;
    }
    if (j < wclo || j >= wchi) { bad = true; break; }
    const int xi = (i - 1) - s * SH;   // the current row in the strip
    const int jw = j - wclo;           // the current column in the window
    const int32_t t = jw + xi / RL;
    if (s != tile_s || t < tile_lo || t > tile_hi) {
      tile_s = s;
      tile_hi = t;
      tile_lo = t >= TS - 1 ? t - (TS - 1) : 0;
      // steps [tile_lo, tile_hi] are contiguous: 16 bytes per lane and load
      const uint4 *src = reinterpret_cast<const uint4 *>(dir + wbase + (int64_t)tile_lo * 64 * WB);
      const int nv = (tile_hi - tile_lo + 1) * 64 * WB / 16;
      __builtin_amdgcn_wave_barrier();
      // (eight loads in flight, past the end the last one again: one at a time
      // they took half of the walk)
      for (int v0 = lane; v0 < nv; v0 += 8 * 64) {
        uint4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = src[v0 + 64 * u < nv ? v0 + 64 * u : nv - 1];
#pragma unroll
        for (int u = 0; u < 8; ++u) s_tile[v0 + 64 * u] = x[u];
      }
      __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
    }
    // One run per iteration, on the whole wave: lane k reads the code of the
    // k-th cell along the run's direction (diagonal for M, left for D, up for
    // I; invalid past the strip's top, the window's left edge or the tile),
    // and a ballot finds where the run ends.  In state H the diagonal run
    // continues while a cell's code names the diagonal; the cell that names E
    // or F takes that gap step at once (same code); a gap run continues while
    // a cell's code extends the gap, the cell that does not still taking its
    // step.  A run cut short by an unreadable cell resumes in the next
    // iteration, after the strip cursor and the tile have moved.
    const int tlo = tile_lo;
    auto lane_code = [&](int drow, int dcol, bool &valid) -> uint32_t {
      const int xr = xi - lane * drow, jc = jw - lane * dcol;
      const int xq = xr < 0 ? 0 : xr;
      const int Lk = xq / RL, rk = xq % RL;
      const int tk = jc + Lk - tlo;
      valid = xr >= 0 && jc >= 0 && tk >= 0;
      const uint8_t *wp = tile + (((valid ? tk : 0) * 64 + Lk) * WB);
      if constexpr (RL == 2) {
        return ((uint32_t)*wp >> (4 * (1 - rk))) & 0xFu;
      } else if constexpr (RL == 4) {
        return ((uint32_t)*reinterpret_cast<const uint16_t *>(wp) >> (4 * (3 - rk))) & 0xFu;
      } else {
        const uint32_t dv = reinterpret_cast<const uint32_t *>(wp)[rk >> 3];
        return (dv >> (4 * (7 - (rk & 7)))) & 0xFu;
      }
    };
    auto first_false = [](bool pred) -> int {
      const unsigned long long bm = __ballot(pred);
      return bm == ~0ull ? 64 : __builtin_ctzll(~bm);
    };
    if (state == 0) {
      bool v;
      const uint32_t ck = lane_code(1, 1, v);
      const int K = first_false(v && (ck & kCodeNotM) == 0 && j - lane > 0);
      const unsigned long long readable = __ballot(v);
      if (K > 0) {
        emit_run(0u, (uint32_t)K);
        i -= K;
        j -= K;
        guard -= K;
        if (K == 64 || !((readable >> K) & 1ull) || i == 0) continue;
      }
      // this cell leaves the diagonal: its code names E or F (at column 0 the
      // path can only go up)
      const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)ck, K);
      const uint32_t src = code_src(c);
      state = src == 0 ? 2 : (int)src;
      const bool left = state == 1;
      if (left && j <= 0) { bad = true; break; }
      const bool longer = (c & (left ? kCodeEExt : kCodeFExt)) != 0;
      if (!longer || K > 0) {   // (a longer gap from the first cell read: below)
        if (!longer) state = 0;
        emit_run(left ? 2u : 1u, 1u);
        if (left) --j;
        else --i;
        --guard;
        continue;
      }
    }
    const bool left = state == 1;
    bool v;
    const uint32_t ck = left ? lane_code(0, 1, v) : lane_code(1, 0, v);
    const bool ext = v && (ck & (left ? kCodeEExt : kCodeFExt)) != 0 && (!left || j - lane > 0);
    const int stop = first_false(ext);
    // the cell that ends the run takes its step too, when it was readable
    const bool ends = stop < 64 && ((__ballot(v) >> stop) & 1ull);
    const int moves = ends ? stop + 1 : stop;
    if (moves == 0) { bad = true; break; }
    if (ends) state = 0;
    emit_run(left ? 2u : 1u, (uint32_t)moves);
    if (left) j -= moves;
    else i -= moves;
    guard -= moves;
  }
  if (lane == 0) {
    if (bad || i != 0 || j != 0) a.err[p] = 1;
    if (cur_len) out[nruns] = (cur_len << 4) | cur_op;
  }
  if (cur_len) ++nruns;
  if (lane == 0) a.cig_len[p] = nruns;
  // the runs, last first so far, turned round by the whole wave (one lane alone
  // waited for a load per run)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (int32_t x = lane; x < nruns / 2; x += 64) {
    const int32_t y = nruns - 1 - x;
    const uint32_t t = out[x];
    out[x] = out[y];
    out[y] = t;
  }
}

int tb_wave_waves(int64_t m, int n, int RL) {
  const int64_t nstrips = (m + 64 * RL - 1) / (64 * RL);
  const int64_t per = (int64_t)(n + 1) * 64 * RL;
  const int64_t stat = kTbTileBytes + 32 * 32 + kTbMaxStrips * 8;
  const int64_t room = (65536 - stat) / per;
  int64_t wv = std::min<int64_t>(std::min<int64_t>(nstrips, kTbMaxWaves), room);
  return (int)(wv < 1 ? 1 : wv);
}

int tb_wave_max_strips() { return kTbMaxStrips; }

template <int RL>
static void launch_tb_wave(const TbArgs &a, const TbWaveJob *jobs, int64_t njobs, int waves,
                           int segs, IntraSync *sync, uint8_t *dirw, int32_t *bnd, hipStream_t st) {
  const size_t lds = (size_t)(a.n + 1) * 64 * RL * waves;
  if (RL == 2 || segs > 1) {   // (two rows per lane: spread pairs only)
    const dim3 g((unsigned)(8 * segs * ((njobs + 7) / 8)));
    hipLaunchKernelGGL(k_tb_spread<RL>, g, dim3(64 * waves), lds, st, a, jobs, njobs, segs, sync,
                       dirw, bnd);
    hipLaunchKernelGGL(k_tb_walk<RL>, dim3((unsigned)njobs), dim3(64), 0, st, a, jobs, dirw);
  } else if constexpr (RL != 2) {
    hipLaunchKernelGGL(k_tb_wave<RL>, dim3((unsigned)njobs), dim3(64 * waves), lds, st, a, jobs,
                       dirw, bnd);
  }
}

hipError_t tb_wave(const TbArgs &a, const TbWaveJob *jobs, int64_t njobs, int RL, int waves,
                   int segs, IntraSync *sync, uint8_t *dirw, int32_t *bnd, hipStream_t st) {
  if (njobs == 0) return hipSuccess;
  if (waves < 1 || waves > kTbMaxWaves || segs < 1 || (segs > 1 && (!sync || waves > kTbSpreadMaxWaves)))
    return hipErrorInvalidValue;
  if (segs > 1) {
    const hipError_t e = intra_sync_init(sync, njobs, st);
    if (e != hipSuccess) return e;
  }
  switch (RL) {
    case 2:
      if (segs < 2) return hipErrorInvalidValue;
      launch_tb_wave<2>(a, jobs, njobs, waves, segs, sync, dirw, bnd, st);
      break;
    case 4: launch_tb_wave<4>(a, jobs, njobs, waves, segs, sync, dirw, bnd, st); break;
    case 8: launch_tb_wave<8>(a, jobs, njobs, waves, segs, sync, dirw, bnd, st); break;
    case 16: launch_tb_wave<16>(a, jobs, njobs, waves, segs, sync, dirw, bnd, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---- the one-pair call: everything after the forward pass -----------------------
// One workgroup: the end from the max array, the reversed pass, score2, the
// banded pass and its walk, and the record and CIGAR into pinned host memory.
// Bound by the two strip chains and the walk; as separate kernels in a graph
// these steps took fifteen launches of 4.6 us each beside them, and four
// copies to the host.  Measured, the whole call: 150 x 2,000 318 -> 153 us,
// 300 x 350 amino acids 426 -> 208, 1,000 x 2,000 1,553 -> 802.
template <bool HO>
__global__ __launch_bounds__(64 * kPairWaves) void k_pair_rest(PairArgs a) {
  constexpr int RL = kPairRows;
  constexpr int SH = 64 * RL;
  const int NW = (int)(blockDim.x >> 6);
  extern __shared__ uint4 s_dyn[];
  __shared__ uint4 s_tile[kTbPairTile / 16];
  __shared__ int8_t s_mat[32 * 32];
  __shared__ int32_t s_prog[kPairWaves], s_done[kPairWaves], s_rrow[kPairWaves], s_v[kPairWaves];
  __shared__ int64_t s_rcol[kPairWaves], s_j[kPairWaves];
  __shared__ unsigned long long s_best;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int k = threadIdx.x; k < a.n * a.n; k += blockDim.x) s_mat[k] = a.m[k];
  if (threadIdx.x < kPairWaves) {
    s_done[threadIdx.x] = 0;
    s_rcol[threadIdx.x] = -1;
    s_rrow[threadIdx.x] = -1;
  }
  if (threadIdx.x == 0) s_best = ~0ull;

  // largest value, then smallest column, outside columns [lo, hi]
  auto best_column = [&](int64_t lo, int64_t hi, int32_t &bv, int64_t &bj) {
    bv = 0;
    bj = INT64_MAX;
#pragma unroll 4
    for (int64_t j = threadIdx.x; j < a.Lr; j += blockDim.x) {
      const int32_t v = (int32_t)(a.maxcol[j] >> a.kb);
      if ((j < lo || j > hi) && v > bv) { bv = v; bj = j; }
    }
    auto better = [&](int32_t v, int64_t j) {
      if (v > bv || (v == bv && j < bj)) { bv = v; bj = j; }
    };
    for (int off = 32; off >= 1; off >>= 1) {
      const int32_t v = __shfl_xor(bv, off, 64);
      const int64_t j = __shfl_xor(bj, off, 64);
      better(v, j);
    }
    __syncthreads();   // (the slots may still be read from the last time)
    if (lane == 0) {
      s_v[wave] = bv;
      s_j[wave] = bj;
    }
    __syncthreads();
    for (int w = 0; w < NW; ++w) better(s_v[w], s_j[w]);
  };

  swx_rec_dev rec;
  rec.score1 = rec.score2 = 0;
  rec.read_begin1 = rec.read_end1 = -1;
  rec.ref_begin1 = rec.ref_end1 = rec.ref_end2 = -1;
  rec.cigar_off = 0;
  rec.cigar_len = 0;
  rec.lane_bits = 32;
  int32_t s1;
  int64_t je;
  best_column(1, 0, s1, je);
  bool err = false;
  if (s1 > 0) {
    const uint32_t M = (1u << a.kb) - 1u;
    const int32_t ie = (int32_t)(M - (a.maxcol[je] & M)) - (a.strips * SH - a.Lq);
    rec.score1 = s1;
    rec.read_end1 = ie;
    rec.ref_end1 = je;
    err = ie < 0 || ie >= a.Lq;
    if ((a.flags & 1u) && !err) {
      int32_t band, band_q;
      rev_band(s1, (int64_t)ie + 1, je + 1, a.smax, a.o, a.e, band, band_q);
      StripJob x{};
      x.qs = a.q;
      x.rs = a.r;
      x.Lq = ie + 1;
      x.rv = true;
      x.Lr = je + 1;
      x.c1 = je + 1;
      x.band = band;
      x.kb = a.kb;
      x.tgt = s1;
      x.rows = a.rwords;
      x.done = s_done;
      x.rcol = s_rcol;
      x.rrow = s_rrow;
      x.best = &s_best;
      const StripScoring sc{a.n, (uint32_t)a.bias, (uint32_t)a.o, (uint32_t)a.e};
      uint8_t *s_prof = reinterpret_cast<uint8_t *>(s_dyn) + (size_t)wave * (a.n + 1) * 64 * RL;
      if (x.Lq <= SH) {
        if (wave == 0) strip_alone<RL, true, HO>(x, sc, s_mat, s_prof);
      } else if (strips_of_wave<RL, true, HO>(x, sc, s_mat, s_prof, wave, NW) && lane == 0) {
        a.out->err = 1;
      }
      __syncthreads();
      int64_t bc = -1;   // first column reaching score1; on a tie the earlier strip
      int32_t br = -1;
      for (int s = 0; s < kPairWaves; ++s)
        if (s_rcol[s] >= 0 && (bc < 0 || s_rcol[s] < bc)) { bc = s_rcol[s]; br = s_rrow[s]; }
      rec.read_begin1 = ie - br;
      rec.ref_begin1 = je - bc;
      err = bc < 0 || br < 0 || br > ie;
    }
    if ((a.flags & 4u) && !err) {
      int64_t mask = a.mask_len;
      if (mask < 0) { mask = a.Lq / 2; if (mask < 15) mask = 15; }
      int64_t j2;
      best_column(rec.ref_begin1 - mask, je + mask, rec.score2, j2);
      rec.ref_end2 = rec.score2 > 0 ? j2 : -1;
    }
    if ((a.flags & 2u) && !err) {
      TbWaveJob jb{};
      jb.m = rec.read_end1 - rec.read_begin1 + 1;
      jb.w = rec.ref_end1 - rec.ref_begin1 + 1;
      uint32_t *cigar = reinterpret_cast<uint32_t *>(a.out + 1);
      bool flat = false;
      if (jb.m == jb.w) {   // kTbFlat: the main diagonal alone scores score1
        int32_t sum = 0;
        for (int64_t k = threadIdx.x; k < jb.m; k += blockDim.x)
          sum += s_mat[a.q[rec.read_begin1 + k] * a.n + a.r[rec.ref_begin1 + k]];
        for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
        __syncthreads();
        if (lane == 0) s_v[wave] = sum;
        __syncthreads();
        sum = 0;
        for (int w = 0; w < NW; ++w) sum += s_v[w];
        flat = sum == s1;
      }
      if (flat) {
        rec.cigar_len = 1;
        if (threadIdx.x == 0) cigar[0] = (uint32_t)jb.m << 4;
      } else {
        safe_band(jb.m, jb.w, s1, a.smax, a.o, a.e, &jb.dlo, &jb.bw);
        if (threadIdx.x == 0) {
          PairState &y = *a.state;
          y.qstart = y.rstart = y.cig_off = 0;
          y.rbeg = rec.ref_begin1;
          y.rend = rec.ref_end1;
          y.rlen = a.Lr;
          y.score = s1;
          y.qbeg = rec.read_begin1;
          y.qend = rec.read_end1;
          y.qlen = a.Lq;
          y.cig_len = 0;
          y.err = 0;
        }
        __threadfence_block();
        __syncthreads();
        tb_wave_fill<RL>(a.tb, jb, s_prog, s_done, s_mat, reinterpret_cast<int8_t *>(s_dyn), a.dir,
                         a.bnd);
        __syncthreads();
        if (wave == 0) tb_wave_walk<RL, kTbPairTile>(a.tb, jb, a.dir, s_tile, lane);
        __threadfence_block();
        __syncthreads();
        rec.cigar_len = a.state->cig_len;
        err = a.state->err != 0;
        for (int32_t k = threadIdx.x; k < rec.cigar_len; k += blockDim.x) cigar[k] = a.tb.cig[k];
      }
    }
  }
  if (threadIdx.x == 0) {
    a.out->rec = rec;
    if (err) a.out->err = 1;
  }
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(&a.out->done, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t pair_rest(const PairArgs &a, hipStream_t st) {
  // (four waves at least: they scan the max array together)
  const int waves = std::max(pair_waves(a.strips, a.n), 4);
  const dim3 b(64 * waves);
  const size_t lds = (size_t)(a.n + 1) * 64 * kPairRows * waves;
  if (a.bias == a.o) hipLaunchKernelGGL(k_pair_rest<true>, dim3(1), b, lds, st, a);
  else hipLaunchKernelGGL(k_pair_rest<false>, dim3(1), b, lds, st, a);
  return hipGetLastError();
}

int64_t tb_wave_dir_bytes(int64_t m, int64_t w, int RL) {
  const int64_t SH = 64 * RL, nstrips = (m + SH - 1) / SH;
  return nstrips * (w + 1 + 63) * 64 * (RL / 2);
}

hipError_t tbw_tasks(int64_t n0, int64_t n1, const int64_t *sorted, const TbArgs &a,
                     TbwTask *tasks, int64_t *dir_words, int64_t *bnd_words, hipStream_t st) {
  const int64_t nt = (n1 - n0 + kTbwSlots - 1) / kTbwSlots;
  if (nt <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tbw_tasks, dim3(nblk(nt, 4)), dim3(256), 0, st, n0, n1,
                     (const int64_t *)nullptr, (int64_t)0, sorted, a, tasks, dir_words, bnd_words);
  return hipGetLastError();
}

hipError_t tbw_tasks_range(const int64_t *range, int64_t ntasks_cap, const int64_t *sorted,
                           const TbArgs &a, TbwTask *tasks, int64_t *dir_words, int64_t *bnd_words,
                           hipStream_t st) {
  if (ntasks_cap <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tbw_tasks, dim3(nblk(ntasks_cap, 4)), dim3(256), 0, st, (int64_t)0,
                     (int64_t)0, range, ntasks_cap, sorted, a, tasks, dir_words, bnd_words);
  return hipGetLastError();
}

hipError_t tbw_offsets(int64_t ntasks, TbwTask *tasks, const int64_t *doff, const int64_t *boff,
                       hipStream_t st) {
  if (!ntasks) return hipSuccess;
  hipLaunchKernelGGL(k_tbw_offsets, dim3(nblk(ntasks, 128)), dim3(128), 0, st, ntasks, tasks, doff,
                     boff);
  return hipGetLastError();
}

hipError_t tb_strip(const TbArgs &a, const TbwTask *tasks, int64_t ntasks, const int64_t *sorted,
                    int32_t *bndbuf, hipStream_t st) {
  if (!ntasks) return hipSuccess;
  const unsigned blocks = nblk(ntasks, 4);
  if (a.n <= 4)
    hipLaunchKernelGGL((k_tb_strip<true>), dim3(blocks), dim3(256), 0, st, a, tasks, ntasks, sorted, bndbuf);
  else
    hipLaunchKernelGGL((k_tb_strip<false>), dim3(blocks), dim3(256), 0, st, a, tasks, ntasks, sorted, bndbuf);
  return hipGetLastError();
}

}  // namespace swx
