// intra_strips.h -- the 32-bit strip sweep of one long pair (device code).
//
// One pair is spread over the 64 lanes of a wave: lane k owns RL consecutive
// query rows of a strip of 64*RL rows and computes column c - k at step c.
// Shared by the kernels that spread a pair's strips over several workgroups
// and by those of the one-pair call.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lanes.h"
#include "swx_internal.h"
#include "swx_kernels.h"

namespace swx {

constexpr int kDppWaveShr1 = 0x138;   // DPP control: lane k reads lane k - 1

// value of src from the lane above; lane 0 takes `top`
__device__ __forceinline__ uint32_t from_above(uint32_t src, uint32_t top) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)top, (int)src, kDppWaveShr1, 0xF, 0xF, false);
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

constexpr int kDppWaveShl1 = 0x130;   // DPP control: lane k reads lane k + 1

// vec moved one lane down (lane k takes lane k + 1) with lane 63 taking its
// own v: a queue of lane 63's values, the newest at lane 63
__device__ __forceinline__ uint32_t shift_in(uint32_t vec, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)vec, kDppWaveShl1, 0xF, 0xF, false);
}

// RL bytes (RL a multiple of 4) of the LDS profile as RL/4 words
template <int RL>
__device__ __forceinline__ void lds_load_words(const uint8_t *src, uint32_t (&w)[RL / 4]) {
  if constexpr (RL % 16 == 0) {
#pragma unroll
    for (int k = 0; k < RL / 16; ++k) {
      const uint4 v = reinterpret_cast<const uint4 *>(src)[k];
      w[4 * k] = v.x; w[4 * k + 1] = v.y; w[4 * k + 2] = v.z; w[4 * k + 3] = v.w;
    }
  } else if constexpr (RL == 8) {
    const uint2 v = *reinterpret_cast<const uint2 *>(src);
    w[0] = v.x; w[1] = v.y;
  } else {
    w[0] = *reinterpret_cast<const uint32_t *>(src);
  }
}

template <int RL>
__device__ __forceinline__ void lds_store_words(uint8_t *dst, const uint32_t (&w)[RL / 4]) {
  if constexpr (RL % 16 == 0) {
#pragma unroll
    for (int k = 0; k < RL / 16; ++k)
      reinterpret_cast<uint4 *>(dst)[k] = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
  } else if constexpr (RL == 8) {
    *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
  } else {
    *reinterpret_cast<uint32_t *>(dst) = w[0];
  }
}

constexpr int64_t kSpinLimit = int64_t(1) << 26;

__device__ __forceinline__ void lds_wave_sync() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

constexpr int kSpreadBlock = 16;
constexpr uint64_t kWordValid = 1ull << 63;

// RL profile bytes of one lane and symbol as words (RL = 2: the low half)
template <int RL>
__device__ __forceinline__ void prof_load(const uint8_t *src, uint32_t (&w)[RL >= 4 ? RL / 4 : 1]) {
  if constexpr (RL >= 4) lds_load_words<RL>(src, w);
  else w[0] = *reinterpret_cast<const uint16_t *>(src);
}

// One pair's job: the sequences (rv: read backwards), columns [cw, c1) of
// which [c0, c1) are written to the max array, the reversed pass's drift band
// (-1: none) and target, the row-code bits, and for several strips the
// hand-over words [strip][c1 - cw] and per-strip records.
struct StripJob {
  const int8_t *qs, *rs;
  int32_t Lq;
  bool rv;
  int64_t Lr, cw, c0, c1;
  int32_t band, kb, tgt;
  uint32_t *mc;
  uint64_t *rows;
  int32_t *done;               // strip s has stored every word it will
  int64_t *rcol;               // reversed pass: first column of strip s reaching the target (-1)
  int32_t *rrow;               // ... and its padded row
  unsigned long long *best;    // ... smallest such column so far (~0: none)
  int32_t row0;                // one strip: padded row of the strip's first row in the row code
  uint32_t anchor;             // one strip, reversed: the score that a path from the first cell starts with
};
struct StripScoring {
  int n;
  uint32_t bias, o, e;
};

// Profile of the RL rows from query index i0: biased scores against every
// symbol, zero outside the query and for the padding symbol n.
template <int RL>
__device__ __forceinline__ void strip_profile(const StripJob &x, const StripScoring &sc,
                                              const int8_t *s_mat, uint8_t *s_prof, int64_t i0) {
  constexpr int XW = RL >= 4 ? RL / 4 : 1;
  const int lane = threadIdx.x & 63;
  int32_t qv[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) {
    const int64_t i = i0 + r;
    qv[r] = (i >= 0 && i < x.Lq) ? (int32_t)x.qs[x.rv ? x.Lq - 1 - i : i] : -1;
  }
  for (int sy = 0; sy <= sc.n; ++sy) {
    uint32_t w[XW];
#pragma unroll
    for (int k = 0; k < XW; ++k) w[k] = 0u;
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const uint32_t b = (qv[r] >= 0 && sy < sc.n) ? (uint32_t)(uint8_t)(s_mat[qv[r] * sc.n + sy] + sc.bias) : 0u;
      w[r >> 2] |= b << (8 * (r & 3));
    }
    uint8_t *dst = s_prof + ((int64_t)sy * 64 + lane) * RL;
    if constexpr (RL >= 4) lds_store_words<RL>(dst, w);
    else *reinterpret_cast<uint16_t *>(dst) = (uint16_t)w[0];
  }
}

// ---- several strips: strips first, first + stride, ... on this wave -----------
// Every producer of a strip is a wave that is running (the launches see to
// that) and no strip waits on a later one, so the waits end; a spin limit
// bounds them all the same (true: it was passed).
//
// Bound by the chain of strips: strip s + 1 follows strip s by the wavefront's
// 63 steps plus what the hand-over takes, once per strip.  The hand-over is one
// 64-bit word per column, valid << 63 | F << 32 | H, stored and loaded with
// relaxed agent-scope atomics: the word is its own flag, so no fence (a write
// back of the L2 per publish) and no progress counter stand between the store
// and the load, and 16 columns go at a time.  The words are cleared before the
// launch.  A block of 16 steps reads its words one block ahead and looks at
// them again only when some were not there yet.  With counters, fences and 64
// columns at a time a strip started 270 steps after the one above, now 110, which
// also makes short lanes (two rows: more strips, shorter steps) pay.
// Measured, 10,000 x 20,000 over 20 workgroups: forward 4.3 -> 2.3 ms,
// reversed 3.5 -> 1.65; a wait that polls without a pause slows the strips
// that work (50 such pairs reversed: 5.1 against 3.5 ms).
template <int RL, bool REV, bool HO>
__device__ __forceinline__ bool strips_of_wave(const StripJob &x, const StripScoring &sc,
                                               const int8_t *s_mat, uint8_t *s_prof, int first,
                                               int stride) {
  constexpr int SH = 64 * RL;
  constexpr int XW = RL >= 4 ? RL / 4 : 1;
  constexpr int kUnroll = RL <= 4 ? kSpreadBlock : (RL == 8 ? 4 : 1);
  constexpr int AGENT = __HIP_MEMORY_SCOPE_AGENT;
  using T = VT<uint32_t>;
  const int lane = threadIdx.x & 63;
  const int n = sc.n;
  const int64_t qp = ((int64_t)x.Lq + SH - 1) / SH * SH;
  const int nstrips = (int)(qp / SH);
  const int64_t qpad = REV ? 0 : qp - x.Lq;   // forward: padding rows on top
  const int kb = x.kb;
  const uint32_t M = (1u << kb) - 1u;
  const int32_t tgt = REV ? x.tgt : 0;
  const int64_t width = x.c1 - x.cw;
  const int8_t *rs = x.rs;
  const bool rv = x.rv;
  const int64_t Lr = x.Lr;
  uint32_t *mc = x.mc;
  const uint32_t vbias = sc.bias, vo = sc.o, ve = sc.e;
  bool spin_fail = false;

  // column window of strip s (the reversed pass bands it)
  auto window = [&](int s, int64_t &clo, int64_t &chi) {
    clo = x.cw;
    chi = x.c1;
    if (REV && x.band >= 0) {
      const int64_t l = (int64_t)s * SH - x.band;
      if (l > clo) clo = l;
      const int64_t h = (int64_t)s * SH + SH + x.band;
      if (h < chi) chi = h;
    }
    if (chi < clo) chi = clo;
  };

  for (int s = first; s < nstrips; s += stride) {
    int64_t clo, chi, plo = 0, phi = 0;
    window(s, clo, chi);
    if (s > 0) window(s - 1, plo, phi);
    uint64_t *out = x.rows + width * (int64_t)s;   // this strip's words
    const uint64_t *in = out - width;            // those of strip s - 1
    const bool hand_over = (s + 1 < nstrips);
    auto finish = [&]() {   // every word of the strip is stored
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (lane == 0) __hip_atomic_store(&x.done[s], 1, __ATOMIC_RELAXED, AGENT);
    };
    // the reversed pass skips a strip that cannot hold an earlier column
    if (chi <= clo ||
        (REV && __hip_atomic_load(x.best, __ATOMIC_RELAXED, AGENT) <= (unsigned long long)clo)) {
      finish();
      continue;
    }

    strip_profile<RL>(x, sc, s_mat, s_prof, (int64_t)s * SH + lane * RL - qpad);
    lds_wave_sync();

    // code offset of this lane's rows: code = M - padded row
    const uint32_t DL = M - (uint32_t)((int64_t)s * SH + lane * RL + RL - 1);

    // words of columns c0 .. c0 + cnt - 1 at lanes 0 .. cnt - 1; a column the
    // row above does not hold reads as a valid zero
    auto fetch = [&](int64_t c0, int cnt) -> uint64_t {
      const int64_t c = c0 + lane;
      const bool have = s > 0 && lane < cnt && c < chi && c >= plo && c < phi;
      return have ? __hip_atomic_load(in + (c - x.cw), __ATOMIC_RELAXED, AGENT) : kWordValid;
    };
    auto ready = [](uint64_t w) { return __ballot((w & kWordValid) != 0) == ~0ull; };
    // the same once they are all there; words the finished strip above never
    // stored read as zero
    auto settle = [&](uint64_t w, int64_t c0, int cnt) -> uint64_t {
      int64_t spins = 0;
      while (!ready(w)) {
        const int32_t done = __hip_atomic_load(&x.done[s - 1], __ATOMIC_RELAXED, AGENT);
        if (done) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        w = fetch(c0, cnt);
        if (done) break;
        if (++spins > kSpinLimit) { spin_fail = true; break; }
        __builtin_amdgcn_s_sleep(1);
      }
      return (w & kWordValid) ? w : kWordValid;
    };
    // reference symbols of columns [c0, c0 + 16) at lanes 0 .. 15 (n past the window)
    auto symbols = [&](int64_t c0) -> uint32_t {
      const int64_t c = c0 + lane;
      return lane < kSpreadBlock && c < chi ? (uint32_t)(uint8_t)rs[rv ? Lr - 1 - c : c] : (uint32_t)n;
    };

    uint32_t H[RL], E[RL];
#pragma unroll
    for (int r = 0; r < RL; ++r) { H[r] = 0u; E[r] = 0u; }
    uint32_t hup_prev = 0u;
    if (s > 0 && clo - 1 >= plo && clo - 1 < phi && clo >= 1) {
      const int64_t c = clo - 1;
      uint64_t w = lane == 0 ? __hip_atomic_load(in + (c - x.cw), __ATOMIC_RELAXED, AGENT) : kWordValid;
      int64_t spins = 0;
      while (!ready(w)) {
        const int32_t done = __hip_atomic_load(&x.done[s - 1], __ATOMIC_RELAXED, AGENT);
        if (done) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (lane == 0) w = __hip_atomic_load(in + (c - x.cw), __ATOMIC_RELAXED, AGENT);
        if (done) break;
        if (++spins > kSpinLimit) { spin_fail = true; break; }
      }
      hup_prev = lane == 0 ? (uint32_t)w : 0u;
    }
    uint32_t hout = 0u, fout = 0u, cmout = 0u;
    uint32_t obH = 0u, obF = 0u, obC = 0u;   // queues of lane 63's outputs, the newest at lane 63
    int64_t newest = clo - 64;               // ... of this column
    auto flush = [&]() {   // the last block's columns
      const int64_t c = newest - 63 + lane;
      if (lane >= 64 - kSpreadBlock && c >= clo && c < chi) {
        if (hand_over)
          __hip_atomic_store(out + (c - x.cw), kWordValid | ((uint64_t)obF << 32) | obH,
                             __ATOMIC_RELAXED, AGENT);
        if (!REV && c >= x.c0 && c < x.c1) atomicMax(&mc[c], obC);
      }
    };
    const int64_t nsteps = (chi - clo) + 63;
    // a step's symbol enters lane 0 one step ahead, with its profile row
    uint32_t sym = from_above((uint32_t)n, lane_value(symbols(clo), 0));
    uint32_t X[XW];
    prof_load<RL>(s_prof + ((int64_t)sym * 64 + lane) * RL, X);
    uint32_t symnext = symbols(clo + 1);
    uint64_t wnext = fetch(clo, kSpreadBlock);
#pragma unroll 1
    for (int64_t t0 = 0; t0 < nsteps; t0 += kSpreadBlock) {
      // this block's words were asked for one block ago; the last block's
      // outputs go out before anything waits
      uint64_t w = wnext;
      const bool here = ready(w);
      const uint32_t symbuf = symnext;
      flush();
      if (REV && (t0 & 63) == 0 && t0 >= 64 &&
          (unsigned long long)(clo + t0 - 63) >= __hip_atomic_load(x.best, __ATOMIC_RELAXED, AGENT))
        break;   // an earlier strip already reached the target at or before here
      if (!here) w = settle(w, clo + t0, kSpreadBlock);
      wnext = fetch(clo + t0 + kSpreadBlock, kSpreadBlock);
      symnext = symbols(clo + t0 + kSpreadBlock + 1);
      const uint32_t hbuf = (uint32_t)w, fbuf = (uint32_t)(w >> 32) & 0x7FFFFFFFu;
#pragma unroll kUnroll
      for (int tm = 0; tm < kSpreadBlock; ++tm) {
        const uint32_t hup = from_above(hout, lane_value(hbuf, tm));
        uint32_t F = from_above(fout, lane_value(fbuf, tm));
        const uint32_t cmin = from_above(cmout, 0u);
        const uint32_t symn = from_above(sym, lane_value(symbuf, tm));
        uint32_t Xn[XW];
        prof_load<RL>(s_prof + ((int64_t)symn * 64 + lane) * RL, Xn);
        uint32_t cm = 0u;
        uint32_t u_next = T::max(hup_prev + __builtin_amdgcn_ubfe(X[0], 0, 8), E[0]);
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          const uint32_t u = u_next;
          if (r + 1 < RL)
            u_next = T::max(H[r] + __builtin_amdgcn_ubfe(X[(r + 1) >> 2], 8 * ((r + 1) & 3), 8), E[r + 1]);
          const uint32_t hb = T::max(u, F);
          const uint32_t hn = T::subs(hb, vbias);
          H[r] = hn;
          const uint32_t enc = (hn << kb) + (uint32_t)(RL - 1 - r);
          cm = cm > enc ? cm : enc;
          const uint32_t ho = HO ? hn : T::subs(hb, vo);   // HO: bias == o
          E[r] = T::max(T::subs(E[r], ve), ho);
          F = T::max(T::subs(F, ve), ho);
        }
        hup_prev = hup;
        hout = H[RL - 1];
        fout = F;
        const uint32_t cml = cm + DL;
        cmout = cmin > cml ? cmin : cml;
        sym = symn;
#pragma unroll
        for (int k = 0; k < XW; ++k) X[k] = Xn[k];
        obH = shift_in(obH, hout);
        obF = shift_in(obF, fout);
        obC = shift_in(obC, cmout);
      }
      newest = clo + t0 + kSpreadBlock - 64;   // step t ends column clo + t - 63
      if constexpr (REV) {
        const int64_t c = newest - 63 + lane;
        const unsigned long long hit =
            __ballot(lane >= 64 - kSpreadBlock && c >= clo && c < chi && tgt > 0 && (int32_t)(obC >> kb) >= tgt);
        if (hit) {
          const int hl = __builtin_ctzll(hit);
          const uint32_t oc = lane_value(obC, hl);
          if (lane == 0) {
            x.rcol[s] = newest - 63 + hl;
            x.rrow[s] = (int32_t)(M - (oc & M));
            atomicMin(x.best, (unsigned long long)(newest - 63 + hl));
          }
          break;
        }
      }
    }
    flush();
    finish();
  }
  return spin_fail;
}

// ---- one strip (Lq <= 64 * RL) on this wave ------------------------------------
// Nothing is handed over, so no row enters lane 0 and only the column maxima
// leave lane 63; padding rows stand on top in both directions, and the lanes
// that hold nothing else are skipped: the reference symbols enter at the first
// lane with a row.  The row code counts padded rows from x.row0 on, so that
// strips of different heights can share one coding (64 * RL + x.row0 rows).
// Every owned column is this wave's alone: its max array words are stored, not
// merged.  Bound by instruction issue of one wave (about
// 48 per step and four rows; the sweep for several strips 73).  Reversed:
// *rcol, *rrow (query row) of the first column reaching the target, or -1;
// with an anchor above every score (Lq < 64 * RL then), the padding row above
// the first one starts from the anchor and holds the gap run that leaves it
// (a forward alignment may end in a deletion run), so that only paths from
// that corner can reach a target above the anchor.  LAST: only the last column's word is wanted, in *rrow.
// best (forward, may be null): the largest value's word and its first column.
struct StripBest {
  uint32_t word;   // max array word, this lane's until whole_wave
  int64_t col;     // -1: no value above 0
  __device__ __forceinline__ void take(uint32_t w, int64_t c, int kb) {
    if ((w >> kb) > (word >> kb)) {   // (a lane's columns come in order)
      word = w;
      col = c;
    }
  }
  __device__ __forceinline__ void whole_wave(int kb) {
    uint32_t v = word >> kb;
    int64_t c = v ? col : INT64_MAX;
    for (int off = 32; off >= 1; off >>= 1) {
      const uint32_t v2 = __shfl_xor(v, off, 64);
      const int64_t c2 = __shfl_xor(c, off, 64);
      if (v2 > v || (v2 == v && c2 < c)) { v = v2; c = c2; }
    }
    const unsigned long long own = __ballot((word >> kb) == v && col == c);
    word = v ? (uint32_t)__builtin_amdgcn_readlane((int)word, __builtin_ctzll(own | (1ull << 63))) : 0u;
    col = v ? c : -1;
  }
};
template <int RL, bool REV, bool HO, bool LAST = false>
__device__ __forceinline__ void strip_alone(const StripJob &x, const StripScoring &sc,
                                            const int8_t *s_mat, uint8_t *s_prof,
                                            StripBest *best = nullptr) {
  constexpr int SH = 64 * RL;
  constexpr int XW = RL >= 4 ? RL / 4 : 1;
  constexpr int kUnroll = RL <= 4 ? kSpreadBlock : (RL == 8 ? 4 : 1);
  using T = VT<uint32_t>;
  const int lane = threadIdx.x & 63;
  const int qpad = SH - x.Lq;
  // the first lane with a row of the query, or with the anchored row above it
  const int top = REV && x.anchor ? qpad - 1 : qpad;
  const int f = top < SH ? top / RL : 63;
  const uint32_t M = (1u << x.kb) - 1u;
  const uint32_t DL = M - (uint32_t)(x.row0 + lane * RL + RL - 1);
  const int64_t clo = x.cw;
  int64_t chi = x.c1;
  if (REV && x.band >= 0 && (int64_t)x.Lq + x.band < chi) chi = (int64_t)x.Lq + x.band;
  if (REV && lane == 0) {
    *x.rcol = -1;
    *x.rrow = -1;
  }
  strip_profile<RL>(x, sc, s_mat, s_prof, lane * RL - qpad);
  lds_wave_sync();
  auto symbols = [&](int64_t c0) -> uint32_t {
    const int64_t c = c0 + lane;
    return lane < kSpreadBlock && c < chi ? (uint32_t)(uint8_t)x.rs[x.rv ? x.Lr - 1 - c : c] : (uint32_t)sc.n;
  };
  const bool enter = lane == f;
  uint32_t H[RL], E[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) { H[r] = 0u; E[r] = 0u; }
  uint32_t hup_prev = 0u, hout = 0u, fout = 0u, cmout = 0u, obC = 0u;
  if constexpr (REV) {
    if (x.anchor) {
#pragma unroll
      for (int r = 0; r < RL; ++r)
        if (enter && r == top - f * RL) {
          H[r] = x.anchor;
          E[r] = x.anchor - sc.o + sc.bias;
        }
      hout = H[RL - 1];   // (the row below may be the next lane's)
    }
  }
  const uint32_t first = lane_value(symbols(clo), 0);   // (by every lane, not inside the choice)
  uint32_t sym = enter ? first : (uint32_t)sc.n;
  uint32_t X[XW];
  prof_load<RL>(s_prof + ((int64_t)sym * 64 + lane) * RL, X);
  uint32_t symnext = symbols(clo + 1);
  const int64_t nsteps = (chi - clo) + 63 - f;
#pragma unroll 1
  for (int64_t t0 = 0; t0 < nsteps; t0 += kSpreadBlock) {
    const uint32_t symbuf = symnext;
    symnext = symbols(clo + t0 + kSpreadBlock + 1);
#pragma unroll kUnroll
    for (int tm = 0; tm < kSpreadBlock; ++tm) {
      const uint32_t hup = from_above(hout, 0u);
      uint32_t F = from_above(fout, 0u);
      const uint32_t cmin = from_above(cmout, 0u);
      const uint32_t snew = lane_value(symbuf, tm);
      const uint32_t sdown = from_above(sym, (uint32_t)sc.n);
      const uint32_t symn = enter ? snew : sdown;
      uint32_t Xn[XW];
      prof_load<RL>(s_prof + ((int64_t)symn * 64 + lane) * RL, Xn);
      uint32_t cm = 0u;
      uint32_t u_next = T::max(hup_prev + __builtin_amdgcn_ubfe(X[0], 0, 8), E[0]);
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const uint32_t u = u_next;
        if (r + 1 < RL)
          u_next = T::max(H[r] + __builtin_amdgcn_ubfe(X[(r + 1) >> 2], 8 * ((r + 1) & 3), 8), E[r + 1]);
        const uint32_t hb = T::max(u, F);
        const uint32_t hn = T::subs(hb, sc.bias);
        H[r] = hn;
        const uint32_t enc = (hn << x.kb) + (uint32_t)(RL - 1 - r);
        cm = cm > enc ? cm : enc;
        const uint32_t ho = HO ? hn : T::subs(hb, sc.o);   // HO: bias == o
        E[r] = T::max(T::subs(E[r], sc.e), ho);
        F = T::max(T::subs(F, sc.e), ho);
      }
      hup_prev = hup;
      hout = H[RL - 1];
      fout = F;
      const uint32_t cml = cm + DL;
      cmout = cmin > cml ? cmin : cml;
      sym = symn;
#pragma unroll
      for (int k = 0; k < XW; ++k) X[k] = Xn[k];
      obC = shift_in(obC, cmout);
    }
    // lanes 48 .. 63 hold the block's 16 columns
    const int64_t c = clo + t0 + kSpreadBlock - 1 - (63 - f) - 63 + lane;
    const bool mine = lane >= 64 - kSpreadBlock && c >= clo && c < chi;
    if constexpr (REV) {
      const unsigned long long hit = __ballot(mine && x.tgt > 0 && (int32_t)(obC >> x.kb) >= x.tgt);
      if (hit) {
        const int hl = __builtin_ctzll(hit);
        if (lane == hl) {
          *x.rcol = c;
          *x.rrow = (int32_t)(M - (obC & M)) - qpad - x.row0;
        }
        break;
      }
    } else if constexpr (LAST) {
      if (mine && c == chi - 1) *x.rrow = (int32_t)obC;
    } else {
      if (mine && c >= x.c0) {
        x.mc[c] = obC;
        if (best) best->take(obC, c, x.kb);
      }
    }
  }
}

// ---- one strip of two pairs on packed 16-bit lanes -------------------------------
// The forward sweep of strip_alone for two pairs (A in the low halves, B in
// the high ones; B may be absent: width 0) whose scores stay below 2^15: one
// packed instruction updates a cell of each.  Row-code bits 16.  M3: every
// lane value stays below 0x7C00, so H is one packed three-way maximum; HO: the
// bias is the gap open penalty.  s_profA, s_profB: a profile each.
template <int RL, bool M3, bool HO>
__device__ __forceinline__ void strip_alone16(const StripJob &x, const StripJob &y,
                                              const StripScoring &sc, const int8_t *s_mat,
                                              uint8_t *s_profA, uint8_t *s_profB,
                                              StripBest &bestA, StripBest &bestB) {
  constexpr int SH = 64 * RL;
  constexpr int kUnroll = RL <= 4 ? kSpreadBlock : 4;
  using T = VT<u16x2>;
  const int lane = threadIdx.x & 63;
  const int qpadA = SH - x.Lq, qpadB = SH - y.Lq;
  const int qpad = qpadA < qpadB ? qpadA : qpadB;
  const int f = qpad < SH ? qpad / RL : 63;   // the first lane with a row of either
  const uint32_t DL = 65535u - (uint32_t)(x.row0 + lane * RL + RL - 1);
  const int64_t wA = x.c1 - x.cw, wB = y.c1 - y.cw;
  const int64_t width = wA > wB ? wA : wB;
  strip_profile<RL>(x, sc, s_mat, s_profA, lane * RL - qpadA);
  strip_profile<RL>(y, sc, s_mat, s_profB, lane * RL - qpadB);
  lds_wave_sync();
  // both pairs' symbols of step offsets [o0, o0 + 16), A in the low byte
  const int8_t *ra = x.rs + x.cw, *rb = y.rs + y.cw;
  auto symbols = [&](int64_t o0) -> uint32_t {
    const int64_t off = o0 + lane;
    const uint32_t a = lane < kSpreadBlock && off < wA ? (uint32_t)(uint8_t)ra[off] : (uint32_t)sc.n;
    const uint32_t b = lane < kSpreadBlock && off < wB ? (uint32_t)(uint8_t)rb[off] : (uint32_t)sc.n;
    return a | (b << 8);
  };
  const bool enter = lane == f;
  const u16x2 vbias = T::splat(sc.bias), vo = T::splat(sc.o), ve = T::splat(sc.e);
  const uint32_t selA = 0x05040100u, selB = 0x07060100u;   // a half of H above a 16-bit code
  const uint32_t none = (uint32_t)sc.n * 0x101u;
  u16x2 H[RL], E[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) { H[r] = T::zero(); E[r] = T::zero(); }
  u16x2 hup_prev = T::zero(), hout = T::zero(), fout = T::zero();
  uint32_t cmoutA = 0u, cmoutB = 0u, obA = 0u, obB = 0u;
  const uint32_t first = lane_value(symbols(0), 0);
  uint32_t sym = enter ? first : none;
  uint32_t XA[RL / 4], XB[RL / 4];
  lds_load_words<RL>(s_profA + ((int64_t)(sym & 0xFFu) * 64 + lane) * RL, XA);
  lds_load_words<RL>(s_profB + ((int64_t)((sym >> 8) & 0xFFu) * 64 + lane) * RL, XB);
  uint32_t symnext = symbols(1);
  const int64_t nsteps = width + 63 - f;
#pragma unroll 1
  for (int64_t t0 = 0; t0 < nsteps; t0 += kSpreadBlock) {
    const uint32_t symbuf = symnext;
    symnext = symbols(t0 + kSpreadBlock + 1);
#pragma unroll kUnroll
    for (int tm = 0; tm < kSpreadBlock; ++tm) {
      const u16x2 hup = T::from(from_above(T::bits(hout), 0u));
      u16x2 F = T::from(from_above(T::bits(fout), 0u));
      const uint32_t cminA = from_above(cmoutA, 0u), cminB = from_above(cmoutB, 0u);
      const uint32_t snew = lane_value(symbuf, tm);
      const uint32_t sdown = from_above(sym, none);
      const uint32_t symn = enter ? snew : sdown;
      uint32_t XnA[RL / 4], XnB[RL / 4];
      lds_load_words<RL>(s_profA + ((int64_t)(symn & 0xFFu) * 64 + lane) * RL, XnA);
      lds_load_words<RL>(s_profB + ((int64_t)((symn >> 8) & 0xFFu) * 64 + lane) * RL, XnB);
      uint32_t cmA = 0u, cmB = 0u;
      auto score_of = [&](int r) -> u16x2 { return T::from(perm(XB[r >> 2], XA[r >> 2], T::sel_const(r & 3))); };
      u16x2 u_next = M3 ? T::add(hup_prev, score_of(0)) : T::max(T::add(hup_prev, score_of(0)), E[0]);
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const u16x2 u = u_next;
        if (r + 1 < RL) {
          u_next = T::add(H[r], score_of(r + 1));
          if constexpr (!M3) u_next = T::max(u_next, E[r + 1]);
        }
        u16x2 hb;
        if constexpr (M3) hb = T::max3(u, E[r], F);
        else hb = T::max(u, F);
        const u16x2 hn = T::subs(hb, vbias);
        H[r] = hn;
        const uint32_t kc = (uint32_t)(RL - 1 - r);
        const uint32_t wa = perm(T::bits(hn), kc, selA), wb = perm(T::bits(hn), kc, selB);
        cmA = cmA > wa ? cmA : wa;
        cmB = cmB > wb ? cmB : wb;
        const u16x2 ho = HO ? hn : T::subs(hb, vo);
        E[r] = T::max(T::subs(E[r], ve), ho);
        F = T::max(T::subs(F, ve), ho);
      }
      hup_prev = hup;
      hout = H[RL - 1];
      fout = F;
      const uint32_t cmlA = cmA + DL, cmlB = cmB + DL;
      cmoutA = cminA > cmlA ? cminA : cmlA;
      cmoutB = cminB > cmlB ? cminB : cmlB;
      sym = symn;
#pragma unroll
      for (int k = 0; k < RL / 4; ++k) { XA[k] = XnA[k]; XB[k] = XnB[k]; }
      obA = shift_in(obA, cmoutA);
      obB = shift_in(obB, cmoutB);
    }
    const int64_t off = t0 + kSpreadBlock - 1 - (63 - f) - 63 + lane;
    if (lane >= 64 - kSpreadBlock && off >= 0) {
      if (off < wA && x.cw + off >= x.c0) {
        x.mc[x.cw + off] = obA;
        bestA.take(obA, x.cw + off, 16);
      }
      if (off < wB && y.cw + off >= y.c0) {
        y.mc[y.cw + off] = obB;
        bestB.take(obB, y.cw + off, 16);
      }
    }
  }
}

}  // namespace swx
