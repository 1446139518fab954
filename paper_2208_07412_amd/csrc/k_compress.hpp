// Track-model cluster compression (encoder and decoder) and the track-cluster
// residual histograms.
//
// Format (stated field by field in include/tpc.h): a header, a directory of
// bit offsets (one per track record, one per (unit,row) block of clusters on
// no track) and an LSB-first bit stream of Exp-Golomb codes.  Positions are
// quantised to 2^-7 cm; a cluster on a track is coded as its residual to an
// integer helix evaluated row by row from the track's fitted parameters, so
// every value in the stream is integer arithmetic and decoding gives the
// quantised clusters whatever the model predicts.
//
// Encoder: one wave per track codes its hits, 64 at a time on a table of the
// helix at the rows they span, and keeps each hit's code for the writing pass
// (with the record's length and the residual histograms); one workgroup per
// (unit,row) the lengths of its clusters on no track; two device scans turn the
// lengths into the directory; a finishing kernel writes the header and checks
// the capacity; the payload is cleared and written, records and row blocks put
// together in LDS and stored in whole words (atomic OR only where a word is
// shared with a neighbour).  Decoder: the record sizes come
// from the directory and the fixed-width hit counts, a scan gives the output
// offsets, and one lane per record decodes it.
#pragma once

#include "common.hpp"

#define CM_MAGIC 0x54434D31u
#define CM_HDR 8
#define CM_VERSION 2u
#define CM_CHUNK 64  // clusters on no track per independently decodable chunk of a row
#define CM_STAGE_WORDS 3072  // LDS words per wave for staging a record
#define CM_QSHIFT 9  // positions quantised to 2^(9-16) cm

// ---------------------------------------------------------------- arithmetic
__device__ __forceinline__ int64_t cm_q(int64_t v) { return (v + 256) >> CM_QSHIFT; }

// a / 2^k rounded to the nearest integer, halves up (arithmetic shift = floor)
__device__ __forceinline__ int64_t cm_rshift(int64_t a, int k) {
  return (a + ((int64_t)1 << (k - 1))) >> k;
}
// a / d rounded to the nearest integer, halves up: floor((2a + d) / 2d).  In
// the helix step 2^25 < d <= 2^31 and |a| < 2^56, so the quotient is below
// 2^31 and the double quotient (two roundings, relative error <= 2^-52) is
// within 2^-21 of it: its floor is off by at most one, which the exact
// remainder repairs.  (A 64-bit integer division is a long software sequence
// on the GPU.)
__device__ __forceinline__ int64_t cm_rdiv(int64_t a, int64_t d) {
  const int64_t n = 2 * a + d, m = 2 * d;
  int64_t q = (int64_t)floor((double)n / (double)m);
  const int64_t r = n - q * m;
  if (r < 0) --q;
  else if (r >= m) ++q;
  return q;
}
// floor(sqrt(n)), n < 2^62: the double square root is within 2^-20 of the root
// (the conversion and the root each round once), so its floor is off by at most
// one either way, which two exact squares decide (0 for n <= 0, which only a
// malformed record reaches).  The root is below 2^31: its square is one 32-bit
// product, where a 64-bit one takes several.
__device__ __forceinline__ int64_t cm_isqrt(int64_t n) {
  if (n <= 0) return 0;
  uint32_t r = (uint32_t)sqrt((double)n);
  r -= (uint64_t)r * r > (uint64_t)n ? 1u : 0u;
  r += (uint64_t)(r + 1) * (r + 1) <= (uint64_t)n ? 1u : 0u;
  return (int64_t)r;
}
// product of two values that fit 32 bits
__device__ __forceinline__ int64_t cm_mul32(int64_t a, int64_t b) {
  return (int64_t)(int32_t)a * (int32_t)b;
}
__device__ __forceinline__ uint64_t cm_zig(int64_t v) {
  return v >= 0 ? (uint64_t)v << 1 : ((uint64_t)(-v) << 1) - 1;
}
__device__ __forceinline__ int64_t cm_unzig(uint64_t u) {
  return (u & 1) ? -(int64_t)((u + 1) >> 1) : (int64_t)(u >> 1);
}
// length of the order-k Exp-Golomb code of v
__device__ __forceinline__ uint32_t cm_eg_len(uint64_t v, int k) {
  const uint64_t q = (v >> k) + 1;
  const uint32_t n = 63 - __builtin_clzll(q);
  return 2 * n + 1 + k;
}

// The order-k Exp-Golomb code of v, first bit lowest, and its length; the
// value holds the whole code up to 64 bits.
__device__ __forceinline__ uint64_t cm_eg_code(uint64_t v, int k, uint32_t& len) {
  const uint64_t q = (v >> k) + 1;
  const uint32_t n = 63 - __builtin_clzll(q);
  len = 2 * n + 1 + k;
  const uint64_t low = q ^ (1ull << n);
  uint64_t c = 1ull << n;
  if (n < 32) c |= low << (n + 1);
  if (2 * n + 1 < 64) c |= (v & ((1ull << k) - 1)) << (2 * n + 1);
  return c;
}

// The same for codes of at most 32 bits.
__device__ __forceinline__ uint32_t cm_eg_code32(uint32_t v, int k, uint32_t& len) {
  const uint32_t q = (v >> k) + 1;
  const uint32_t n = 31 - __builtin_clz(q);
  len = 2 * n + 1 + k;
  return (1u << n) | ((q ^ (1u << n)) << (n + 1)) | ((v & ((1u << k) - 1)) << (2 * n + 1));
}

// OR of the bits v (up to 64) into LDS words from bit position at on.
__device__ __forceinline__ void cm_lds_or(uint32_t* words, uint32_t at, uint64_t v) {
  uint32_t* w = words + (at >> 5);
  const uint32_t sh = at & 31;
  const uint64_t lo = v << sh;
  if ((uint32_t)lo) atomicOr(&w[0], (uint32_t)lo);
  if ((uint32_t)(lo >> 32)) atomicOr(&w[1], (uint32_t)(lo >> 32));
  const uint32_t top = sh ? (uint32_t)(v >> (64 - sh)) : 0u;
  if (top) atomicOr(&w[2], top);
}

// Words put together in LDS (word 0 = payload word first) stored into the
// stream, by lanes i0, i0 + di, ...: the bits [b0, b1) are this writer's, so
// words inside them are stored plainly, those at their ends by atomic OR.
__device__ __forceinline__ void cm_store_words(const uint32_t* words, uint32_t* payload,
                                               uint64_t limit, uint64_t b0, uint64_t b1,
                                               uint32_t i0, uint32_t di) {
  if (b1 <= b0) return;
  const uint64_t first = b0 >> 5, n = ((b1 + 31) >> 5) - first;
  for (uint64_t i = i0; i < n; i += di) {
    const uint64_t at = first + i;
    if (at >= limit) continue;
    if (at * 32 >= b0 && (at + 1) * 32 <= b1) payload[at] = words[i];
    else if (words[i]) atomicOr(&payload[at], words[i]);
  }
}

// Integer helix of one track (y, z in 2^-16 cm; sin phi, tan lambda in 2^-30;
// C in 2^-46 per cm), stepped outward one row at a time.  Sc is
// floor(sqrt(2^60 - S^2)) of the current S, kept so that a step computes one
// such root for its new S instead of two.
struct CmModel {
  int64_t Y, Z, S, T, C, Sc;
  int row;
  bool frozen;
};

struct CmParams {  // the track's integers as stored in its record
  int64_t Y, Z, S, T, K;
};

// From the float32 parameters: each scaled by a power of two (exact) and
// rounded to the nearest integer, ties to even.
__device__ __forceinline__ CmParams cm_params(const float* p, int32_t z_anchor) {
  CmParams m;
  const int64_t lim = ((int64_t)1 << 30) - 1;
  int64_t S = (int64_t)rintf(p[2] * 1073741824.0f);
  int64_t T = (int64_t)rintf(p[3] * 1073741824.0f);
  int64_t K = (int64_t)rintf(p[4] * 65536.0f);
  S = S > lim ? lim : (S < -lim ? -lim : S);
  T = T > 4 * lim ? 4 * lim : (T < -4 * lim ? -4 * lim : T);
  K = K > 20 * 65536 ? 20 * 65536 : (K < -20 * 65536 ? -20 * 65536 : K);
  m.Y = (int64_t)rintf(p[0] * 65536.0f);
  m.Z = (int64_t)rintf(p[1] * 65536.0f) + z_anchor;
  m.S = S;
  m.T = T;
  m.K = K;
  return m;
}

__device__ __forceinline__ CmModel cm_model(const CmParams& q, int64_t b30, int row) {
  return CmModel{q.Y, q.Z, q.S, q.T, -b30 * q.K, cm_isqrt(((int64_t)1 << 60) - q.S * q.S), row,
                 false};
}

__device__ __forceinline__ void cm_step(CmModel& m, const int32_t* xfx) {
  const int a = m.row;
  m.row = a + 1;
  if (m.frozen || a + 1 >= NROW) return;
  const int64_t D = (int64_t)xfx[a + 1] - xfx[a];
  const int64_t S1 = m.S + cm_rshift(m.C * D, 32);
  const int64_t smax = ((int64_t)1 << 30) - ((int64_t)1 << 20);
  if (S1 >= smax || S1 <= -smax) {
    m.frozen = true;
    return;
  }
  const int64_t one = (int64_t)1 << 60;
  // row distances, S (below 2^30 here), F (below 2^31: S1 leaves a root above
  // 2^25) and the root with F fit 32 bits
  const int64_t c1 = cm_isqrt(one - cm_mul32(S1, S1));
  const int64_t F = cm_rdiv((m.S + S1) * ((int64_t)1 << 24), m.Sc + c1);
  m.Y += cm_rshift(cm_mul32(D, F), 24);
  const int64_t L = cm_rshift(cm_mul32(D, cm_isqrt(((int64_t)1 << 48) + cm_mul32(F, F))), 24);
  m.Z += cm_rshift(m.T * L, 30);
  m.S = S1;
  m.Sc = c1;
}

// (unit,row) of cluster c: the last entry of crow[0..n_ur) not above c
__device__ __forceinline__ uint32_t cm_find_ur(const uint32_t* crow, uint32_t n_ur, uint32_t c) {
  uint32_t lo = 0, hi = n_ur;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (crow[mid] <= c) lo = mid;
    else hi = mid;
  }
  return lo;
}

// ------------------------------------------------------------- bit writing
// One lane's sequential writer over a contiguous bit range: completed words
// are OR-ed into the (cleared) stream, the last partial word at the end.
struct CmWriter {
  uint32_t* w;
  uint64_t limit;  // payload words (no store beyond them, whatever the lengths)
  uint64_t pos;
  uint64_t acc;   // pending bits, the lowest at stream position (pos & ~31)
  uint32_t nacc;  // pending bit count = pos & 31 plus what was added
  __device__ void init(uint32_t* words, uint64_t n_words, uint64_t bitpos) {
    w = words;
    limit = n_words;
    pos = bitpos;
    acc = 0;
    nacc = (uint32_t)(bitpos & 31);
  }
  __device__ void store(uint64_t word, uint32_t v) {
    if (word < limit && v) atomicOr(&w[word], v);
  }
  __device__ void put(uint64_t v, uint32_t n) {  // n <= 32
    if (n == 0) return;
    v &= (n == 64) ? ~0ull : ((1ull << n) - 1);
    acc |= v << nacc;
    nacc += n;
    pos += n;
    if (nacc >= 32) {
      store((pos - nacc) >> 5, (uint32_t)acc);
      acc >>= 32;
      nacc -= 32;
    }
  }
  __device__ void eg(uint64_t v, int k) {
    const uint64_t q = (v >> k) + 1;
    const uint32_t n = 63 - __builtin_clzll(q);
    // n zeros, a one, the n low bits of q, the k low bits of v
    for (uint32_t z = n; z > 0;) {
      const uint32_t m = z > 32 ? 32 : z;
      put(0, m);
      z -= m;
    }
    put(1, 1);
    put(q, n);
    put(v, k);
  }
  __device__ void flush() {
    if (nacc) store((pos - nacc) >> 5, (uint32_t)acc);
    nacc = 0;
    acc = 0;
  }
};

// ------------------------------------------------------------- bit reading
// Sequential reader of a bit range; w points at payload word woff (a staged
// copy in LDS, or the payload itself with woff = 0).
// LSB-first reader over payload words w (w[0] is payload word woff) with a
// 64-bit bit buffer: one word read per 32 bits consumed.  Bits at or past
// `end` read as zero; a read that would pass `end` (or a zero prefix longer
// than 31) marks the reader bad and moves it to `end`.  P is the word
// pointer: global, or LDS for a staged record (an LDS pointer keeps the
// reads off the counter that the decoder's global stores also raise, so a
// read does not wait for the stores before it).
typedef const __attribute__((address_space(3))) uint32_t lds_u32;
template <typename P>
struct CmReaderT {
  P w;
  uint64_t pos, end;  // next bit, end of the readable bits (payload bits)
  bool bad;
  uint64_t woff;
  uint64_t buf;    // bits from pos on; nbuf of them loaded, zeros above
  uint32_t nbuf;
  uint64_t wnext;  // payload index of the next word to load
  __device__ CmReaderT(P w_, uint64_t pos_, uint64_t end_, bool bad_, uint64_t woff_)
      : w(w_), pos(0), end(end_), bad(bad_), woff(woff_), buf(0), nbuf(0), wnext(0) {
    seek(pos_);
  }
  __device__ void seek(uint64_t p) {
    pos = p;
    buf = 0;
    nbuf = 0;
    wnext = p >> 5;
    if (p < end) {
      buf = (uint64_t)(w[wnext - woff] >> (uint32_t)(p & 31));
      nbuf = 32 - (uint32_t)(p & 31);
      ++wnext;
    }
  }
  // at least 32 loaded bits, or every word up to the one holding end - 1
  __device__ void fill() {
    if (nbuf < 32 && (wnext << 5) < end) {
      buf |= (uint64_t)w[wnext - woff] << nbuf;
      nbuf += 32;
      ++wnext;
    }
  }
  __device__ void skip(uint32_t n) {
    buf >>= n;
    nbuf -= n;
    pos += n;
  }
  __device__ void fail() {
    bad = true;
    pos = end;
    buf = 0;
    nbuf = 0;
  }
  __device__ uint64_t get(uint32_t n) {  // n <= 32
    if (n == 0) return 0;
    if (pos + n > end) {
      fail();
      return 0;
    }
    fill();
    const uint64_t v = buf & ((1ull << n) - 1);
    skip(n);
    return v;
  }
  // up to 32 bits from pos on without advancing (bits past the end read 0)
  __device__ uint32_t peek32() {
    if (pos >= end) return 0;
    fill();
    uint32_t v = (uint32_t)buf;
    const uint64_t avail = end - pos;
    if (avail < 32) v &= (1u << (uint32_t)avail) - 1u;
    return v;
  }
  __device__ uint64_t eg(int k) {
    // the zero prefix: the trailing zeros of the next 32 bits (LSB first)
    const uint32_t v = peek32();
    if (v == 0) {  // no one bit among the next 32: malformed
      fail();
      return 0;
    }
    const uint32_t n = (uint32_t)__builtin_ctz(v);
    skip(n + 1);
    const uint64_t q = (1ull << n) | get(n);
    return ((q - 1) << k) | get(k);
  }
};
typedef CmReaderT<const uint32_t*> CmReader;

// -------------------------------------------------------------- cluster view
struct CmClusters {
  const uint32_t* crow;
  const int32_t *y, *z;
  const uint16_t *qtot, *qmax;
  const uint8_t* flags;
  const uint32_t* n_dev;
  uint32_t cap;
  uint32_t n_ur;
};

struct CmTracks {
  const float* par;
  const uint8_t* row;
  const int32_t* z_anchor;
  const uint32_t* hit_start;
  const uint32_t* hits;
  const int32_t* cluster_track;
  const uint32_t* n_dev;
  uint32_t cap, hit_cap;
};

__device__ __forceinline__ uint32_t cm_cluster_len(uint16_t qt, uint16_t qm) {
  return cm_eg_len(qt, 6) + cm_eg_len(qm, 5) + 2;
}
__device__ __forceinline__ void cm_cluster_put(CmWriter& b, uint16_t qt, uint16_t qm, uint8_t f) {
  b.eg(qt, 6);
  b.eg(qm, 5);
  b.put(f & 3u, 2);
}

// (unit,row) of cluster c found by a whole wave (every lane gets it): the
// last entry of crow[0..n_ur) not above c, as cm_find_ur; each round probes
// 64 evenly spaced entries, so 5,472 rows take three dependent loads.
__device__ __forceinline__ uint32_t cm_find_ur_wave(const uint32_t* crow, uint32_t n_ur,
                                                    uint32_t c) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t lo = 0, hi = n_ur;
  while (hi - lo > 1) {  // uniform
    const uint32_t step = (hi - lo + 63) / 64;
    const uint32_t p = lo + lane * step;
    // the probes not above c are a prefix of the lanes (crow does not decrease)
    const uint64_t b = __ballot(p < hi && crow[p] <= c);
    lo += (b ? 63u - (uint32_t)__builtin_clzll(b) : 0u) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

__device__ __forceinline__ uint32_t cm_wave_incl_max(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v = max(v, o);
  }
  return v;
}

// The helix m at every row from m.row (< NROW) to the last, one wave: q(y)
// and q(z) at row r in ty[r] and tz[r].  Along a track C is constant, so the
// S after each step is S0 plus a prefix sum of per-step increments, and a
// step's changes of y and z depend only on the S before and after it: wave
// prefix sums give the same integers as cm_step row after row.  The first
// step whose S leaves the range freezes that step and all after it.  Rows past
// row_end are left out where they would take another round.  Ends with the
// table visible to the whole wave.
__device__ __forceinline__ void cm_helix_rows(const CmModel& m, const int32_t* xs, int64_t* ty,
                                              int64_t* tz, int row_end) {
  const uint32_t lane = threadIdx.x & 63;
  const int64_t one = (int64_t)1 << 60;
  const int64_t smax = ((int64_t)1 << 30) - ((int64_t)1 << 20);
  int64_t S = m.S, Sc = m.Sc, Y = m.Y, Z = m.Z;
  bool frozen = false;
  if (lane == 0) {
    ty[m.row] = cm_q(Y);
    tz[m.row] = cm_q(Z);
  }
  for (int base = m.row; base < row_end && base + 1 < NROW; base += 64) {  // uniform
    const int a = base + (int)lane;  // this lane's step: row a to row a + 1
    const bool valid = a + 1 < NROW;
    const int64_t D = valid ? (int64_t)xs[a + 1] - xs[a] : 0;
    const int64_t inc = valid ? cm_rshift(m.C * D, 32) : 0;
    const int64_t S1 = S + (int64_t)wave_incl_scan((uint64_t)inc);
    const int64_t S0 = S1 - inc;
    const uint64_t out = __ballot(valid && (S1 >= smax || S1 <= -smax));
    const uint32_t first_out = out ? (uint32_t)__builtin_ctzll(out) : 64u;
    const bool live = valid && !frozen && lane < first_out;  // a prefix of the lanes
    const int64_t c1 = live ? cm_isqrt(one - cm_mul32(S1, S1)) : 0;
    const int64_t c_up = __shfl_up(c1, 1, 64);
    const int64_t c0 = lane == 0 ? Sc : c_up;
    int64_t dY = 0, dZ = 0;
    if (live) {
      const int64_t F = cm_rdiv((S0 + S1) * ((int64_t)1 << 24), c0 + c1);
      dY = cm_rshift(cm_mul32(D, F), 24);
      const int64_t L = cm_rshift(cm_mul32(D, cm_isqrt(((int64_t)1 << 48) + cm_mul32(F, F))), 24);
      dZ = cm_rshift(m.T * L, 30);
    }
    const int64_t Y1 = Y + (int64_t)wave_incl_scan((uint64_t)dY);
    const int64_t Z1 = Z + (int64_t)wave_incl_scan((uint64_t)dZ);
    if (valid) {
      ty[a + 1] = cm_q(Y1);
      tz[a + 1] = cm_q(Z1);
    }
    // the state after the last of these 64 steps (S and its root matter only
    // while nothing is frozen)
    Y = __shfl(Y1, 63, 64);
    Z = __shfl(Z1, 63, 64);
    S = __shfl(S1, 63, 64);
    Sc = __shfl(c1, 63, 64);
    if (out) frozen = true;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A hit's code as the sizing pass keeps it for the writing pass: the first 57
// bits of the code and its length in the top 7 bits; the next 57 bits in a
// second word where the code has more; length CM_LONG where it has more than
// 114 (the writing pass then codes the track anew).
#define CM_KEEP 57
#define CM_LONG 127u

// The code of one hit and its length (parts: row step, y and z residual,
// charges, flags), kept in res[hh] (and res[res_cap + hh]) when `keep`.
__device__ __forceinline__ uint32_t cm_hit_code(uint64_t stp, uint64_t zy, uint64_t zz, uint16_t qt,
                                                uint16_t qm, uint8_t fl, bool keep,
                                                uint64_t* __restrict__ res, uint32_t res_cap,
                                                uint32_t hh) {
  // row steps (at most 152: 15 bits) and charges (16 bits: 27 and 28 bits)
  // always have short codes, residuals below 2^15 too (29 bits)
  uint32_t l0, l1, l2, l3, l4;
  const uint64_t c0 = cm_eg_code32((uint32_t)stp, 0, l0);
  uint64_t c1, c2;
  if (__ballot(((zy | zz) >> 15) != 0) == 0) {
    c1 = cm_eg_code32((uint32_t)zy, 2, l1);
    c2 = cm_eg_code32((uint32_t)zz, 2, l2);
  } else {
    c1 = cm_eg_code(zy, 2, l1);
    c2 = cm_eg_code(zz, 2, l2);
  }
  const uint64_t c3 = cm_eg_code32(qt, 6, l3), c4 = cm_eg_code32(qm, 5, l4);
  const uint32_t len = l0 + l1 + l2 + l3 + l4 + 2;
  if (!keep) return len;
  if (len <= CM_KEEP) {
    uint64_t v = fl & 3u;
    v = (v << l4) | c4;
    v = (v << l3) | c3;
    v = (v << l2) | c2;
    v = (v << l1) | c1;
    v = (v << l0) | c0;
    res[hh] = v | ((uint64_t)len << CM_KEEP);
  } else if (len <= 2 * CM_KEEP && l1 <= 64 && l2 <= 64) {
    unsigned __int128 v = fl & 3u;
    v = (v << l4) | c4;
    v = (v << l3) | c3;
    v = (v << l2) | c2;
    v = (v << l1) | c1;
    v = (v << l0) | c0;
    res[hh] = ((uint64_t)v & ((1ull << CM_KEEP) - 1)) | ((uint64_t)len << CM_KEEP);
    res[(size_t)res_cap + hh] = (uint64_t)(v >> CM_KEEP);
  } else {
    res[hh] = (uint64_t)CM_LONG << CM_KEEP;
  }
  return len;
}

// Per-wave LDS of the track passes: the helix table and row starts of the
// sizing pass, or the writing pass's record (which needs either).
#define CM_REC_WORDS 1024  // most words of a record put together in LDS
union CmTrackLds {
  struct {
    int64_t ty[NROW], tz[NROW];  // q(y), q(z) of the helix per row
    uint32_t rw[NROW + 1];       // row starts of the track's unit
  } t;
  uint32_t rec[CM_REC_WORDS + 4];
};

// One track hit by hit, whatever its order and rows: a hit's (unit,row) is the
// largest reached so far (rows are searched forward only), the helix is taken
// at the highest row reached so far (it is never stepped back).  Calls
// hit(active, hit, cluster, row step, row of the helix) for 64 hits at a time by
// the whole wave; true if a hit lies past the clusters or below its track's row.
template <class Fn>
__device__ bool cm_track_hits(const CmClusters& cl, const uint32_t* __restrict__ hits,
                              const uint32_t* rw, uint32_t ub, bool staged, uint32_t n_cl,
                              uint32_t h0, uint32_t h1, uint32_t ur0, int r0, int rt, Fn hit) {
  const uint32_t lane = threadIdx.x & 63;
  bool bad = false;
  uint32_t ur_c = ur0;  // the (unit,row) reached so far
  int prev_c = r0;      // the previous hit's row (the track's row before the first)
  int mrow_c = rt;      // the helix's row so far
  for (uint32_t base = h0; base < h1; base += 64) {  // uniform
    const uint32_t hh = base + lane;
    const bool act = hh < h1;
    uint32_t c = act ? hits[hh] : 0u;
    if (c >= n_cl) {
      bad = bad || act;
      c = 0;
    }
    uint32_t f;
    if (staged && c >= rw[0] && c < rw[NROW]) {
      uint32_t lo = 0, hi = NROW;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (rw[mid] <= c) lo = mid;
        else hi = mid;
      }
      f = ub + lo;
    } else {
      f = cm_find_ur(cl.crow, cl.n_ur, c);
    }
    const uint32_t u = cm_wave_incl_max(act ? max(f, ur_c) : ur_c);
    const int r = (int)(u % NROW);
    const int r_up = __shfl_up(r, 1, 64);
    const int prev = lane == 0 ? prev_c : r_up;
    const int step = r - prev - (hh > h0 ? 1 : 0);
    if (act && step < 0) bad = true;
    const int mr = (int)cm_wave_incl_max((uint32_t)(act ? max(r, mrow_c) : mrow_c));
    hit(act, hh, c, step < 0 ? (uint64_t)0 : (uint64_t)step, mr);
    // the carries: the last hit of these 64
    const int last = (int)min(63u, h1 - 1 - base);
    ur_c = __shfl(u, last, 64);
    prev_c = __shfl(r, last, 64);
    mrow_c = __shfl(mr, last, 64);
  }
  return bad;
}

// Per-track record lengths, the hits' codes (kept for the writing pass), the
// track's unit and the residual histograms (per workgroup in LDS, then added to
// the caller's).  One wave takes CM_RUN consecutive tracks, which mostly lie in
// one unit, so its row starts stay staged in LDS from track to track.  A track of
// at most 64 hits in ascending rows of one unit (any that the library fits up to
// that length) is coded in one go: every hit's row from a search of the staged
// starts, the helix up to the last hit's row; others go hit by hit (same codes).
// Bound by instruction issue (the integer helix: 64-bit products, FP64 roots).
// On the 2 ms slice (3.7e5 tracks, 1.3e7 hits) 0.71 ms, 0.92 before; held to five
// waves per SIMD (94 VGPRs; four 0.09 ms slower, six spills).  Loading the next
// tracks' hits and fields ahead was slower (0.83 ms: more registers than it hides).
#define CM_RUN 8
#define CM_FIXED (8 + 16 + 8 + 5 * 32)  // bits of a record's fixed fields
// tracks per wave: CM_RUN, fewer where that would leave waves of the grid without any
__device__ __forceinline__ uint32_t cm_run(uint32_t n) {
  const uint32_t waves = gridDim.x * (blockDim.x >> 6);
  return min((uint32_t)CM_RUN, (n + waves - 1) / waves);
}
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_cm_track_bits(CmClusters cl, CmTracks tr, int64_t b30,
                                                       const DevParams* __restrict__ P,
                                                       uint32_t* __restrict__ tbits,
                                                       uint16_t* __restrict__ tunit,
                                                       uint32_t* __restrict__ hist_out,
                                                       uint64_t* __restrict__ res, uint32_t res_cap,
                                                       DevStatus* st) {
  __shared__ uint32_t h[256];
  __shared__ int32_t xs[NROW];
  __shared__ CmTrackLds lds[4];
  if (failed_wg(st)) return;
  for (uint32_t i = threadIdx.x; i < 256; i += blockDim.x) h[i] = 0;
  for (uint32_t i = threadIdx.x; i < NROW; i += blockDim.x) xs[i] = P->xfx[i];
  __syncthreads();
  const uint32_t n = scan_count(tr.n_dev, tr.cap);
  const uint32_t n_cl = scan_count(cl.n_dev, cl.cap);
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int64_t* ty = lds[w].t.ty;
  int64_t* tz = lds[w].t.tz;
  uint32_t* rw = lds[w].t.rw;
  const bool staged = cl.n_ur >= NROW;
  const uint32_t run = cm_run(n), n_run = run ? (n + run - 1) / run : 0;
  uint32_t ub = 0xFFFFFFFFu;  // first (unit,row) of the staged unit
  uint32_t stride;
  for (uint32_t g = xcd_wave_item(n_run, stride); g < n_run; g += stride) {
    for (uint32_t j = g * run; j < min(n, (g + 1) * run); ++j) {  // uniform per wave
      uint32_t h0 = uni(tr.hit_start[j]), h1 = uni(tr.hit_start[j + 1]);
      if (h1 > tr.hit_cap) h1 = tr.hit_cap;
      if (h0 > h1) h0 = h1;
      const bool act = lane < h1 - h0;
      const uint32_t c = act ? tr.hits[h0 + lane] : 0u;
      const bool in = c < n_cl;
      // the first hits' cluster fields, on their way while their rows are found
      const uint32_t cs = in ? c : 0u;
      int32_t cy = 0, cz = 0;
      uint16_t qt = 0, qm = 0;
      uint8_t fl = 0;
      if (act && n_cl > 0) {
        cy = cl.y[cs];
        cz = cl.z[cs];
        qt = cl.qtot[cs];
        qm = cl.qmax[cs];
        fl = cl.flags[cs];
      }
      const int r0 = uni((int)tr.row[j]);
      const int rt = r0 < NROW ? r0 : NROW - 1;  // a helix at a row past the last is never stepped
      const CmParams q = cm_params(tr.par + (size_t)j * 5, tr.z_anchor[j]);
      uint32_t ur0 = 0;
      if (h1 > h0) {
        const uint32_t c_first = uni(in ? c : 0u);
        if (!staged || ub == 0xFFFFFFFFu || c_first < rw[0] || c_first >= rw[NROW]) {
          const uint32_t f = uni(cm_find_ur_wave(cl.crow, cl.n_ur, c_first));
          if (staged) {
            ub = f / NROW * NROW;  // ub + NROW <= n_ur: n_ur is a multiple of NROW
            for (uint32_t k = lane; k <= NROW; k += 64) rw[k] = cl.crow[ub + k];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
          }
          ur0 = f;
        }
      }
      // rows of the first 64 hits in the staged unit
      uint32_t lo = 0;
      bool plain = false;
      if (staged && h1 > h0) {
        const bool here = in && c >= rw[0] && c < rw[NROW];
        uint32_t hi = NROW;
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (rw[mid] <= c) lo = mid;
          else hi = mid;
        }
        ur0 = ub + uni(lo);  // as found above: the first hit lies in the staged unit
        const int up = (int)__shfl_up(lo, 1, 64);
        const bool rises = lane == 0 ? (int)lo >= r0 : (int)lo > up;
        plain = h1 - h0 <= 64 && __ballot(act && !(here && rises)) == 0;
      }
      const bool keep = h1 <= res_cap;
      uint32_t len = 0;
      bool bad = false;
      if (plain) {  // uniform
        const int r_last = (int)__builtin_amdgcn_readlane((int)lo, (int)(h1 - h0 - 1));
        cm_helix_rows(cm_model(q, b30, rt), xs, ty, tz, r_last);
        const int up = (int)__shfl_up(lo, 1, 64);
        if (act) {
          const int64_t dy = cm_q(cy) - ty[lo], dz = cm_q(cz) - tz[lo];
          const uint64_t stp = lane == 0 ? (uint64_t)((int)lo - r0) : (uint64_t)((int)lo - up - 1);
          len = cm_hit_code(stp, cm_zig(dy), cm_zig(dz), qt, qm, fl, keep, res, res_cap, h0 + lane);
          if (hist_out) {
            atomicAdd(&h[(dy < -64 ? -64 : dy > 63 ? 63 : dy) + 64], 1u);
            atomicAdd(&h[128 + (dz < -64 ? -64 : dz > 63 ? 63 : dz) + 64], 1u);
          }
        }
      } else {
        cm_helix_rows(cm_model(q, b30, rt), xs, ty, tz, NROW - 1);
        bad = cm_track_hits(cl, tr.hits, rw, ub, staged && h1 > h0, n_cl, h0, h1, ur0, r0, rt,
                            [&](bool a, uint32_t hh, uint32_t cc, uint64_t stp, int mr) {
          if (!a) return;
          const int64_t dy = cm_q(cl.y[cc]) - ty[mr], dz = cm_q(cl.z[cc]) - tz[mr];
          len += cm_hit_code(stp, cm_zig(dy), cm_zig(dz), cl.qtot[cc], cl.qmax[cc], cl.flags[cc],
                             keep, res, res_cap, hh);
          if (hist_out) {
            atomicAdd(&h[(dy < -64 ? -64 : dy > 63 ? 63 : dy) + 64], 1u);
            atomicAdd(&h[128 + (dz < -64 ? -64 : dz > 63 ? 63 : dz) + 64], 1u);
          }
        });
      }
      const uint64_t tot = CM_FIXED + (uint64_t)__shfl(wave_incl_scan((uint64_t)len), 63, 64);
      const bool any_bad = __ballot(bad) != 0;
      if (lane == 0) {
        if (any_bad) latch(st, TPC_ERR_INPUT);
        tbits[j] = (uint32_t)(tot < 0xFFFFFFFFull ? tot : 0xFFFFFFFFull);
        tunit[j] = (uint16_t)(ur0 / NROW);
      }
      // the wave's LDS reads are done before the next track overwrites them
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
  if (hist_out)
    for (uint32_t i = threadIdx.x; i < 256; i += blockDim.x)
      if (h[i]) atomicAdd(&hist_out[i], h[i]);
}

// Clusters on no track of one (unit,row), one wave: each lane's cluster code
// length, with the drift position relative to the previous such cluster.
// Calls fn(lane's cluster, its bit offset in the row block, yq zig, z code,
// z order) for every such cluster; returns the block's length.
template <class Fn>
__device__ uint64_t cm_row(const CmClusters& cl, const int32_t* __restrict__ ct, uint32_t ur,
                           uint64_t base, Fn fn) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t n_cl = scan_count(cl.n_dev, cl.cap);
  uint32_t c0 = cl.crow[ur], c1 = cl.crow[ur + 1];
  if (c1 > n_cl) c1 = n_cl;
  if (c0 > c1) c0 = c1;
  // the count first
  uint32_t cnt = 0;
  for (uint32_t b = c0; b < c1; b += 64) {
    const uint32_t c = b + lane;
    const bool un = c < c1 && ct[c] < 0;
    cnt += (uint32_t)__popcll(__ballot(un));
  }
  uint64_t off = base;
  const uint64_t cnt_len = cm_eg_len(cnt, 0);
  fn.count(cnt, off);
  // chunks of CM_CHUNK clusters: a 32-bit field per chunk after the first
  // (its bit offset from the end of the fields), each chunk's first z whole
  const uint32_t n_chunks = (cnt + CM_CHUNK - 1) / CM_CHUNK;
  const uint64_t fields = off + cnt_len;
  off = fields + 32ull * (n_chunks > 1 ? n_chunks - 1 : 0);
  const uint64_t chunk0 = off;
  int64_t zprev = 0;
  uint32_t rank0 = 0;  // clusters on no track in earlier batches
  for (uint32_t b = c0; b < c1; b += 64) {
    const uint32_t c = b + lane;
    const bool un = c < c1 && ct[c] < 0;
    const uint64_t mask = __ballot(un);
    int64_t zq = 0, yq = 0;
    uint32_t len = 0;
    if (un) {
      zq = cm_q(cl.z[c]);
      yq = cm_q(cl.y[c]);
    }
    // the previous cluster on no track: the highest set lane below, else the
    // carry from earlier batches
    const uint64_t below = mask & ((1ull << lane) - 1);
    const uint32_t rank = rank0 + (uint32_t)__popcll(below);
    const int src = below ? 63 - __builtin_clzll(below) : (int)lane;
    const int64_t zp_lane = __shfl(zq, src, 64);
    const bool first = rank % CM_CHUNK == 0;
    const int64_t zp = below ? zp_lane : zprev;
    uint64_t zcode = 0;
    int zk = 12;
    if (un) {
      if (first) {
        zcode = cm_zig(zq);
        zk = 12;
      } else {
        zcode = cm_zig(zq - zp);
        zk = 6;
      }
      len = cm_eg_len(cm_zig(yq), 10) + cm_eg_len(zcode, zk) + cm_cluster_len(cl.qtot[c], cl.qmax[c]);
    }
    // exclusive prefix of the lengths in lane order
    uint64_t incl = wave_incl_scan((uint64_t)len);
    const uint64_t tot = __shfl(incl, 63, 64);
    if (un) {
      const uint64_t at = off + incl - len;
      if (first && rank > 0) fn.field(at - chunk0, fields + 32ull * (rank / CM_CHUNK - 1));
      fn.cluster(c, at, cm_zig(yq), zcode, zk);
    }
    off += tot;
    if (mask) {  // uniform
      const int last = 63 - __builtin_clzll(mask);
      zprev = __shfl(zq, last, 64);
      rank0 += (uint32_t)__popcll(mask);
    }
  }
  return off - base;
}

struct CmRowLen {
  __device__ void count(uint32_t, uint64_t) const {}
  __device__ void field(uint64_t, uint64_t) const {}
  __device__ void cluster(uint32_t, uint64_t, uint64_t, uint64_t, int) const {}
};

// Row passes, one workgroup per (unit,row): the row's clusters on no track are
// listed in LDS in order (eight clusters per thread and scan), so that each is
// coded by a thread of its own with the one before it at hand.  Rows with more
// than CM_ROW_LIST of them go wave by wave (cm_row; same codes).  Lengths and
// writing on the 2 ms slice 0.07 and 0.13 ms, with a wave per row 0.21 and 0.42.
#define CM_ROW_LIST 4096
__device__ __forceinline__ uint32_t cm_row_list(const CmClusters& cl,
                                                const int32_t* __restrict__ ct, uint32_t ur,
                                                uint32_t* list, uint32_t* lds_scan) {
  const uint32_t n_cl = scan_count(cl.n_dev, cl.cap);
  uint32_t c0 = cl.crow[ur], c1 = cl.crow[ur + 1];
  if (c1 > n_cl) c1 = n_cl;
  if (c0 > c1) c0 = c1;
  uint32_t cnt = 0;
  for (uint32_t b = c0; b < c1; b += 256 * 8) {  // uniform
    const uint32_t first = b + threadIdx.x * 8;
    uint32_t m = 0;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
      if (first + k < c1 && ct[first + k] < 0) m |= 1u << k;
    uint32_t tot;
    uint32_t at = cnt + block_excl_scan<uint32_t, 256>((uint32_t)__popc(m), lds_scan, tot);
    for (; m; m &= m - 1, ++at)
      if (at < CM_ROW_LIST) list[at] = first + (uint32_t)__builtin_ctz(m);
    cnt += tot;
  }
  __syncthreads();
  return cnt;
}

// Codes of the i-th listed cluster, given the one before it.
struct CmRowCode {
  uint64_t c[4];
  uint32_t l[4], len;  // y, z, qtot, qmax codes; all with the 2 bits of flags
};
__device__ __forceinline__ CmRowCode cm_row_code(const CmClusters& cl, const uint32_t* list,
                                                 uint32_t i) {
  const uint32_t c = list[i];
  const int64_t zq = cm_q(cl.z[c]);
  CmRowCode r;
  r.c[0] = cm_eg_code(cm_zig(cm_q(cl.y[c])), 10, r.l[0]);
  if (i % CM_CHUNK == 0) r.c[1] = cm_eg_code(cm_zig(zq), 12, r.l[1]);
  else r.c[1] = cm_eg_code(cm_zig(zq - cm_q(cl.z[list[i - 1]])), 6, r.l[1]);
  r.c[2] = cm_eg_code(cl.qtot[c], 6, r.l[2]);
  r.c[3] = cm_eg_code(cl.qmax[c], 5, r.l[3]);
  r.len = r.l[0] + r.l[1] + r.l[2] + r.l[3] + 2;
  return r;
}

__global__ __launch_bounds__(256) void k_cm_row_bits(CmClusters cl, const int32_t* __restrict__ ct,
                                                     uint32_t* __restrict__ rbits,
                                                     const DevStatus* st) {
  __shared__ uint32_t list[CM_ROW_LIST];
  __shared__ uint32_t lds_scan[256 / 64 + 1];
  if (failed(st)) return;
  for (uint32_t ur = blockIdx.x; ur < cl.n_ur; ur += gridDim.x) {
    const uint32_t cnt = cm_row_list(cl, ct, ur, list, lds_scan);
    uint64_t len;
    if (cnt <= CM_ROW_LIST) {  // uniform
      uint32_t mine = 0, tot;
      for (uint32_t i = threadIdx.x; i < cnt; i += 256) mine += cm_row_code(cl, list, i).len;
      block_excl_scan<uint32_t, 256>(mine, lds_scan, tot);
      const uint32_t n_chunks = (cnt + CM_CHUNK - 1) / CM_CHUNK;
      len = (uint64_t)cm_eg_len(cnt, 0) + 32ull * (n_chunks > 1 ? n_chunks - 1 : 0) + tot;
    } else {
      len = threadIdx.x < 64 ? cm_row(cl, ct, ur, 0, CmRowLen{}) : 0;
    }
    if (threadIdx.x == 0) rbits[ur] = (uint32_t)(len < 0xFFFFFFFFull ? len : 0xFFFFFFFFull);
    __syncthreads();  // the list is read before the next row's
  }
}

// Directory entries from the scans: track j at stream[CM_HDR + j], row block
// ur at stream[CM_HDR + n_tracks + 1 + ur] (after the tracks' total).
struct CmEmitTrack {
  uint32_t* s;
  uint32_t cap;
  __device__ void operator()(uint32_t j, unsigned long long pre, unsigned long long) const {
    if (CM_HDR + (uint64_t)j < cap) s[CM_HDR + j] = (uint32_t)pre;
  }
};
struct CmEmitRow {
  uint32_t* s;
  uint32_t cap;
  const uint32_t* n_tracks_dev;
  uint32_t tr_cap;
  const unsigned long long* track_total;
  __device__ void operator()(uint32_t ur, unsigned long long pre, unsigned long long) const {
    const uint64_t i = CM_HDR + (uint64_t)scan_count(n_tracks_dev, tr_cap) + 1 + ur;
    if (i < cap) s[i] = (uint32_t)(pre + *track_total);
  }
};
struct CmEmitOff {
  uint32_t* out;
  __device__ void operator()(uint32_t i, unsigned long long pre, unsigned long long) const {
    out[i] = (uint32_t)pre;
  }
};
struct CmGetU32 {
  const uint32_t* a;
  __device__ unsigned long long operator()(uint32_t i) const { return a[i]; }
};

// Header, the closing directory entries, the size check.  tot[0] = tracks'
// bits, tot[1] = rows' bits; info[0] = words needed (0 after an error).
__global__ void k_cm_finish(uint32_t* __restrict__ s, uint32_t cap, uint32_t n_units,
                            const uint32_t* n_tracks_dev, uint32_t tr_cap,
                            const uint32_t* hit_start, const uint32_t* n_cl_dev, uint32_t cl_cap,
                            const unsigned long long* tot, uint32_t* n_words_out,
                            uint32_t* info, DevStatus* st) {
  info[0] = 0;
  if (failed(st)) return;
  const uint32_t n_tr = scan_count(n_tracks_dev, tr_cap);
  const uint32_t n_ur = n_units * NROW;
  const unsigned long long bits = tot[0] + tot[1];
  const uint64_t dir = CM_HDR + (uint64_t)n_tr + 1 + n_ur + 1;
  const uint64_t need = dir + (bits + 31) / 32;
  *n_words_out = (uint32_t)(need < 0xFFFFFFFFull ? need : 0xFFFFFFFFull);
  if (bits > 0xFFFFFFFFull || need > cap) {
    latch(st, TPC_ERR_CAPACITY, (uint32_t)(need < 0xFFFFFFFFull ? need : 0xFFFFFFFFull));
    return;
  }
  s[0] = CM_MAGIC;
  s[1] = CM_VERSION;
  s[2] = n_units;
  s[3] = n_tr;
  s[4] = scan_count(n_cl_dev, cl_cap);
  s[5] = n_tr ? hit_start[n_tr] : 0;
  s[6] = (uint32_t)bits;
  s[7] = 0;
  s[CM_HDR + n_tr] = (uint32_t)tot[0];
  s[dir - 1] = (uint32_t)bits;
  info[0] = (uint32_t)need;
  info[1] = (uint32_t)dir;
}

// clear the payload words [dir, need)
__global__ void k_cm_clear(uint32_t* __restrict__ s, const uint32_t* info, const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t need = info[0], dir = info[1];
  for (uint32_t i = dir + blockIdx.x * blockDim.x + threadIdx.x; i < need;
       i += gridDim.x * blockDim.x)
    s[i] = 0;
}

// One track's record coded anew, hit by hit, by a wave (a track whose codes were
// not all kept).
__device__ void cm_track_anew(const CmClusters& cl, const CmTracks& tr, int64_t b30,
                              const int32_t* xfx, uint32_t* __restrict__ s, uint32_t* payload,
                              uint64_t pw, uint32_t n_cl, uint32_t j, CmTrackLds& lds) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t h0 = uni(tr.hit_start[j]), h1 = uni(tr.hit_start[j + 1]);
  if (h1 > tr.hit_cap) h1 = tr.hit_cap;
  if (h0 > h1) h0 = h1;
  const uint64_t start = uni(s[CM_HDR + j]);
  const int r0 = uni((int)tr.row[j]);
  const CmParams q = cm_params(tr.par + (size_t)j * 5, tr.z_anchor[j]);
  uint32_t ur0 = 0;
  if (h1 > h0) {
    const uint32_t c = tr.hits[h0];
    ur0 = cm_find_ur_wave(cl.crow, cl.n_ur, c < n_cl ? c : 0);
  }
  const int rt = r0 < NROW ? r0 : NROW - 1;
  int64_t* ty = lds.t.ty;
  int64_t* tz = lds.t.tz;
  cm_helix_rows(cm_model(q, b30, rt), xfx, ty, tz, NROW - 1);
  if (lane == 0) {
    CmWriter wr;
    wr.init(payload, pw, start);
    wr.put(h1 - h0, 8);
    wr.put(ur0 / NROW, 16);
    wr.put((uint32_t)r0, 8);
    wr.put((uint32_t)(int32_t)q.Y, 32);
    wr.put((uint32_t)(int32_t)q.Z, 32);
    wr.put((uint32_t)(int32_t)q.S, 32);
    wr.put((uint32_t)(int32_t)q.T, 32);
    wr.put((uint32_t)(int32_t)q.K, 32);
    wr.flush();
  }
  uint64_t off = start + CM_FIXED;
  cm_track_hits(cl, tr.hits, nullptr, 0, false, n_cl, h0, h1, ur0, r0, rt,
                [&](bool a, uint32_t hh, uint32_t cc, uint64_t stp, int mr) {
    uint64_t zy = 0, zz = 0, hl = 0;
    uint16_t qt = 0, qm = 0;
    uint8_t fl = 0;
    if (a) {
      zy = cm_zig(cm_q(cl.y[cc]) - ty[mr]);
      zz = cm_zig(cm_q(cl.z[cc]) - tz[mr]);
      qt = cl.qtot[cc];
      qm = cl.qmax[cc];
      fl = cl.flags[cc];
      hl = cm_eg_len(stp, 0) + cm_eg_len(zy, 2) + cm_eg_len(zz, 2) + cm_cluster_len(qt, qm);
    }
    const uint64_t incl = wave_incl_scan(hl);
    if (a) {
      CmWriter wr;
      wr.init(payload, pw, off + incl - hl);
      wr.eg(stp, 0);
      wr.eg(zy, 2);
      wr.eg(zz, 2);
      cm_cluster_put(wr, qt, qm, fl);
      wr.flush();
    }
    off += __shfl(incl, 63, 64);
  });
  // the wave's LDS reads are done before the table is overwritten
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The track records at their directory offsets.  A wave takes up to CM_RUN
// consecutive tracks: their records are one run of bits and their hits one run of
// kept codes, so lane k makes the fixed fields of track k, every lane places a
// hit's code (at the codes before it and the fixed fields up to its track's), all
// in LDS, and the run is stored in whole words.  No cluster, row or helix is
// read again.  Bound by latency: a few dependent loads per run.  On the 2 ms slice
// (3.7e5 tracks, 6e7 bytes of records) 0.15 ms; 0.40 with a wave per track, 1.01
// with every hit's row searched, its charges gathered and its codes written bit
// group by bit group.
__global__ __launch_bounds__(256) void k_cm_track_write(CmClusters cl, CmTracks tr, int64_t b30,
                                                        const DevParams* __restrict__ P,
                                                        const uint16_t* __restrict__ tunit,
                                                        uint32_t* __restrict__ s,
                                                        const uint32_t* info,
                                                        const uint64_t* __restrict__ res,
                                                        uint32_t res_cap, DevStatus* st) {
  __shared__ CmTrackLds lds[4];
  if (failed(st) || info[0] == 0) return;
  const uint32_t n = scan_count(tr.n_dev, tr.cap);
  const uint32_t n_cl = scan_count(cl.n_dev, cl.cap);
  uint32_t* payload = s + info[1];
  const uint64_t pw = info[0] - info[1];
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t* rec = lds[w].rec;
  const uint32_t run = cm_run(n), n_run = run ? (n + run - 1) / run : 0;
  const uint32_t hit_end = min(tr.hit_cap, res_cap);
  uint32_t stride;
  for (uint32_t g = xcd_wave_item(n_run, stride); g < n_run; g += stride) {
    const uint32_t j0 = g * run, m_all = min(run, n - j0);
    // lane k: first hit, record start and fixed fields of track j0 + k
    uint32_t hs = 0xFFFFFFFFu, dir = 0;
    if (lane <= m_all) {
      hs = tr.hit_start[j0 + lane];
      dir = s[CM_HDR + j0 + lane];
    }
    uint32_t f[6] = {0, 0, 0, 0, 0, 0};
    if (lane < m_all) {
      const CmParams q = cm_params(tr.par + (size_t)(j0 + lane) * 5, tr.z_anchor[j0 + lane]);
      f[0] = ((uint32_t)tunit[j0 + lane] << 8) | ((uint32_t)tr.row[j0 + lane] << 24);
      f[1] = (uint32_t)(int32_t)q.Y;
      f[2] = (uint32_t)(int32_t)q.Z;
      f[3] = (uint32_t)(int32_t)q.S;
      f[4] = (uint32_t)(int32_t)q.T;
      f[5] = (uint32_t)(int32_t)q.K;
    }
    const uint32_t hs_next = (uint32_t)__shfl((int)hs, (int)min(lane + 1, 63u));
    f[0] |= (hs_next - hs) & 255u;
    // lanes whose track has its hits in order and kept
    const uint64_t good = __ballot(lane < m_all && hs <= hs_next && hs_next <= hit_end);
    for (uint32_t t = 0; t < m_all;) {  // uniform
      const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)dir, (int)t);
      const uint32_t h0 = (uint32_t)__builtin_amdgcn_readlane((int)hs, (int)t);
      const uint32_t sh = d0 & 31;
      // tracks t, t + 1, ... whose records fit the LDS words together
      const uint32_t dir_next = (uint32_t)__shfl((int)dir, (int)min(lane + 1, 63u));
      const uint64_t ok = __ballot((good >> lane & 1) && lane >= t && dir_next >= d0 &&
                                   dir_next - d0 <= 32 * (CM_REC_WORDS - 1));
      const uint64_t stop = ~(ok >> t);
      uint32_t m = stop ? (uint32_t)__builtin_ctzll(stop) : 64u;
      bool kept = m > 0;
      if (kept) {
        const uint32_t h1 = (uint32_t)__builtin_amdgcn_readlane((int)hs, (int)(t + m));
        const uint32_t d1 = (uint32_t)__builtin_amdgcn_readlane((int)dir, (int)(t + m));
        const uint32_t words = (sh + (d1 - d0) + 31) >> 5;
        for (uint32_t i = lane; i < words + 3; i += 64) rec[i] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane >= t && lane < t + m) {
#pragma unroll
          for (uint32_t i = 0; i < 6; ++i) cm_lds_or(rec, sh + (dir - d0) + 32 * i, f[i]);
        }
        bool too_long = false;
        uint32_t at0 = sh;
        for (uint32_t base = h0; base < h1; base += 64) {  // uniform
          const uint32_t hh = base + lane;
          const bool act = hh < h1;
          const uint64_t v = act ? res[hh] : 0;
          const uint32_t len = (uint32_t)(v >> CM_KEEP);
          too_long = too_long || len == CM_LONG;
          const uint32_t incl = wave_incl_scan(len);
          uint32_t fixed = CM_FIXED;  // fixed fields of the tracks from t to the hit's
#pragma unroll
          for (uint32_t k = 1; k < CM_RUN; ++k)
            if (k < m && hh >= (uint32_t)__builtin_amdgcn_readlane((int)hs, (int)(t + k)))
              fixed += CM_FIXED;
          const uint32_t at = at0 + fixed + incl - len;
          if (act && at + len <= 32 * words) {  // inside the run whatever the lengths say
            cm_lds_or(rec, at, v & ((1ull << CM_KEEP) - 1));
            if (len > CM_KEEP && len <= 2 * CM_KEEP)
              cm_lds_or(rec, at + CM_KEEP, res[(size_t)res_cap + hh]);
          }
          at0 += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        kept = __ballot(too_long) == 0;
        if (kept) cm_store_words(rec, payload, pw, d0, d1, lane, 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      } else {
        m = 1;
      }
      if (!kept)
        for (uint32_t k = 0; k < m; ++k)
          cm_track_anew(cl, tr, b30, P->xfx, s, payload, pw, n_cl, j0 + t + k, lds[w]);
      t += m;
    }
  }
}

struct CmRowPut {
  const CmClusters* cl;
  uint32_t* payload;
  uint64_t pw;  // payload words
  __device__ void count(uint32_t cnt, uint64_t off) const {
    if ((threadIdx.x & 63) == 0) {
      CmWriter w;
      w.init(payload, pw, off);
      w.eg(cnt, 0);
      w.flush();
    }
  }
  // a chunk's 32-bit offset field (its value < 2^32: payload offsets are)
  __device__ void field(uint64_t v, uint64_t off) const {
    CmWriter w;
    w.init(payload, pw, off);
    w.put((uint32_t)v, 32);
    w.flush();
  }
  __device__ void cluster(uint32_t c, uint64_t off, uint64_t yz, uint64_t zcode, int zk) const {
    CmWriter w;
    w.init(payload, pw, off);
    w.eg(yz, 10);
    w.eg(zcode, zk);
    cm_cluster_put(w, cl->qtot[c], cl->qmax[c], cl->flags[c]);
    w.flush();
  }
};

// The row blocks, one workgroup per (unit,row): 256 listed clusters at a time,
// their codes placed by a scan of their lengths, put together in LDS.
#define CM_ROW_WORDS 1280  // 256 codes of at most 139 bits, and the shift of the first
__global__ __launch_bounds__(256) void k_cm_row_write(CmClusters cl, const int32_t* __restrict__ ct,
                                                      uint32_t* __restrict__ s,
                                                      const uint32_t* n_tracks_dev, uint32_t tr_cap,
                                                      const uint32_t* info, const DevStatus* st) {
  __shared__ uint32_t list[CM_ROW_LIST];
  __shared__ uint32_t words[CM_ROW_WORDS + 4];
  __shared__ uint32_t lds_scan[256 / 64 + 1];
  if (failed(st) || info[0] == 0) return;
  const uint32_t n_tr = scan_count(n_tracks_dev, tr_cap);
  uint32_t* payload = s + info[1];
  const uint64_t pw = info[0] - info[1];
  for (uint32_t ur = blockIdx.x; ur < cl.n_ur; ur += gridDim.x) {
    const uint64_t base = s[CM_HDR + n_tr + 1 + ur];
    const uint32_t cnt = cm_row_list(cl, ct, ur, list, lds_scan);
    if (cnt > CM_ROW_LIST) {  // uniform
      if (threadIdx.x < 64) cm_row(cl, ct, ur, base, CmRowPut{&cl, payload, pw});
      __syncthreads();
      continue;
    }
    const uint32_t n_chunks = (cnt + CM_CHUNK - 1) / CM_CHUNK;
    const CmRowPut put{&cl, payload, pw};
    if (threadIdx.x < 64) put.count(cnt, base);
    const uint64_t fields = base + cm_eg_len(cnt, 0);
    const uint64_t chunk0 = fields + 32ull * (n_chunks > 1 ? n_chunks - 1 : 0);
    uint64_t off = chunk0;
    for (uint32_t i0 = 0; i0 < cnt; i0 += 256) {  // uniform
      for (uint32_t k = threadIdx.x; k < CM_ROW_WORDS + 4; k += 256) words[k] = 0;
      const uint32_t i = i0 + threadIdx.x;
      CmRowCode r;
      r.len = 0;
      if (i < cnt) r = cm_row_code(cl, list, i);
      uint32_t tot;
      const uint32_t pre = block_excl_scan<uint32_t, 256>(r.len, lds_scan, tot);  // has barriers
      if (i < cnt) {
        uint32_t at = (uint32_t)(off & 31) + pre;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          cm_lds_or(words, at, r.c[k]);
          at += r.l[k];
        }
        cm_lds_or(words, at, cl.flags[list[i]] & 3u);
        if (i % CM_CHUNK == 0 && i > 0)
          put.field(off + pre - chunk0, fields + 32ull * (i / CM_CHUNK - 1));
      }
      __syncthreads();
      cm_store_words(words, payload, pw, off, off + tot, threadIdx.x, 256);
      off += tot;
      __syncthreads();
    }
    __syncthreads();  // the list is read before the next row's
  }
}

// ------------------------------------------------------------------ decoder
struct CmDecOut {
  uint32_t capacity;
  uint16_t* unit;
  uint8_t* row;
  int32_t *y, *z;
  uint16_t *qtot, *qmax;
  uint8_t* flags;
  int32_t* track;
};

// Header checks; info = {n_units, n_tracks, n_clusters, payload bits, dir
// words, records (tracks + rows), ok}.
__global__ void k_cm_dec_header(const uint32_t* __restrict__ s, uint32_t n_words, uint32_t max_units,
                                uint32_t max_tracks, uint32_t out_cap, uint32_t* n_out,
                                uint32_t* info, DevStatus* st) {
  info[6] = 0;
  if (failed(st)) return;
  if (n_words < CM_HDR || s[0] != CM_MAGIC || s[1] != CM_VERSION || s[7] != 0) {
    latch(st, TPC_ERR_INPUT);
    return;
  }
  const uint32_t nu = s[2], nt = s[3], nc = s[4], bits = s[6];
  const uint64_t dir = CM_HDR + (uint64_t)nt + 1 + (uint64_t)nu * NROW + 1;
  if (nu > max_units || nt > max_tracks || dir > n_words || bits > (n_words - dir) * 32ull ||
      s[CM_HDR + nt + 1 + (uint64_t)nu * NROW] != bits || s[CM_HDR] != 0 ||
      s[CM_HDR + nt] != s[CM_HDR + nt + 1]) {  // the rows begin where the tracks end
    latch(st, TPC_ERR_INPUT);
    return;
  }
  *n_out = nc;
  if (nc > out_cap) {
    latch(st, TPC_ERR_CAPACITY, nc);
    return;
  }
  info[0] = nu;
  info[1] = nt;
  info[2] = nc;
  info[3] = bits;
  info[4] = (uint32_t)dir;
  info[5] = nt + nu * NROW;
  info[6] = 1;
}

// Clusters per record: a track's fixed-width hit count, a row's count code.
__global__ void k_cm_dec_counts(const uint32_t* __restrict__ s, const uint32_t* info,
                                uint32_t* __restrict__ cnt, DevStatus* st) {
  if (failed(st) || !info[6]) return;
  const uint32_t nt = info[1], nrec = info[5];
  CmReader r{s + info[4], 0, info[3], false, 0};
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nrec; i += gridDim.x * blockDim.x) {
    r.bad = false;
    r.seek(s[CM_HDR + (i < nt ? i : i + 1)]);
    cnt[i] = (uint32_t)(i < nt ? r.get(8) : r.eg(0));
    if (r.bad || cnt[i] > 0xFFFFFFu) {
      cnt[i] = 0;
      latch(st, TPC_ERR_INPUT);
    }
  }
}

// Track record i decoded from r at output offset k; false if it is malformed
// or does not end at `end`.
template <typename Reader>
__device__ bool cm_decode_record(Reader& r, uint32_t i, uint32_t nu, uint32_t nt, uint32_t nc,
                                 uint32_t k, uint64_t end, int64_t b30, const int32_t* xfx,
                                 const CmDecOut& o) {
  bool bad = false;
  if (i < nt) {
    const uint32_t nh = (uint32_t)r.get(8);
    const uint32_t unit = (uint32_t)r.get(16);
    const int r0 = (int)r.get(8);
    CmParams q;
    q.Y = (int32_t)r.get(32);
    q.Z = (int32_t)r.get(32);
    q.S = (int32_t)r.get(32);
    q.T = (int32_t)r.get(32);
    q.K = (int32_t)r.get(32);
    if (unit >= nu || r0 >= NROW) bad = true;
    CmModel m = cm_model(q, b30, r0);
    int prev = r0;
    for (uint32_t h = 0; h < nh && !bad && !r.bad; ++h, ++k) {
      const uint64_t stp = r.eg(0);
      const int rr = prev + (int)(stp > NROW ? NROW : stp) + (h > 0 ? 1 : 0);
      if (rr >= NROW || k >= nc || k >= o.capacity) {
        bad = true;
        break;
      }
      prev = rr;
      while (m.row < rr) cm_step(m, xfx);
      const int64_t yq = cm_q(m.Y) + cm_unzig(r.eg(2));
      const int64_t zq = cm_q(m.Z) + cm_unzig(r.eg(2));
      o.unit[k] = (uint16_t)unit;
      o.row[k] = (uint8_t)rr;
      o.y[k] = (int32_t)(yq << CM_QSHIFT);
      o.z[k] = (int32_t)(zq << CM_QSHIFT);
      o.qtot[k] = (uint16_t)r.eg(6);
      o.qmax[k] = (uint16_t)r.eg(5);
      o.flags[k] = (uint8_t)r.get(2);
      o.track[k] = (int32_t)i;
    }
  }
  return !(bad || r.bad || r.pos != end);
}

// One chunk of row record ur (k-th, `count` clusters) from r, written at
// output index k0 on; false if malformed or not ending at `end`.
template <typename Reader>
__device__ bool cm_decode_chunk(Reader& r, uint32_t ur, uint32_t count, uint32_t k0, uint32_t nc,
                                uint64_t end, const CmDecOut& o) {
  int64_t zprev = 0;
  uint32_t k = k0;
  for (uint32_t c = 0; c < count && !r.bad; ++c, ++k) {
    if (k >= nc || k >= o.capacity) return false;
    const int64_t yq = cm_unzig(r.eg(10));
    const int64_t zq = c == 0 ? cm_unzig(r.eg(12)) : zprev + cm_unzig(r.eg(6));
    zprev = zq;
    o.unit[k] = (uint16_t)(ur / NROW);
    o.row[k] = (uint8_t)(ur % NROW);
    o.y[k] = (int32_t)(yq << CM_QSHIFT);
    o.z[k] = (int32_t)(zq << CM_QSHIFT);
    o.qtot[k] = (uint16_t)r.eg(6);
    o.qmax[k] = (uint16_t)r.eg(5);
    o.flags[k] = (uint8_t)r.get(2);
    o.track[k] = -1;
  }
  return !(r.bad || r.pos != end);
}

// Row record ur at bits [b0, b1): the count and the chunk fields, then lane
// l decodes chunks l, l + 64, ...; every chunk must end where the next one
// (or the record) ends.  Reader: the row's bits (staged in LDS, or global).
template <typename Reader>
__device__ void cm_decode_row(Reader r, uint32_t ur, uint32_t k_row, uint32_t nc, uint64_t b0,
                              uint64_t b1, const CmDecOut& o, DevStatus* st) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t n = r.eg(0);
  if (r.bad || n > 0xFFFFFFu) {
    if (lane == 0) latch(st, TPC_ERR_INPUT);
    return;
  }
  const uint32_t m = ((uint32_t)n + CM_CHUNK - 1) / CM_CHUNK;
  const uint64_t fields = r.pos;
  const uint64_t chunk0 = fields + 32ull * (m > 1 ? m - 1 : 0);
  if (m == 0) {
    if (lane == 0 && r.pos != b1) latch(st, TPC_ERR_INPUT);
    return;
  }
  if (chunk0 > b1) {
    if (lane == 0) latch(st, TPC_ERR_INPUT);
    return;
  }
  for (uint32_t k = lane; k < m; k += 64) {
    uint64_t cs = chunk0, ce = b1;
    if (k > 0) {
      r.seek(fields + 32ull * (k - 1));
      cs = chunk0 + r.get(32);
    }
    if (k + 1 < m) {
      r.seek(fields + 32ull * k);
      ce = chunk0 + r.get(32);
    }
    bool ok = !r.bad && cs <= ce && ce <= b1;
    if (ok) {
      const uint64_t end_save = r.end;
      r.end = ce;  // reads stop at the chunk's end
      r.seek(cs);
      const uint32_t count = min((uint32_t)n - CM_CHUNK * k, (uint32_t)CM_CHUNK);
      ok = cm_decode_chunk(r, ur, count, k_row + CM_CHUNK * k, nc, ce, o);
      r.end = end_save;
      r.bad = false;
    }
    if (!ok) latch(st, TPC_ERR_INPUT);
  }
}

// Row records: one wave per record, its bits first copied into the wave's
// part of LDS when they fit, one lane per chunk.
__global__ __launch_bounds__(256) void k_cm_dec_rows(const uint32_t* __restrict__ s,
                                                     const uint32_t* info,
                                                     const uint32_t* __restrict__ off,
                                                     const unsigned long long* total,
                                                     CmDecOut o, DevStatus* st) {
  __shared__ uint32_t stage[4][CM_STAGE_WORDS];
  if (failed(st) || !info[6]) return;
  const uint32_t nt = info[1], nc = info[2], nrec = info[5];
  const uint64_t bits = info[3];
  const uint32_t* pay = s + info[4];
  if (blockIdx.x == 0 && threadIdx.x == 0 && *total != nc) latch(st, TPC_ERR_INPUT);
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (uint32_t i = nt + blockIdx.x * 4 + w; i < nrec; i += gridDim.x * 4) {
    uint64_t b0 = s[CM_HDR + i + 1], b1 = s[CM_HDR + i + 2];
    if (b0 > bits) b0 = bits;
    if (b1 > bits) b1 = bits;
    if (b1 < b0) b1 = b0;
    const uint64_t w0 = b0 >> 5, w1 = (b1 + 31) >> 5;
    const bool staged = w1 - w0 <= CM_STAGE_WORDS;
    if (staged) {
      for (uint64_t k = lane; k < w1 - w0; k += 64) stage[w][k] = pay[w0 + k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (staged) {
      cm_decode_row(CmReaderT<lds_u32*>((lds_u32*)stage[w], b0, b1, false, w0), i - nt, off[i], nc,
                    b0, b1, o, st);
    } else {
      cm_decode_row(CmReader(pay, b0, b1, false, 0), i - nt, off[i], nc, b0, b1, o, st);
    }
    // the wave's LDS reads are done before the next record overwrites it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Track records: 64 per wave, one per lane; the wave's records' bits are
// first copied into its part of LDS when they fit (a dependent chain of
// global reads is what bounds a sequential decoder), else read from the
// payload.
__global__ __launch_bounds__(256) void k_cm_dec_tracks(const uint32_t* __restrict__ s,
                                                       const uint32_t* info,
                                                       const uint32_t* __restrict__ off,
                                                       int64_t b30, const DevParams* __restrict__ P,
                                                       CmDecOut o, DevStatus* st) {
  __shared__ uint32_t stage[4][CM_STAGE_WORDS];
  __shared__ int32_t xs[NROW];  // row radii: the helix steps read them per lane
  if (failed_wg(st) || !info[6]) return;
  for (uint32_t i = threadIdx.x; i < NROW; i += blockDim.x) xs[i] = P->xfx[i];
  __syncthreads();
  const uint32_t nu = info[0], nt = info[1], nc = info[2];
  const uint64_t bits = info[3];
  const uint32_t* pay = s + info[4];
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t n_groups = (nt + 63) / 64;
  for (uint32_t g = blockIdx.x * 4 + w; g < n_groups; g += gridDim.x * 4) {
    const uint32_t i0 = g * 64;
    const uint32_t i1 = min(i0 + 64, nt);
    // the wave's bit range: from the first record's start to the last one's end
    uint64_t b0 = s[CM_HDR + i0];
    uint64_t b1 = s[CM_HDR + i1];
    if (b0 > bits) b0 = bits;
    if (b1 > bits) b1 = bits;
    if (b1 < b0) b1 = b0;
    const uint64_t w0 = b0 >> 5, w1 = (b1 + 31) >> 5;
    const bool staged = w1 - w0 <= CM_STAGE_WORDS;
    if (staged) {
      for (uint64_t k = lane; k < w1 - w0; k += 64) stage[w][k] = pay[w0 + k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t i = i0 + lane;
    if (i < i1) {
      const uint64_t start = s[CM_HDR + i];
      const uint64_t end = s[CM_HDR + i + 1];
      // from LDS when the record lies in the staged range (reads stop at its
      // end), else (a malformed directory) from the payload
      const bool in_lds = staged && start >= b0 && end <= b1;
      bool ok;
      if (in_lds) {
        CmReaderT<lds_u32*> r((lds_u32*)stage[w], start, b1, false, w0);
        ok = cm_decode_record(r, i, nu, nt, nc, off[i], end, b30, xs, o);
      } else {
        CmReader r(pay, start, bits, false, 0);
        ok = cm_decode_record(r, i, nu, nt, nc, off[i], end, b30, xs, o);
      }
      if (!ok) latch(st, TPC_ERR_INPUT);
    }
    // the wave's LDS reads are done before the next group overwrites it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------- decoder in two steps (the default)
// Parsing is serial per record (or chunk of a row), the rest is not: the first
// step only parses, one lane per track or chunk, and stores one 16-byte raw
// record per cluster at its output index; the second turns the raw records into
// the output arrays in contiguous runs, the tracks' helices evaluated by one wave
// per track at all its rows (as the encoder does).  A one-step decoder steps each
// helix row by row in its lane and stores eight scattered values per cluster:
// tracks 0.89 and rows 0.30 ms on a chunk of 37 collisions (6.4e6 clusters), where
// the two steps take 0.15 and 0.10 (parsing: the serial chain of the longest
// records) and 0.13 and 0.01 ms (outputs).
struct CmRaw {
  uint32_t y, z;  // tracks: zigzag residuals; rows: quantised positions (low 32 bits)
  uint32_t q;     // qtot | qmax << 16
  uint32_t at;    // row | flags << 8 | unit << 16
};

// Bit reader that keeps nothing but a position: a code is cut out of a 32-bit
// window of two adjacent words, several codes out of one window where they fit.
// Reads past the last word see that word again; a malformed record then ends at
// the wrong position, which the caller checks.
template <typename P>
struct CmWindow {
  P w;
  uint32_t last;  // index of the last word
  uint32_t pos;   // bit position relative to w[0]
  bool bad;
  __device__ uint32_t window() const {
    const uint32_t i = min(pos >> 5, last);
    return __builtin_amdgcn_alignbit(w[min(i + 1, last)], w[i], pos & 31);
  }
  __device__ uint32_t read(uint32_t n) {  // n <= 32
    const uint32_t v = window();
    pos += n;
    return n >= 32 ? v : v & ((1u << n) - 1u);
  }
  // order-k code from a window of its own (low 32 bits of the value)
  __device__ uint32_t eg(int k) {
    const uint32_t v = window();
    if (v == 0) {  // no one bit among the next 32: malformed
      bad = true;
      return 0;
    }
    const uint32_t n = (uint32_t)__builtin_ctz(v), len = 2 * n + 1 + k;
    if (len <= 32) {
      pos += len;
      return cut(v, n, k);
    }
    pos += n + 1;
    const uint32_t low = read(n);
    const uint64_t q = (1ull << n) | low;
    return (uint32_t)((q - 1) << k) | read(k);
  }
  __device__ static uint32_t cut(uint32_t v, uint32_t n, int k) {
    const uint32_t low = __builtin_amdgcn_ubfe(v, n + 1, n);
    return ((((1u << n) | low) - 1u) << k) | __builtin_amdgcn_ubfe(v, 2 * n + 1, k);
  }
  // the next code of a window v of which `used` bits are taken; false (and
  // nothing taken) if it does not end inside
  __device__ static bool next(uint32_t& v, uint32_t& used, int k, uint32_t& out) {
    const uint32_t n = (uint32_t)__builtin_ctz(v | 0x80000000u), len = 2 * n + 1 + k;
    if (used + len > 32 || v == 0) return false;
    out = cut(v, n, k);
    v = len < 32 ? v >> len : 0u;
    used += len;
    return true;
  }
  // three codes, out of one window where they fit
  __device__ void eg3(int k0, int k1, int k2, uint32_t& a, uint32_t& b, uint32_t& c) {
    uint32_t v = window(), used = 0;
    if (next(v, used, k0, a) && next(v, used, k1, b) && next(v, used, k2, c)) {
      pos += used;
    } else {
      a = eg(k0);
      b = eg(k1);
      c = eg(k2);
    }
  }
  // the charges and flags of a cluster
  __device__ void charges(uint32_t& qt, uint32_t& qm, uint32_t& fl) {
    uint32_t v = window(), used = 0;
    if (next(v, used, 6, qt) && next(v, used, 5, qm) && used <= 30) {
      fl = v & 3u;
      pos += used + 2;
    } else {
      qt = eg(6);
      qm = eg(5);
      fl = read(2);
    }
  }
};
__device__ __forceinline__ uint32_t cm_unzig32(uint32_t u) { return (u >> 1) ^ (0u - (u & 1u)); }

// A track record parsed by its lane: raw records from output index k on, the
// fixed fields (row and unit, Y, Z, S, T, K) into fields[6].  False if it is
// malformed or does not end at `end` (relative to the reader's first word).
template <typename R>
__device__ __forceinline__ bool cm_parse_track(R& r, uint32_t nu, uint32_t nc, uint32_t cap,
                                               uint32_t k, uint32_t end, CmRaw* __restrict__ raw,
                                               uint32_t* __restrict__ fields) {
  const uint32_t nh = r.read(8), unit = r.read(16), r0 = r.read(8);
  fields[0] = unit | (r0 << 16);
  for (int i = 1; i < 6; ++i) fields[i] = r.read(32);
  if (unit >= nu || r0 >= NROW) return false;
  uint32_t row = r0;
  for (uint32_t h = 0; h < nh; ++h, ++k) {
    uint32_t stp, zy, zz, qt, qm, fl;
    r.eg3(0, 2, 2, stp, zy, zz);
    r.charges(qt, qm, fl);
    row += min(stp, (uint32_t)NROW) + (h > 0 ? 1u : 0u);
    if (r.bad || row >= NROW || k >= nc || k >= cap) return false;
    raw[k] = CmRaw{zy, zz, (qt & 0xFFFFu) | (qm << 16), row | (fl << 8) | (unit << 16)};
  }
  return r.pos == end;
}

// Track records, 64 per wave and workgroup, one per lane, the group's bits staged
// in LDS (64 records of the 2 ms slice average 3,050 words).
#define CM_PARSE_TRACK_WORDS 4096
#define CM_PARSE_ROW_WORDS 2048  // a row's clusters on no track: 1,900 at 20,500 time bins
__global__ __launch_bounds__(64) void k_cm_parse_tracks(const uint32_t* __restrict__ s,
                                                         const uint32_t* info,
                                                         const uint32_t* __restrict__ off,
                                                         uint32_t cap, CmRaw* __restrict__ raw,
                                                         uint32_t* __restrict__ fields,
                                                         DevStatus* st) {
  __shared__ uint32_t stage[CM_PARSE_TRACK_WORDS];
  if (failed(st) || !info[6]) return;
  const uint32_t nu = info[0], nt = info[1], nc = info[2];
  const uint64_t bits = info[3];
  const uint32_t* pay = s + info[4];
  const uint32_t lane = threadIdx.x;
  const uint32_t n_groups = (nt + 63) / 64;
  for (uint32_t g = blockIdx.x; g < n_groups; g += gridDim.x) {
    const uint32_t i0 = g * 64;
    const uint32_t i1 = min(i0 + 64, nt);
    // the wave's bit range: from the first record's start to the last one's end
    uint64_t b0 = s[CM_HDR + i0];
    uint64_t b1 = s[CM_HDR + i1];
    if (b0 > bits) b0 = bits;
    if (b1 > bits) b1 = bits;
    if (b1 < b0) b1 = b0;
    const uint64_t w0 = b0 >> 5, w1 = (b1 + 31) >> 5;
    const bool staged = w1 - w0 <= CM_PARSE_TRACK_WORDS;
    if (staged) {
      for (uint64_t k = lane; k < w1 - w0; k += 64) stage[k] = pay[w0 + k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t i = i0 + lane;
    if (i < i1) {
      const uint64_t start = s[CM_HDR + i], end = s[CM_HDR + i + 1];
      bool ok = start <= end && end <= bits && bits > 0;
      if (ok) {
        // from LDS when the record lies in the staged range, else (a long
        // group, or a malformed directory) from the payload
        uint32_t* f = fields + (size_t)i * 6;
        if (staged && start >= b0 && end <= b1 && w1 > w0) {
          CmWindow<lds_u32*> r{(lds_u32*)stage, (uint32_t)(w1 - w0 - 1), (uint32_t)(start - w0 * 32),
                               false};
          ok = cm_parse_track(r, nu, nc, cap, off[i], (uint32_t)(end - w0 * 32), raw, f);
        } else {
          const uint64_t p0 = start >> 5, p1 = (bits + 31) >> 5;
          CmWindow<const uint32_t*> r{pay + p0, (uint32_t)(p1 > p0 ? p1 - p0 - 1 : 0),
                                      (uint32_t)(start & 31), false};
          ok = p1 > p0 && cm_parse_track(r, nu, nc, cap, off[i], (uint32_t)(end - p0 * 32), raw, f);
        }
      }
      if (!ok) latch(st, TPC_ERR_INPUT);
    }
    // the wave's LDS reads are done before the next group overwrites it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// One row record by a wave, lane l its chunks l, l + 64, ...; r at the record's
// start, b1 its end, both relative to the reader's first word.  False if
// malformed; every chunk must end where the next one (or the record) ends.
template <typename R>
__device__ __forceinline__ bool cm_parse_row(R r, uint32_t ur, uint32_t k_row, uint32_t nc,
                                             uint32_t cap, uint32_t b1, CmRaw* __restrict__ raw) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t n = r.eg(0);
  if (r.bad || n > 0xFFFFFFu) return false;
  const uint32_t m = (n + CM_CHUNK - 1) / CM_CHUNK;
  if (m == 0) return r.pos == b1;
  const uint32_t fields = r.pos;
  if (fields + 32ull * (m - 1) > b1) return false;
  const uint32_t chunk0 = fields + 32u * (m - 1);
  const uint32_t at = (ur % NROW) | ((ur / NROW) << 16);
  bool ok = true;
  for (uint32_t k = lane; k < m; k += 64) {
    uint32_t cs = chunk0, ce = b1;
    if (k > 0) {
      r.pos = fields + 32u * (k - 1);
      cs = chunk0 + r.read(32);
    }
    if (k + 1 < m) {
      r.pos = fields + 32u * k;
      ce = chunk0 + r.read(32);
    }
    if (cs < chunk0 || cs > ce || ce > b1) {
      ok = false;
      break;
    }
    r.pos = cs;
    const uint32_t count = min(n - CM_CHUNK * k, (uint32_t)CM_CHUNK);
    uint32_t o = k_row + CM_CHUNK * k, z = 0;
    for (uint32_t c = 0; c < count; ++c, ++o) {
      uint32_t qt, qm, fl;
      const uint32_t y = cm_unzig32(r.eg(10));
      z += cm_unzig32(r.eg(c == 0 ? 12 : 6));
      r.charges(qt, qm, fl);
      if (r.bad || o >= nc || o >= cap) {
        ok = false;
        break;
      }
      raw[o] = CmRaw{y, z, (qt & 0xFFFFu) | (qm << 16), at | (fl << 8)};
    }
    if (r.pos != ce) ok = false;
    if (!ok) break;
  }
  return ok;
}

__global__ __launch_bounds__(256) void k_cm_parse_rows(const uint32_t* __restrict__ s,
                                                       const uint32_t* info,
                                                       const uint32_t* __restrict__ off,
                                                       const unsigned long long* total,
                                                       uint32_t cap, CmRaw* __restrict__ raw,
                                                       DevStatus* st) {
  __shared__ uint32_t stage[4][CM_PARSE_ROW_WORDS];
  if (failed(st) || !info[6]) return;
  const uint32_t nt = info[1], nc = info[2], nrec = info[5];
  const uint64_t bits = info[3];
  const uint32_t* pay = s + info[4];
  if (blockIdx.x == 0 && threadIdx.x == 0 && *total != nc) latch(st, TPC_ERR_INPUT);
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (uint32_t i = nt + blockIdx.x * 4 + w; i < nrec; i += gridDim.x * 4) {
    uint64_t b0 = s[CM_HDR + i + 1], b1 = s[CM_HDR + i + 2];
    if (b0 > bits) b0 = bits;
    if (b1 > bits) b1 = bits;
    const uint64_t w0 = b0 >> 5, w1 = (b1 + 31) >> 5;
    const bool sane = b1 > b0;  // a record has at least its count's bit
    const bool staged = sane && w1 - w0 <= CM_PARSE_ROW_WORDS;
    if (staged) {
      for (uint64_t k = lane; k < w1 - w0; k += 64) stage[w][k] = pay[w0 + k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    bool ok = sane;
    if (staged) {
      ok = cm_parse_row(CmWindow<lds_u32*>{(lds_u32*)stage[w], (uint32_t)(w1 - w0 - 1),
                                           (uint32_t)(b0 & 31), false},
                        i - nt, off[i], nc, cap, (uint32_t)(b1 - w0 * 32), raw);
    } else if (sane) {
      ok = cm_parse_row(CmWindow<const uint32_t*>{pay + w0, (uint32_t)(w1 - w0 - 1),
                                                  (uint32_t)(b0 & 31), false},
                        i - nt, off[i], nc, cap, (uint32_t)(b1 - w0 * 32), raw);
    }
    if (!ok) latch(st, TPC_ERR_INPUT);
    // the wave's LDS reads are done before the next record overwrites it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

__device__ __forceinline__ void cm_raw_out(const CmDecOut& o, uint32_t k, const CmRaw& v,
                                           uint32_t yq, uint32_t zq, int32_t track) {
  o.unit[k] = (uint16_t)(v.at >> 16);
  o.row[k] = (uint8_t)v.at;
  o.y[k] = (int32_t)(yq << CM_QSHIFT);
  o.z[k] = (int32_t)(zq << CM_QSHIFT);
  o.qtot[k] = (uint16_t)v.q;
  o.qmax[k] = (uint16_t)(v.q >> 16);
  o.flags[k] = (uint8_t)(v.at >> 8) & 3u;
  o.track[k] = track;
}

// The outputs of the tracks' hits, one wave per track.
__global__ __launch_bounds__(256) void k_cm_dec_model(const uint32_t* info,
                                                      const uint32_t* __restrict__ off,
                                                      const uint32_t* __restrict__ cnt,
                                                      const CmRaw* __restrict__ raw,
                                                      const uint32_t* __restrict__ fields,
                                                      int64_t b30, const DevParams* __restrict__ P,
                                                      CmDecOut o, const DevStatus* st) {
  __shared__ int32_t xs[NROW];
  __shared__ int64_t tab[4][2][NROW];
  if (failed(st) || !info[6]) return;
  for (uint32_t i = threadIdx.x; i < NROW; i += blockDim.x) xs[i] = P->xfx[i];
  __syncthreads();
  const uint32_t nt = info[1], w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int64_t* ty = tab[w][0];
  int64_t* tz = tab[w][1];
  uint32_t stride;
  for (uint32_t i = xcd_wave_item(nt, stride); i < nt; i += stride) {  // uniform per wave
    const uint32_t k0 = uni(off[i]), nh = uni(cnt[i]);
    if (nh == 0) continue;
    CmRaw v{0, 0, 0, 0};
    if (lane < nh) v = raw[k0 + lane];
    const uint32_t* f = fields + (size_t)i * 6;
    const CmParams q{(int32_t)f[1], (int32_t)f[2], (int32_t)f[3], (int32_t)f[4], (int32_t)f[5]};
    // the last row bounds the helix's table (rows ascend)
    const int r_last = (int)uni(raw[k0 + nh - 1].at & 255u);
    cm_helix_rows(cm_model(q, b30, (int)uni(f[0] >> 16)), xs, ty, tz, r_last);
    for (uint32_t h = lane; h < nh; h += 64) {
      if (h >= 64) v = raw[k0 + h];
      const uint32_t r = v.at & 255u;
      cm_raw_out(o, k0 + h, v, (uint32_t)ty[r] + cm_unzig32(v.y), (uint32_t)tz[r] + cm_unzig32(v.z),
                 (int32_t)i);
    }
    // the wave's LDS reads are done before the next track overwrites them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// The outputs of the clusters on no track: those after the tracks' hits.
__global__ __launch_bounds__(256) void k_cm_dec_rest(const uint32_t* info,
                                                     const uint32_t* __restrict__ off,
                                                     const CmRaw* __restrict__ raw, CmDecOut o,
                                                     const DevStatus* st) {
  if (failed(st) || !info[6]) return;
  const uint32_t nt = info[1], nc = info[2];
  const uint32_t k0 = info[5] > nt ? off[nt] : nc;
  for (uint32_t k = k0 + blockIdx.x * blockDim.x + threadIdx.x; k < nc;
       k += gridDim.x * blockDim.x) {
    const CmRaw v = raw[k];
    cm_raw_out(o, k, v, v.y, v.z, -1);
  }
}
