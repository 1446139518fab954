// Segment merging (sector boundaries, looper legs) and the continuous-readout
// T0 / z fit of the merged tracks.
//
// A segment's two ends (innermost and outermost hit) carry their global
// position, drift z and the tangent of the segment's outward fit there.  Ends
// are binned by (frame, side, 30.5 cm squares of the bending plane, 12 cm of
// drift); one lane per end finds the ends close to it in the 3 x 3 x 7 cells
// around it (every joinable pair has ends within 35 cm in drift and 30 cm in the
// bending plane, so the cells hold all candidates); the pairs go through the
// joining rule, and join segments by a lock-free union-find that always hangs the larger root under
// the smaller, so the final root of a component is its smallest segment
// whatever the order of the unions.  The members of each component are then
// sorted by (root, index), and 8 or 16 lanes per component fit all its hits in
// FP64, added up in ascending segment order: the algebraic circle fit about the
// centroid, the line of drift z against the unwrapped azimuth, the beam-axis
// crossing and T0.  The arithmetic follows the joining rule and the fit as
// stated in include/tpc.h.
#pragma once

#include "common.hpp"

#define MG_GAP 30.0
#define MG_DZMAX 35.0
#define MG_PERP 0.5
#define MG_DZ 1.0
#define MG_DZ_ARC 0.02
#define MG_SIN 0.1
#define MG_DC_REL 0.2
#define MG_DC_ABS 1e-3
#define MG_C_LINE 1e-4
#define MG_TIE 1e-9
// drift cells (cm), MG_ZR of which are above MG_DZMAX (fewer candidates outside the
// gate in finer ones: 37 collisions merged in 808, 792, 772 and 779 us with MG_ZR
// 1, 2, 3 and 4)
#define MG_ZR 3
#define MG_ZBIN (36.0 / MG_ZR)
#define MG_XYBIN 30.5  // bending-plane cell (cm), above MG_GAP with its tie band
#define MG_XY0 260.0   // the cells cover [-MG_XY0, MG_XY0) in x and y (outer radius ~247 cm)
#define MG_NXY 18      // cells per axis: ceil(2 MG_XY0 / MG_XYBIN)
#define MG_FIT 12     // doubles per merged-track fit record

struct MgSegs {  // per segment (track), device SoA
  double *C, *tgl;
  double* e;     // [n * 10]: per end X, Y, z, tx, ty
};

__device__ __forceinline__ uint32_t mg_ur_of(const uint32_t* crow, uint32_t n_ur, uint32_t c) {
  uint32_t lo = 0, hi = n_ur;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (crow[mid] <= c) lo = mid;
    else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ double mg_wrap(double a) {
  while (a > M_PI) a -= 2 * M_PI;
  while (a <= -M_PI) a += 2 * M_PI;
  return a;
}

__device__ __forceinline__ bool mg_cut(double v, double cut, bool& tie) {
  if (fabs(v - cut) <= MG_TIE * cut) tie = true;
  return v <= cut;
}

// Bending-plane cell index of a coordinate (clamped: a pair within MG_GAP
// still falls in neighbouring cells).
__device__ __forceinline__ uint32_t mg_xy_bin(double v) {
  double b = floor((v + MG_XY0) / MG_XYBIN);
  if (!(b >= 0.0)) b = 0.0;
  if (b > MG_NXY - 1) b = MG_NXY - 1;
  return (uint32_t)b;
}

// Per segment: frame-side, curvature, dip and the two ends; per end its cell.
__global__ void k_mg_segments(const uint32_t* __restrict__ crow, uint32_t n_ur,
                              const int32_t* __restrict__ y_fx, const int32_t* __restrict__ z_fx,
                              const uint32_t* n_cl_dev, uint32_t cl_cap,
                              const float* __restrict__ par, const uint8_t* __restrict__ trow,
                              const uint32_t* __restrict__ hit_start,
                              const uint32_t* __restrict__ hits, uint32_t hit_cap,
                              const uint32_t* n_trk_dev, uint32_t trk_cap,
                              const double* __restrict__ cs18, double bz_b, uint32_t nzb,
                              MgSegs S, uint32_t* __restrict__ cell_of_end,
                              uint32_t* __restrict__ cell_cnt, const DevParams* __restrict__ P,
                              const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t n = scan_count(n_trk_dev, trk_cap);
  const uint32_t n_cl = scan_count(n_cl_dev, cl_cap);
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
    uint32_t h0 = hit_start[j], h1 = hit_start[j + 1];
    if (h1 > hit_cap) h1 = hit_cap;
    bool ok = h1 > h0;
    uint32_t c0 = 0, c1 = 0;
    if (ok) {
      c0 = hits[h0];
      c1 = hits[h1 - 1];
      ok = c0 < n_cl && c1 < n_cl;
    }
    if (!ok) {
      cell_of_end[2 * j] = cell_of_end[2 * j + 1] = 0xFFFFFFFFu;
      continue;
    }
    const uint32_t ur0 = mg_ur_of(crow, n_ur, c0), ur1 = mg_ur_of(crow, n_ur, c1);
    const uint32_t unit = ur0 / NROW, sector = unit % 36;
    const uint32_t fs = (unit / 36) * 2 + sector / 18;
    const double C = -bz_b * (double)par[(size_t)j * 5 + 4];
    S.C[j] = C;
    S.tgl[j] = (double)par[(size_t)j * 5 + 3];
    const double ca = cs18[2 * (sector % 18)], sa = cs18[2 * (sector % 18) + 1];
    const double xp = P->xd[trow[j] < NROW ? trow[j] : 0];
    const double sp = (double)par[(size_t)j * 5 + 2];
    const int rows[2] = {(int)(ur0 % NROW), (int)(ur1 % NROW)};
    const uint32_t cs[2] = {c0, c1};
    for (int e = 0; e < 2; ++e) {
      const double x = P->xd[rows[e]], y = y_fx[cs[e]] / 65536.0;
      double snp = sp + C * (x - xp);
      if (snp > 0.999999) snp = 0.999999;
      if (snp < -0.999999) snp = -0.999999;
      const double cp = sqrt(1.0 - snp * snp);
      double* E = S.e + (size_t)j * 10 + 5 * e;
      E[0] = x * ca - y * sa;
      E[1] = x * sa + y * ca;
      E[2] = z_fx[cs[e]] / 65536.0;
      E[3] = cp * ca - snp * sa;
      E[4] = cp * sa + snp * ca;
      int64_t zb = (int64_t)floor((E[2] + 1.0) / MG_ZBIN);
      if (zb < 0) zb = 0;
      if (zb >= (int64_t)nzb) zb = nzb - 1;
      const uint32_t cell = ((fs * MG_NXY + mg_xy_bin(E[1])) * MG_NXY + mg_xy_bin(E[0])) * nzb +
                            (uint32_t)zb;
      cell_of_end[2 * j + e] = cell;
      atomicAdd(&cell_cnt[cell], 1u);
    }
  }
}

__device__ __forceinline__ uint32_t mg_find(const uint32_t* parent, uint32_t x) {
  uint32_t p = __atomic_load_n(&parent[x], __ATOMIC_RELAXED);
  while (p != x) {
    x = p;
    p = __atomic_load_n(&parent[x], __ATOMIC_RELAXED);
  }
  return x;
}

__device__ __forceinline__ void mg_union(uint32_t* parent, uint32_t a, uint32_t b) {
  while (true) {
    uint32_t ra = mg_find(parent, a), rb = mg_find(parent, b);
    if (ra == rb) return;
    if (ra < rb) {
      const uint32_t t = ra;
      ra = rb;
      rb = t;
    }
    // hang the larger root under the smaller; retry if it stopped being a root
    if (atomicCAS(&parent[ra], ra, rb) == ra) return;
    a = ra;
    b = rb;
  }
}

// End b seen from end a of a segment with curvature C and dip tgl.
__device__ __forceinline__ bool mg_follows(double C, double tgl, const double* a, const double* b,
                                           bool& tie) {
  const double dx = b[0] - a[0], dy = b[1] - a[1];
  double perp, arc, tx, ty;
  if (fabs(C) >= MG_C_LINE) {
    const double r = 1.0 / C;
    const double cx = a[0] - r * a[4], cy = a[1] + r * a[3];
    const double ux = a[0] - cx, uy = a[1] - cy, vx = b[0] - cx, vy = b[1] - cy;
    const double vr = sqrt(vx * vx + vy * vy);
    perp = fabs(vr - fabs(r));
    const double dpsi = atan2(ux * vy - uy * vx, ux * vx + uy * vy);
    arc = dpsi / C;
    // the tangent where b projects onto the circle (radius vector turned a
    // quarter turn in the sense of the motion)
    tx = C > 0 ? -vy / vr : vy / vr;
    ty = C > 0 ? vx / vr : -vx / vr;
  } else {
    perp = fabs(a[3] * dy - a[4] * dx);
    arc = a[3] * dx + a[4] * dy;
    tx = a[3];
    ty = a[4];
  }
  bool ok = mg_cut(perp, MG_PERP, tie);
  ok &= mg_cut(fabs(arc), MG_GAP, tie);
  ok &= mg_cut(fabs(b[2] - a[2] - tgl * arc), MG_DZ + MG_DZ_ARC * fabs(arc), tie);
  ok &= mg_cut(fabs(tx * b[4] - ty * b[3]), MG_SIN, tie);
  return ok;
}

// What the pair search needs of an end, in cell order: position (drift z in
// 2^-16 cm, exact) with 2 * segment + end, and the tangent, curvature and dip.
struct MgPos {
  float x, y;
  int32_t z;
  uint32_t id;
};
struct MgDir {
  float tx, ty, C, tgl;
};
// The ends into their cells (in any order within a cell: the unions do not
// depend on it).
__global__ void k_mg_fill_cells(const uint32_t* __restrict__ cell_of_end, const uint32_t* n_trk_dev,
                                uint32_t trk_cap, uint32_t* __restrict__ cursor, MgSegs S,
                                MgPos* __restrict__ pos, MgDir* __restrict__ dir,
                                const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t n_ends = 2 * scan_count(n_trk_dev, trk_cap);  // only this call's ends
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n_ends;
       e += gridDim.x * blockDim.x) {
    const uint32_t c = cell_of_end[e], j = e >> 1;
    if (c == 0xFFFFFFFFu) continue;
    const double* E = S.e + (size_t)j * 10 + 5 * (e & 1);
    const uint32_t k = atomicAdd(&cursor[c], 1u);
    pos[k] = MgPos{(float)E[0], (float)E[1], (int32_t)(E[2] * 65536.0), e};
    dir[k] = MgDir{(float)E[3], (float)E[4], (float)S.C[j], (float)S.tgl[j]};
  }
}

// A cut in FP32: clearly missed, or within a part in a thousand (a NaN counts
// as within).  The FP32 errors stay below a third of that: coordinates are good to
// 8e-6 cm and steps to d = 2.3e-5, so distances off a circle to 1e-4 cm where the
// cut's margin is 5e-4.  At a distance q |r| from the centre the arc is good to d / q
// and the tangent's turn to d |C| / q: pairs near a centre go on to the FP64 test, and
// with |C| + |tan lambda| / 8 < q the errors of the drift are below 2.5e-4 (the
// margin is 1e-3) and those of the sine below 3e-5 (1e-4).
__device__ __forceinline__ void mg_cut32(float v, float cut, bool& missed, bool& close) {
  missed |= v > cut * 1.001f;
  close |= !(v < cut * 0.999f || v > cut * 1.001f);
}

// mg_follows in FP32: with s and p the components of the step across and along
// the tangent and q = |centre to b| / |r|, the distance off the circle is
// |2 s + C d^2| / (1 + q), the arc 2 atan(u) / C with u = C p / (q + 1 + C s) and
// the tangent there (tx - C dy, ty + C dx) / q, none of which cancels for stiff
// tracks.  atan(u) / u is an interpolation in u^2 at Chebyshev points of [0, 1]
// (relative error 1e-6).
__device__ __forceinline__ void mg_follows32(const MgDir& a, const MgDir& b, float dx, float dy,
                                             float dz, bool& missed, bool& close) {
  const float aC = fabsf(a.C);
  const float C = aC >= (float)MG_C_LINE ? a.C : 0.0f;
  const float s = a.ty * dx - a.tx * dy, p = a.tx * dx + a.ty * dy;
  const float c1 = 1.0f + C * s, c2 = C * p;
  const float q = __builtin_amdgcn_sqrtf(c1 * c1 + c2 * c2);
  const float perp = fabsf(2.0f * s + C * (s * s + p * p)) * __builtin_amdgcn_rcpf(1.0f + q);
  const float iqc = __builtin_amdgcn_rcpf(q + c1), u = c2 * iqc, t = u * u;
  float k = 0.00764835393f;
  k = k * t - 0.0363604315f;
  k = k * t + 0.0831264555f;
  k = k * t - 0.134478644f;
  k = k * t + 0.198720396f;
  k = k * t - 0.333256781f;
  k = k * t + 0.999999225f;
  const float arc = 2.0f * p * iqc * k, len = fabsf(arc);
  // either form, towards the centre or around the circle, beyond the error bounds
  // (one comparison for both limits; a NaN in either is close)
  close |= fabsf(aC - (float)MG_C_LINE) < 1e-8f || !(c1 > 0.1f) ||
           !(aC + 0.125f * fabsf(a.tgl) < fminf(q, 1.0f));
  mg_cut32(perp, (float)MG_PERP, missed, close);
  mg_cut32(len, (float)MG_GAP, missed, close);
  mg_cut32(fabsf(dz - a.tgl * arc), (float)MG_DZ + (float)MG_DZ_ARC * len, missed, close);
  mg_cut32(fabsf((a.tx - C * dy) * b.ty - (a.ty + C * dx) * b.tx), (float)MG_SIN * q, missed,
           close);
}

// Whether a pair has to go through the FP64 test: not if a cut is clearly missed
// and none is so close that FP64 could call it a near tie.
__device__ __forceinline__ bool mg_maybe(const MgPos& pa, const MgPos& pb, const MgDir& a,
                                         const MgDir& b) {
  const float dx = pb.x - pa.x, dy = pb.y - pa.y, dz = (float)(pb.z - pa.z) * (1.0f / 65536.0f);
  bool missed = false, close = false;
  mg_cut32(__builtin_amdgcn_sqrtf(dx * dx + dy * dy), (float)MG_GAP, missed, close);
  const float ca = fabsf(a.C), cb = fabsf(b.C);
  mg_cut32(fabsf(ca - cb), (float)MG_DC_REL * fmaxf(ca, cb) + (float)MG_DC_ABS, missed, close);
  mg_follows32(a, b, dx, dy, dz, missed, close);
  mg_follows32(b, a, -dx, -dy, -dz, missed, close);
  return close || !missed;
}

// The joining test of ends e and f in FP64 (the same either way round): the
// gates and cuts, then the union; near ties flag both segments.
__device__ __forceinline__ void mg_pair_check(const MgSegs& S, uint32_t e, uint32_t f,
                                              uint32_t* parent, uint8_t* near_tie) {
  const uint32_t A = e >> 1, B = f >> 1;
  const double* a = S.e + (size_t)A * 10 + 5 * (e & 1);
  const double* b = S.e + (size_t)B * 10 + 5 * (f & 1);
  const double ax = a[0], ay = a[1], bx = b[0], by = b[1];
  const double d2 = (ax - bx) * (ax - bx) + (ay - by) * (ay - by);
  // beyond the near-tie band of the gap cut nothing can pass or tie (squared
  // distances: the band's margin of 2e-9 dwarfs the rounding)
  constexpr double g = MG_GAP * (1 + 2 * MG_TIE);
  if (!(fabs(a[2] - b[2]) <= MG_DZMAX) || !(d2 <= g * g)) return;
  const double dxy = sqrt(d2);
  const double ca = fabs(S.C[A]), cb = fabs(S.C[B]), cm = ca > cb ? ca : cb;
  bool tie = false;
  bool ok = mg_cut(dxy, MG_GAP, tie);
  if (ok) {
    ok = mg_cut(fabs(ca - cb), MG_DC_REL * cm + MG_DC_ABS, tie);
#pragma unroll 1
    for (int way = 0; way < 2; ++way) {  // b seen from a, a seen from b
      const uint32_t J = way ? B : A;
      ok &= mg_follows(S.C[J], S.tgl[J], way ? b : a, way ? a : b, tie);
    }
  }
  if (tie) {
    near_tie[A] = 1;
    near_tie[B] = 1;
  }
  if (ok) mg_union(parent, A, B);
}

// One lane per end, ends taken in cell order (the lanes of a wave mostly
// share their cells and so scan the same neighbour cells in step).  Of the
// 3 x 3 x 7 cells around an end half are scanned, so that a pair is met once:
// the rest of its own cell and the MG_ZR cells above in drift, and four neighbouring
// columns of 2 MG_ZR + 1 drift cells, each a run of consecutive ends.  A wave takes
// 64 ends and one of the five runs at a time (a grid of a few waves per SIMD
// strides over these), four candidates loaded together and the next four on
// their way.  Pairs that pass the gates on drift z and distance go to a queue of
// the wave in LDS, and every 64 of them are tested in FP32 by the 64 lanes
// together; the few that FP32 cannot rule out go to a second queue for the FP64
// test (two helix extrapolations with an arc tangent each), 64 at a time again.
// On a chunk of 37 collisions (139,000 segments) 316 us; 1364 with one wave per 64
// ends for all 27 cells, every gated pair tested in FP64, a candidate at a time.
#define MG_SCAN 4
#define MG_RUNS 5
#define MG_QCAP (64 + 64 * MG_SCAN)
#define MG_PAIR_BLOCKS 1024  // four per CU: the registers hold four waves per SIMD
__global__ __launch_bounds__(256, 4) void k_mg_pairs(
    MgSegs S, uint32_t nzb, const uint32_t* total_dev, const uint32_t* __restrict__ cell_off,
    const uint32_t* __restrict__ cell_of_end, const MgPos* __restrict__ pos,
    const MgDir* __restrict__ dir, uint32_t* __restrict__ parent, uint8_t* __restrict__ near_tie,
    const DevStatus* st) {
  __shared__ uint32_t qa[4][MG_QCAP], qb[4][MG_QCAP];  // gated pairs: places in cell order
  __shared__ uint32_t ra[4][128], rb[4][128];          // pairs for FP64: ends
  if (failed(st)) return;
  const uint32_t total = *total_dev;
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint64_t below = (1ull << lane) - 1ull;
  auto in_order = [] {  // a wave's LDS writes before its reads, and the reverse
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  uint32_t qn = 0, rn = 0;  // queued pairs (the same in every lane)
  const uint32_t items = (total + 63) / 64 * MG_RUNS;
  // one step past the items empties the queues
  const uint32_t nw = gridDim.x * 4;
  for (uint32_t item = blockIdx.x * 4 + w;; item += nw) {  // uniform per wave
    const bool last = item >= items;
    const uint32_t run = item % MG_RUNS, t = item / MG_RUNS * 64 + lane;
    MgPos me{0, 0, 0, 0};
    uint32_t k0 = 0, len = 0;
    if (!last && t < total) {
      me = pos[t];
      const uint32_t cell = cell_of_end[me.id];
      const uint32_t zb = cell % nzb, xy = cell / nzb, ix = xy % MG_NXY, iy = xy / MG_NXY % MG_NXY;
      const uint32_t up = min((uint32_t)MG_ZR, nzb - 1 - zb), dn = min((uint32_t)MG_ZR, zb);
      if (run == 0) {
        k0 = t + 1;
        len = cell_off[cell + up + 1] - k0;
      } else {
        // runs 1 to 4: (dx, dy) = (1, 0), (-1, 1), (0, 1), (1, 1)
        const int x2 = (int)ix + (run == 1 ? 1 : (int)run - 3), y2 = (int)iy + (run > 1);
        if (x2 >= 0 && x2 < MG_NXY && y2 < MG_NXY) {
          const uint32_t cb = cell + (uint32_t)((run > 1 ? MG_NXY : 0) + x2 - (int)ix) * nzb;
          k0 = cell_off[cb - dn];
          len = cell_off[cb + up + 1] - k0;
        }
      }
    }
    const uint32_t maxlen = (uint32_t)wave_max_i32((int32_t)len);
    const uint32_t full = last ? 1 : 64;  // pairs that are tested together
    // a round's candidates (an end that exists, in every lane)
    auto load = [&](uint32_t it, MgPos (&c)[MG_SCAN]) {
#pragma unroll
      for (uint32_t i = 0; i < MG_SCAN; ++i) c[i] = pos[min(k0 + it + i, total - 1)];
    };
    MgPos cur[MG_SCAN], nxt[MG_SCAN];
    if (maxlen) load(0, cur);
    uint32_t it = 0;
    do {
      if (maxlen) {
        load(it + MG_SCAN, nxt);
#pragma unroll
        for (uint32_t i = 0; i < MG_SCAN; ++i) {
          const float ex = me.x - cur[i].x, ey = me.y - cur[i].y;
          const int32_t ez = me.z - cur[i].z;
          // drift exactly; distance with a margin above the FP32 positions' errors
          constexpr float g = (float)MG_GAP + 1e-3f;
          constexpr int32_t gz = (int32_t)(MG_DZMAX * 65536);
          const bool pass = it + i < len && ez <= gz && ez >= -gz && ex * ex + ey * ey <= g * g &&
                            (cur[i].id ^ me.id) > 1;  // not the segment's own ends
          const uint64_t m = __ballot(pass);
          const uint32_t at = qn + (uint32_t)__popcll(m & below);
          if (pass) {
            qa[w][at] = t;
            qb[w][at] = k0 + it + i;
          }
          qn += (uint32_t)__popcll(m);
          cur[i] = nxt[i];
        }
      }
      while (qn >= full) {  // uniform: the newest pairs, one per lane
        in_order();
        const uint32_t m = min(qn, 64u);
        bool go = false;
        uint32_t e = 0, f = 0;
        if (lane < m) {
          const uint32_t a = qa[w][qn - m + lane], b = qb[w][qn - m + lane];
          const MgPos pa = pos[a], pb = pos[b];
          go = mg_maybe(pa, pb, dir[a], dir[b]);
          e = pa.id;
          f = pb.id;
        }
        qn -= m;
        const uint64_t mask = __ballot(go);
        const uint32_t at = rn + (uint32_t)__popcll(mask & below);
        if (go) {
          ra[w][at] = e;
          rb[w][at] = f;
        }
        rn += (uint32_t)__popcll(mask);
        in_order();
        if (rn >= 64) {  // uniform
          mg_pair_check(S, ra[w][rn - 64 + lane], rb[w][rn - 64 + lane], parent, near_tie);
          rn -= 64;
          in_order();
        }
      }
      it += MG_SCAN;
    } while (it < maxlen);
    if (last) break;
  }
  if (lane < rn) mg_pair_check(S, ra[w][lane], rb[w][lane], parent, near_tie);
}

// Global position and drift of every hit of every track (the fit reads the
// positions three times): one thread per hit, its cluster's (unit,row) found by a
// binary search of the row starts (one lane per track walking its hits took 0.68
// ms on a 2 ms Pb-Pb slice, the longest tracks setting the pace; per hit: 0.28 ms,
// bound by the gathers of the clusters: the search's first steps in LDS took no
// more than 6% off).
__global__ void k_mg_hits(const uint32_t* __restrict__ crow, uint32_t n_ur,
                          const int32_t* __restrict__ y_fx, const int32_t* __restrict__ z_fx,
                          const uint32_t* n_cl_dev, uint32_t cl_cap,
                          const uint32_t* __restrict__ hit_start,
                          const uint32_t* __restrict__ hits, uint32_t hit_cap,
                          const uint32_t* n_trk_dev, uint32_t trk_cap,
                          const double* __restrict__ cs18, double* __restrict__ hxy,
                          int32_t* __restrict__ hz, const DevParams* __restrict__ P,
                          const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t n = scan_count(n_trk_dev, trk_cap);
  const uint32_t n_cl = scan_count(n_cl_dev, cl_cap);
  uint32_t nh = n ? hit_start[n] : 0;  // the tracks' hits are [0, hit_start[n])
  if (nh > hit_cap) nh = hit_cap;
  for (uint32_t h = blockIdx.x * blockDim.x + threadIdx.x; h < nh; h += gridDim.x * blockDim.x) {
    const uint32_t c = hits[h] < n_cl ? hits[h] : 0;
    const uint32_t ur = mg_ur_of(crow, n_ur, c);
    const uint32_t s18 = (ur / NROW) % 36 % 18;
    const double ca = cs18[2 * s18], sa = cs18[2 * s18 + 1];
    const double x = P->xd[ur % NROW], y = y_fx[c] / 65536.0;
    hxy[2 * (size_t)h] = x * ca - y * sa;
    hxy[2 * (size_t)h + 1] = x * sa + y * ca;
    hz[h] = z_fx[c];
  }
}

// Everything that the call starts from: no ends in the cells, every segment a
// root, fit records (n_fit doubles) and the count of merged tracks zero.
__global__ void k_mg_init(uint32_t* __restrict__ cell_cnt, uint32_t n_cells,
                          double* __restrict__ fit, uint32_t n_fit, uint32_t* __restrict__ parent,
                          uint8_t* __restrict__ near_tie, uint32_t* __restrict__ idx, uint32_t cap,
                          uint32_t* __restrict__ n_merged, const DevStatus* st) {
  const uint32_t i0 = blockIdx.x * blockDim.x + threadIdx.x, di = gridDim.x * blockDim.x;
  for (uint32_t i = i0; i < n_fit; i += di) fit[i] = 0.0;
  if (failed(st)) return;
  for (uint32_t i = i0; i < n_cells; i += di) cell_cnt[i] = 0;
  for (uint32_t j = i0; j < cap; j += di) {
    parent[j] = j;
    near_tie[j] = 0;
    idx[j] = j;
  }
  if (i0 == 0) *n_merged = 0;
}

// label = the root; the roots are counted, one atomic per workgroup.
__global__ __launch_bounds__(256) void k_mg_labels(const uint32_t* __restrict__ parent,
                                                   const uint32_t* n_trk_dev, uint32_t trk_cap,
                                                   int32_t* __restrict__ label,
                                                   uint32_t* __restrict__ key,
                                                   uint32_t* __restrict__ n_merged,
                                                   const DevStatus* st) {
  __shared__ uint32_t roots;
  if (failed(st)) return;
  if (threadIdx.x == 0) roots = 0;
  __syncthreads();
  const uint32_t n = scan_count(n_trk_dev, trk_cap);
  uint32_t mine = 0;
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
    const uint32_t r = mg_find(parent, j);
    label[j] = (int32_t)r;
    key[j] = r;
    mine += r == j;
  }
  if (mine) atomicAdd(&roots, mine);
  __syncthreads();
  if (threadIdx.x == 0 && roots) atomicAdd(n_merged, roots);
}

// Eight lanes' values of one array, in the lanes' order.
__device__ __forceinline__ void mg_row(const double* lds, double (&x)[8]) {
  const double2* v = reinterpret_cast<const double2*>(lds);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double2 t = v[i];
    x[2 * i] = t.x;
    x[2 * i + 1] = t.y;
  }
}

// G lanes per component (the first of its run in the sorted members): the FP64
// helix fit of all its hits, members in ascending index.  The lanes take a
// member's hits G at a time and compute their terms (the arc tangent of the
// azimuth above all) together; the sums and the unwrapped azimuth are still
// added hit by hit in their order, each lane adding up one sum from the terms
// that the lanes leave in LDS, so the results are those of one lane.  (A term of
// +0 stands for the lanes past a member's last hit: it changes no sum, none of
// which can be -0.)  lds: [64 / G][6][G + 2] doubles (padded: 16-byte reads
// spread over the banks).
template <int G>
__device__ __forceinline__ void mg_fit_rows(const uint32_t* __restrict__ skey,
                                            const uint32_t* __restrict__ sidx, uint32_t n,
                                            const uint32_t* __restrict__ hit_start,
                                            uint32_t hit_cap, const double* __restrict__ hxy,
                                            const int32_t* __restrict__ hz,
                                            double* __restrict__ fit, double* rows) {
  const uint32_t g = threadIdx.x / G, q = threadIdx.x % G;
  double(*lds)[G + 2] = reinterpret_cast<double(*)[G + 2]>(rows) + 6 * g;
  lds[5][q] = 1.0;
  auto in_order = [] {  // a wave's LDS writes before its reads, and the reverse
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto of_lane = [](double v, int k) { return __shfl(v, k, G); };
  const double2* xy = reinterpret_cast<const double2*>(hxy);  // by k_mg_hits
  // the arrays whose products are this lane's sum in the second pass, of
  // u, v, uu, vv, uv: uu, vv, uv, uuu, vvv, uvv, vuu
  const uint32_t fa = 0x4432010u >> 4 * (q & 7) & 7, fb = 0x0110110u >> 4 * (q & 7) & 7;
  for (uint32_t i = blockIdx.x * (64 / G) + g; i < n; i += gridDim.x * (64 / G)) {
    const uint32_t root = skey[i];
    if (i > 0 && skey[i - 1] == root) continue;
    uint32_t end = i + 1;
    while (end < n && skey[end] == root) ++end;
    double* f = fit + (size_t)root * MG_FIT;
    double out[MG_FIT] = {};
    auto store = [&] {
#pragma unroll
      for (int k = 0; k < MG_FIT; ++k)
        if (q == k % G) f[k] = out[k];
    };
    // step(p, z, cnt): this lane's hit of the next cnt, loaded a step ahead
    auto each = [&](auto with_z, auto&& step) {
      for (uint32_t m = i; m < end; ++m) {
        const uint32_t j = sidx[m], h0 = hit_start[j];
        const uint32_t h1 = min(hit_start[j + 1], hit_cap);
        if (h0 >= h1) continue;
        double2 p = xy[min(h0 + q, h1 - 1)];
        int32_t z = with_z ? hz[min(h0 + q, h1 - 1)] : 0;
        for (uint32_t h = h0; h < h1; h += G) {
          const uint32_t hn = min(h + G + q, h1 - 1);
          const double2 pn = xy[hn];
          const int32_t zn = with_z ? hz[hn] : 0;
          step(p, z, min(h1 - h, G));
          p = pn;
          z = zn;
        }
      }
    };
    double sum = 0;
    // adds the products of two arrays in order
    auto add = [&](const double* a, const double* b) {
#pragma unroll
      for (int half = 0; half < G; half += 8) {
        double x[8], y[8];
        mg_row(a + half, x);
        mg_row(b + half, y);
#pragma unroll
        for (int k = 0; k < 8; ++k) sum = fma(x[k], y[k], sum);
      }
    };
    int64_t nh = 0;
    each(std::false_type(), [&](const double2& p, int32_t, uint32_t cnt) {
      const bool have = q < cnt;
      lds[0][q] = have ? p.x : 0.0;
      lds[1][q] = have ? p.y : 0.0;
      nh += cnt;
      in_order();
#pragma unroll
      for (int half = 0; half < G; half += 8) {
        double x[8];
        mg_row(lds[q & 1] + half, x);
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += x[k];
      }
      in_order();
    });
    out[0] = (double)(end - i);
    out[1] = (double)nh;
    const double mx = nh ? of_lane(sum, 0) / nh : 0, my = nh ? of_lane(sum, 1) / nh : 0;
    sum = 0;
    each(std::false_type(), [&](const double2& p, int32_t, uint32_t cnt) {
      const bool have = q < cnt;
      const double u = have ? p.x - mx : 0.0, v = have ? p.y - my : 0.0;
      lds[0][q] = u;
      lds[1][q] = v;
      lds[2][q] = u * u;
      lds[3][q] = v * v;
      lds[4][q] = u * v;
      in_order();
      add(lds[fa], lds[fb]);
      in_order();
    });
    const double suu = of_lane(sum, 0), svv = of_lane(sum, 1), suv = of_lane(sum, 2);
    const double suuu = of_lane(sum, 3), svvv = of_lane(sum, 4), suvv = of_lane(sum, 5);
    const double svuu = of_lane(sum, 6);
    const double det = suu * svv - suv * suv;
    if (nh < 3 || !(fabs(det) > 0)) {
      store();
      continue;
    }
    const double b1 = 0.5 * (suuu + suvv), b2 = 0.5 * (svvv + svuu);
    const double uc = (b1 * svv - b2 * suv) / det, vc = (suu * b2 - suv * b1) / det;
    const double xc = mx + uc, yc = my + vc;
    out[2] = xc;
    out[3] = yc;
    out[4] = sqrt(uc * uc + vc * vc + (suu + svv) / nh);
    out[9] = 1;
    double psi_prev = 0, acc = 0, pmin = 0, pmax = 0;
    bool first = true;
    sum = 0;
    each(std::true_type(), [&](const double2& p, int32_t z, uint32_t cnt) {
      // (a lane past the last hit repeats that hit)
      const double psi = atan2(p.y - yc, p.x - xc);
      const double up = __shfl_up(psi, 1, G);
      lds[0][q] = (q == 0 && first) || q >= cnt ? 0.0 : mg_wrap(psi - (q == 0 ? psi_prev : up));
      first = false;
      psi_prev = of_lane(psi, G - 1);
      in_order();
      // the azimuth up to this lane's hit, steps added in order
      double a = 0;
#pragma unroll
      for (int half = 0; half < G; half += 8) {
        double x[8];
        mg_row(lds[0] + half, x);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          acc += x[k];
          if (q == half + k) a = acc;
        }
      }
      in_order();
      if (a < pmin) pmin = a;
      if (a > pmax) pmax = a;
      const bool have = q < cnt;
      lds[0][q] = have ? a : 0.0;
      lds[1][q] = have ? z / 65536.0 : 0.0;
      in_order();
      add(lds[q >> 1 & 1], lds[q & 1 ? 0 : 5]);  // acc, acc acc, z, z acc
      in_order();
    });
#pragma unroll
    for (int k = 1; k < G; k *= 2) {
      const double lo = __shfl_xor(pmin, k, G), hi = __shfl_xor(pmax, k, G);
      if (lo < pmin) pmin = lo;
      if (hi > pmax) pmax = hi;
    }
    const double sp = of_lane(sum, 0), sp2 = of_lane(sum, 1), sz = of_lane(sum, 2);
    const double szp = of_lane(sum, 3);
    const double dd = nh * sp2 - sp * sp;
    if (!(dd > 0)) {
      store();
      continue;
    }
    const double slope = (nh * szp - sp * sz) / dd, icpt = (sz - slope * sp) / nh;
    out[5] = slope;
    out[8] = fabs(slope) / out[4];
    out[10] = pmax - pmin;
    if (pmax - pmin < 2 * M_PI) {
      const double psi0 = atan2(-yc, -xc);
      double a = acc + mg_wrap(psi0 - psi_prev);
      if (slope >= 0) {
        while (a < pmax) a += 2 * M_PI;
        while (a - 2 * M_PI >= pmax) a -= 2 * M_PI;
      } else {
        while (a > pmin) a -= 2 * M_PI;
        while (a + 2 * M_PI <= pmin) a += 2 * M_PI;
      }
      const double zd0 = icpt + slope * a;
      out[6] = zd0;
      out[7] = 2.0 * (zd0 - 250.0);
      out[9] = 3;
    }
    store();
  }
}

// Bound by the FP64 instructions and the LDS traffic on large frames, where 8
// lanes per component waste fewer of both (half of 16 have no sum to add up),
// and on small ones by the longest component, whose hits are one chain that 16
// lanes shorten: on 139,000 segments 219 us with 8 lanes, 305 with 16 and 566
// with one; the whole call on one small collision 128, 111 and 350 us.  Four waves
// per SIMD, so the arrays are read eight values at a time: with both widths in the
// kernel the compiler's own choice of 172 registers took 299 us on the large one.
#define MG_FIT_WIDE 32768  // segments from which 8 lanes take a component
__global__ __launch_bounds__(64, 4) void k_mg_fit(const uint32_t* __restrict__ skey,
                                               const uint32_t* __restrict__ sidx,
                                               const uint32_t* n_trk_dev, uint32_t trk_cap,
                                               const uint32_t* __restrict__ hit_start,
                                               uint32_t hit_cap, const double* __restrict__ hxy,
                                               const int32_t* __restrict__ hz,
                                               double* __restrict__ fit, const DevStatus* st) {
  __shared__ __align__(16) double rows[8 * 6 * 10];
  static_assert(8 * 6 * 10 >= 4 * 6 * 18, "LDS of both widths");
  if (failed(st)) return;
  const uint32_t n = scan_count(n_trk_dev, trk_cap);
  if (n >= MG_FIT_WIDE) mg_fit_rows<8>(skey, sidx, n, hit_start, hit_cap, hxy, hz, fit, rows);
  else mg_fit_rows<16>(skey, sidx, n, hit_start, hit_cap, hxy, hz, fit, rows);
}

// One pass of a stable least-significant-digit radix sort of (key, value)
// pairs on the 8-bit digit at `shift`: the count step writes, per block of
// MG_SORT_BLOCK elements, the count of each digit; the scatter step places each
// element at its digit's position, ranking equal digits in index order (a wave's
// lanes by ballot, the waves of a block one after the other).  DIRECT (up to
// MG_SORT_DIRECT blocks, by capacity): the counts are bins[block * 256 + digit] and
// every block adds up its positions itself; beyond, bins[digit * nb + block] are
// scanned in place between the steps (a launch or two more, where a block would
// read more than that many counts per digit).  As many passes as the labels'
// bits need order them with equal keys in index order.
#define MG_SORT_DIRECT 512
#define MG_SORT_BLOCK 1024
template <bool SCATTER, bool DIRECT>
__global__ __launch_bounds__(256) void k_mg_rsort(const uint32_t* __restrict__ kin,
                                                  const uint32_t* __restrict__ vin,
                                                  const uint32_t* n_dev, uint32_t cap, int shift,
                                                  uint32_t* __restrict__ bins,
                                                  uint32_t* __restrict__ kout,
                                                  uint32_t* __restrict__ vout,
                                                  const DevStatus* st) {
  if (failed(st)) return;
  __shared__ uint32_t h[4][256];
  const uint32_t n = scan_count(n_dev, cap);
  const uint32_t nb = (n + MG_SORT_BLOCK - 1) / MG_SORT_BLOCK;
  if (blockIdx.x >= nb) return;  // uniform per workgroup
  const uint32_t b0 = blockIdx.x * MG_SORT_BLOCK;
  const uint32_t m = min((uint32_t)MG_SORT_BLOCK, n - b0);
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j][threadIdx.x] = 0;
  __syncthreads();
  uint32_t dig[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t i = 256u * w + 64u * j + lane;
    dig[j] = i < m ? (kin[b0 + i] >> shift) & 255u : 0u;
    if (i < m) atomicAdd(&h[w][dig[j]], 1u);
  }
  __syncthreads();
  const uint32_t d = threadIdx.x;
  const uint32_t c0 = h[0][d], c1 = h[1][d], c2 = h[2][d], c3 = h[3][d];
  const size_t bi = DIRECT ? (size_t)blockIdx.x * 256u + d : (size_t)d * nb + blockIdx.x;
  if (!SCATTER) {
    bins[bi] = c0 + c1 + c2 + c3;
    return;
  }
  uint32_t base;
  if (DIRECT) {
    __shared__ uint32_t lds[256 / 64 + 1];
    uint32_t all = 0, before = 0, total;
#pragma unroll 8
    for (uint32_t l = 0; l < nb; ++l) {
      const uint32_t v = bins[(size_t)l * 256u + d];
      all += v;
      before += l < blockIdx.x ? v : 0u;
    }
    base = block_excl_scan<uint32_t, 256>(all, lds, total) + before;
  } else {
    base = bins[bi];
  }
  __syncthreads();
  h[0][d] = base;
  h[1][d] = base + c0;
  h[2][d] = base + c0 + c1;
  h[3][d] = base + c0 + c1 + c2;
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t i = 256u * w + 64u * j + lane;
    const bool v = i < m;
    uint64_t eq = __ballot(v);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool on = (dig[j] >> bit) & 1u;
      const uint64_t bb = __ballot(on);
      eq &= on ? bb : ~bb;
    }
    if (v) {
      const uint32_t pos = h[w][dig[j]] + (uint32_t)__popcll(eq & below);
      kout[pos] = kin[b0 + i];
      vout[pos] = vin[b0 + i];
    }
    // the highest lane of each digit advances the digit's position
    if (v && (eq >> lane) == 1ull) h[w][dig[j]] += (uint32_t)__popcll(eq);
  }
}
