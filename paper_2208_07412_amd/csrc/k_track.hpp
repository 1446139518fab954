// Kalman track following, conflict resolution, refit and output.
//
// One tracklet per lane.  The state is (y, z - z_anchor, sin phi, tan lambda,
// q/pT) at the local x of a pad row; z is kept relative to the tracklet's
// first cluster so that FP32 keeps full precision in long time frames.  The
// covariance is a packed 5x5 upper triangle in registers.  Propagation is
// the exact helix in a uniform Bz field (no material, no process noise).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "k_cluster.hpp"
#include "k_links.hpp"

#define XCD_GROUPS 8  // sort groups of the following: one per XCD

#define FX_SCALE 1.52587890625e-05  // 2^-16

enum { TF_NOT_PD = 1, TF_REFIT_FAIL = 2, TF_FP64 = 4, TF_FP64_FAIL = 8, TF_TO_FP64 = 16 };

template <typename T>
struct Trk {
  T p[5];
  T c[15];
};

__device__ __forceinline__ constexpr int PI(int i, int j) {  // i <= j
  return i * 5 - i * (i - 1) / 2 + (j - i);
}

template <typename T>
__device__ __forceinline__ T cov(const T* c, int i, int j) {
  return i <= j ? c[PI(i, j)] : c[PI(j, i)];
}

// per-precision views of the parameter block
template <typename T>
struct PV;
template <>
struct PV<float> {
  const DevParams32* P;
  __device__ float x(int r) const { return P->x[r]; }
  __device__ float hw(int r) const { return P->hw[r]; }
  __device__ float vy(int r) const { return P->vy[r]; }
  __device__ float vz(int r) const { return P->vz[r]; }
  __device__ float chi2_max() const { return P->chi2_max; }
  __device__ float snp_max() const { return P->snp_max; }
  __device__ float b() const { return P->bz_b; }
  __device__ float c0_snp2() const { return P->c0_snp2; }
  __device__ float c0_tgl2() const { return P->c0_tgl2; }
  __device__ float c0_qpt2() const { return P->c0_qpt2; }
  __device__ float qpt_clamp() const { return P->qpt_clamp; }
  __device__ float edge_margin() const { return P->edge_margin; }
  __device__ float refit_snp_max() const { return P->refit_snp_max; }
  __device__ float c0r(int i) const { return P->c0r2[i]; }
};
template <>
struct PV<double> {
  const DevParams* P;
  __device__ double x(int r) const { return P->xd[r]; }
  __device__ double hw(int r) const { return P->hwd[r]; }
  __device__ double vy(int r) const { return P->vyd[r]; }
  __device__ double vz(int r) const { return P->vzd[r]; }
  __device__ double chi2_max() const { return P->chi2_max_d; }
  __device__ double snp_max() const { return P->snp_max_d; }
  __device__ double b() const { return P->bz_b_d; }
  __device__ double c0_snp2() const { return P->c0_snp2_d; }
  __device__ double c0_tgl2() const { return P->c0_tgl2_d; }
  __device__ double c0_qpt2() const { return P->c0_qpt2_d; }
  __device__ double qpt_clamp() const { return P->qpt_clamp_d; }
  __device__ double edge_margin() const { return P->edge_margin_d; }
  __device__ double refit_snp_max() const { return P->refit_snp_max_d; }
  __device__ double c0r(int i) const { return P->c0r2_d[i]; }
};

// Low-order parts of y and sin phi carried beside an FP32 state.  Over many
// rows a stiff track adds almost the same increment C dx to sin phi at every
// step, so FP32 rounding errs the same way each time and the sum drifts like
// a curvature offset of about ulp(sin phi) / dx; adding each increment with
// an error-free two-sum and keeping the rounding error removes the drift.
template <typename T>
struct LoParts {
  T y, s;
};

// a + b = hi + lo exactly (two-sum); lo accumulates into *acc
template <typename T>
__device__ __forceinline__ T two_sum_acc(T a, T b, T* acc) {
  const T b2 = b + *acc;
  const T hi = a + b2;
  const T bb = hi - a;
  *acc = (a - (hi - bb)) + (b2 - bb);
  return hi;
}

// exact row-to-row distance from the integer radii
template <typename T>
__device__ __forceinline__ T row_dx(const DevParams32* P, int r1, int r2) {
  return (T)(P->xfx[r2] - P->xfx[r1]) * (T)FX_SCALE;
}

// d(signed arc)/dC at fixed dx: integral over u in [0, dx] of
// u * s / (1 - s^2)^(3/2), s = s1 + C u, by 8-point Gauss-Legendre.
template <typename T>
__device__ __forceinline__ T darc_dc(T s1, T C, T dx) {
  const T X[8] = {(T)0.01985507175123188, (T)0.10166676129318664, (T)0.2372337950418355,
                  (T)0.4082826787521751,  (T)0.5917173212478249,  (T)0.7627662049581645,
                  (T)0.8983332387068134,  (T)0.9801449282487681};
  const T Wt[8] = {(T)0.05061426814518813, (T)0.11119051722668724, (T)0.15685332293894363,
                   (T)0.18134189168918100, (T)0.18134189168918100, (T)0.15685332293894363,
                   (T)0.11119051722668724, (T)0.05061426814518813};
  T acc = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const T s = s1 + C * dx * X[i];
    const T w = (T)1 - s * s;
    acc += Wt[i] * X[i] * s / (w * sqrt(w));
  }
  return acc * dx * dx;
}

// FP32: the same quadrature with w^(-3/2) from the hardware reciprocal square
// root (a Jacobian element: a few ulp are far below what the fit resolves).
template <>
__device__ __forceinline__ float darc_dc<float>(float s1, float C, float dx) {
  const float Cdx = C * dx;
  const float X[8] = {0.01985507175123188f, 0.10166676129318664f, 0.2372337950418355f,
                      0.4082826787521751f,  0.5917173212478249f,  0.7627662049581645f,
                      0.8983332387068134f,  0.9801449282487681f};
  const float Wt[8] = {0.05061426814518813f, 0.11119051722668724f, 0.15685332293894363f,
                       0.18134189168918100f, 0.18134189168918100f, 0.15685332293894363f,
                       0.11119051722668724f, 0.05061426814518813f};
  float acc = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float s = s1 + Cdx * X[i];
    const float r = __builtin_amdgcn_rsqf(1.0f - s * s);
    acc += (Wt[i] * X[i]) * s * (r * r * r);
  }
  return acc * dx * dx;
}

// Off-diagonal elements of the helix Jacobian d(state after)/d(state before)
// over one step.  Every other element is that of the identity: the Jacobian
// is unit upper triangular in (y, z, sin phi, tan lambda, q/pT).
template <typename T>
struct HJac {
  T j02, j04, j12, j13, j14, j24;
};

// Helix step of the state over dx; with J also the Jacobian.  Returns false
// (state untouched) if |sin phi| would reach snp_lim.
template <typename T>
__device__ __forceinline__ bool helix_step(T p[5], T dx, const PV<T>& pv, T snp_lim,
                                           LoParts<T>* lo, HJac<T>* J) {
  const T b = pv.b();
  const T C = -b * p[4];
  const T s1 = p[2];
  T slo = lo ? lo->s : (T)0;
  const T s2 = lo ? two_sum_acc(s1, C * dx, &slo) : s1 + C * dx;
  if (!(fabs(s2) < snp_lim)) return false;
  T c1, c2, ic1, ic2, iD, f, chord, L;
  const T N = s1 + s2;
  if constexpr (std::is_same<T, float>::value) {
    // FP32: hardware reciprocal and reciprocal square root (about 1 ulp)
    // instead of correctly rounded division and square root, and the series
    // of asin(h)/h for the small turning angles of one row step
    ic1 = __builtin_amdgcn_rsqf(1.0f - s1 * s1);
    ic2 = __builtin_amdgcn_rsqf(1.0f - s2 * s2);
    c1 = (1.0f - s1 * s1) * ic1;
    c2 = (1.0f - s2 * s2) * ic2;
    iD = __builtin_amdgcn_rcpf(c1 + c2);
    f = N * iD;
    const float q = 1.0f + f * f;
    chord = fabsf(dx) * (q * __builtin_amdgcn_rsqf(q));
    float h = chord * fabsf(C) * 0.5f;
    if (h > 1.0f) h = 1.0f;
    if (h < 0.1f) {
      const float h2 = h * h;
      L = chord * (1.0f + h2 * (1.0f / 6.0f + h2 * (3.0f / 40.0f + h2 * (5.0f / 112.0f +
                                                                         h2 * (35.0f / 1152.0f)))));
    } else {
      L = chord * asinf(h) / h;
    }
  } else {
    c1 = sqrt((T)1 - s1 * s1);
    c2 = sqrt((T)1 - s2 * s2);
    ic1 = (T)1 / c1;
    ic2 = (T)1 / c2;
    iD = (T)1 / (c1 + c2);
    f = N * iD;
    chord = fabs(dx) * sqrt((T)1 + f * f);
    T h = chord * fabs(C) * (T)0.5;
    if (h > (T)1) h = (T)1;
    L = h > (T)0 ? chord * asin(h) / h : chord;
  }
  const T D = c1 + c2;
  const T A = dx >= (T)0 ? L : -L;
  if (J) {
    const T iD2 = iD * iD;
    J->j02 = dx * ((T)2 * D + N * (s1 * ic1 + s2 * ic2)) * iD2;
    J->j04 = -b * dx * dx * (D + N * s2 * ic2) * iD2;
    J->j12 = p[3] * dx * N * (ic1 * ic2 * iD);
    J->j13 = A;
    J->j14 = -b * p[3] * darc_dc(s1, C, dx);
    J->j24 = -b * dx;
  }
  if (lo) {
    p[0] = two_sum_acc(p[0], dx * f, &lo->y);
    lo->s = slo;
  } else {
    p[0] += dx * f;
  }
  p[1] += p[3] * A;
  p[2] = s2;
  return true;
}

// Helix propagation over dx; with_cov also transports the covariance,
// C <- J C J^T.  Returns false (state untouched) if |sin phi| would reach
// snp_lim.
template <typename T>
__device__ __forceinline__ bool propagate(Trk<T>& k, T dx, const PV<T>& pv, bool with_cov,
                                          T snp_lim, LoParts<T>* lo = nullptr) {
  HJac<T> J;
  if (!helix_step(k.p, dx, pv, snp_lim, lo, with_cov ? &J : nullptr)) return false;
  if (with_cov) {
    const T j02 = J.j02, j04 = J.j04, j12 = J.j12, j13 = J.j13, j14 = J.j14, j24 = J.j24;
    T m[5][5];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
      for (int j = 0; j < 5; ++j) m[i][j] = cov(k.c, i, j);
    T t[5][5];  // J * M
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      t[0][j] = m[0][j] + j02 * m[2][j] + j04 * m[4][j];
      t[1][j] = m[1][j] + j12 * m[2][j] + j13 * m[3][j] + j14 * m[4][j];
      t[2][j] = m[2][j] + j24 * m[4][j];
      t[3][j] = m[3][j];
      t[4][j] = m[4][j];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {  // (J M) J^T, upper triangle
      const T col[5] = {t[i][0] + j02 * t[i][2] + j04 * t[i][4],
                        t[i][1] + j12 * t[i][2] + j13 * t[i][3] + j14 * t[i][4],
                        t[i][2] + j24 * t[i][4], t[i][3], t[i][4]};
#pragma unroll
      for (int j = i; j < 5; ++j) k.c[PI(i, j)] = col[j];
    }
  }
  return true;
}

// inverse of the residual covariance S = C_yz + V, once per row
template <typename T>
struct SInv {
  T i00, i01, i11;
};
template <typename T>
__device__ __forceinline__ SInv<T> s_inverse(const Trk<T>& k, T vy, T vz) {
  const T S00 = k.c[0] + vy, S01 = k.c[1], S11 = k.c[5] + vz;
  const T rd = (T)1 / (S00 * S11 - S01 * S01);
  return SInv<T>{S11 * rd, -S01 * rd, S00 * rd};
}

template <typename T>
__device__ __forceinline__ T chi2_of(const Trk<T>& k, T my, T mz, const SInv<T>& si) {
  const T r0 = my - k.p[0], r1 = mz - k.p[1];
  return r0 * r0 * si.i00 + (T)2 * r0 * r1 * si.i01 + r1 * r1 * si.i11;
}

// Kalman update with a (y, z) measurement, si the inverse residual
// covariance.  Returns false (state untouched) if |sin phi| >= 1 afterwards.
template <typename T>
__device__ __forceinline__ bool update(Trk<T>& k, T my, T mz, const SInv<T>& si) {
  const T r0 = my - k.p[0], r1 = mz - k.p[1];
  const T I00 = si.i00, I01 = si.i01, I11 = si.i11;
  T K0[5], K1[5], c0[5], c1v[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    c0[i] = cov(k.c, 0, i);
    c1v[i] = cov(k.c, 1, i);
    K0[i] = c0[i] * I00 + c1v[i] * I01;
    K1[i] = c0[i] * I01 + c1v[i] * I11;
  }
  const T np2 = k.p[2] + K0[2] * r0 + K1[2] * r1;
  if (!(fabs(np2) < (T)1)) return false;
#pragma unroll
  for (int i = 0; i < 5; ++i) k.p[i] += K0[i] * r0 + K1[i] * r1;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = i; j < 5; ++j) k.c[PI(i, j)] -= K0[i] * c0[j] + K1[i] * c1v[j];
  return true;
}

template <typename T>
__device__ __forceinline__ void c0_reset(Trk<T>& k, const PV<T>& pv, int r) {
#pragma unroll
  for (int i = 0; i < 15; ++i) k.c[i] = 0;
  k.c[PI(0, 0)] = pv.vy(r);
  k.c[PI(1, 1)] = pv.vz(r);
  k.c[PI(2, 2)] = pv.c0_snp2();
  k.c[PI(3, 3)] = pv.c0_tgl2();
  k.c[PI(4, 4)] = pv.c0_qpt2();
}

// unit-row of a cluster: the last ur with crow[ur] <= c
__device__ __forceinline__ uint32_t cluster_ur(const uint32_t* crow, uint32_t n_ur, uint32_t c) {
  uint32_t a = 0, b = n_ur;
  while (b - a > 1) {
    const uint32_t m = (a + b) >> 1;
    if (crow[m] <= c) a = m;
    else b = m;
  }
  return a;
}

struct FollowOut {
  int32_t* hits;      // [cap*152], rows [lo, hi] written
  float* state;       // [cap*6]: pass-B state + its row
  uint16_t* nhits;    // [cap]
  uint16_t* range;    // [cap]: lo | hi << 8
  uint8_t* ok;        // [cap]
  uint8_t* krow;      // [cap*152]: rows of the kept hits, ascending (after resolution)
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// Raw buffer resource over a device array (uniform base, no range limit:
// callers read inside the array; word 3 = 32-bit data format).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)0xFFFFFFFF,
                                           0x00020000);
}

// The better of two lanes' candidates (least chi2, the lower index on ties;
// -1 if neither has one), the other lane being the one that the DPP control
// CTRL names (a permutation of the lanes of each four).
template <int CTRL>
__device__ __forceinline__ void better_of(int32_t& best, float& bchi, int2& bq) {
  const int32_t ob = __builtin_amdgcn_mov_dpp(best, CTRL, 0xF, 0xF, false);
  const float oc = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(bchi), CTRL, 0xF, 0xF, false));
  const int32_t ox = __builtin_amdgcn_mov_dpp(bq.x, CTRL, 0xF, 0xF, false);
  const int32_t oy = __builtin_amdgcn_mov_dpp(bq.y, CTRL, 0xF, 0xF, false);
  const bool take = ob >= 0 && (best < 0 || oc < bchi || (oc == bchi && ob < best));
  best = take ? ob : best;
  bchi = take ? oc : bchi;
  bq.x = take ? ox : bq.x;
  bq.y = take ? oy : bq.y;
}

// Best candidate of row ur for the track state k: the cluster with the least
// chi2 within the cut, the lower index on ties (-1 if none).  Only the grid
// blocks within the z residual bound that chi2 alone sets (plus a margin) are
// scanned; bq receives the chosen cluster's position.  With a group of G > 1
// lanes (all holding k, and all calling), each lane takes every G-th pair of
// candidates and the group's best is agreed on at the end: the same cluster.
__device__ __forceinline__ int32_t search_row(const ClusterView& cl, const uint32_t* cblk,
                                              uint32_t nblk, uint32_t ur, const Trk<float>& k,
                                              int32_t anchor, float vz, const SInv<float>& si,
                                              float chi2max, uint32_t& n_cand, int2& bq,
                                              uint32_t G = 1, uint32_t sub = 0) {
  // the hardware square root (1 ulp): the margin of 3 bins below covers it
  const float w = __builtin_amdgcn_sqrtf(chi2max * (k.c[5] + vz));
  const float zabs = k.p[1] + (float)anchor * (float)FX_SCALE;
  const float flo = floorf(2.0f * (zabs - w)) - 3.0f, fhi = ceilf(2.0f * (zabs + w)) + 3.0f;
  // NaN or out-of-range windows collapse to an empty or clamped block range
  int32_t blo = flo > 0.0f ? (flo < 1.0e6f ? ((int32_t)flo >> CG_BSHIFT) : (int32_t)nblk) : 0;
  int32_t bhi = fhi >= 0.0f ? (fhi < 1.0e6f ? ((int32_t)fhi >> CG_BSHIFT) : (int32_t)nblk - 1) : -1;
  if (!(fhi >= 0.0f) || !(flo == flo)) bhi = -1;
  if (blo > (int32_t)nblk - 1) blo = nblk - 1;
  if (bhi > (int32_t)nblk - 1) bhi = nblk - 1;
  // Every load below is a cache line of its own per lane, and the following
  // is bound by their number: the row bounds come in one 8-byte load, the two
  // grid entries in one 16-byte load when the range spans at most 3 blocks,
  // the candidates two per 16-byte load.  Same clamps as row_range.
  // (buffer loads: the compiler keeps them whole; every read lies inside the
  // arrays, the row's own table included)
  const u32x2 rb = __builtin_amdgcn_raw_buffer_load_b64(buffer_of(cl.crow), (int)(ur * 4u), 0, 0);
  const uint32_t cap = cl.capacity;
  const uint32_t s0 = rb.x < cap ? rb.x : cap, s1 = rb.y < cap ? rb.y : cap;
  int32_t ilo = blo < 0 ? 0 : blo, ihi = bhi + 1 > (int32_t)nblk ? (int32_t)nblk : bhi + 1;
  if (ihi < ilo) ihi = ilo;
  const size_t rowe = (size_t)ur * (nblk + 1);
  uint32_t a, b;
  if (ihi - ilo <= 3 && ilo + 3 <= (int32_t)nblk) {
    const u32x4 e = __builtin_amdgcn_raw_buffer_load_b128(buffer_of(cblk), (int)((rowe + ilo) * 4u),
                                                          0, 0);
    const int d = ihi - ilo;
    a = e.x;
    b = d == 0 ? e.x : d == 1 ? e.y : d == 2 ? e.z : e.w;
  } else {
    a = cblk[rowe + ilo];
    b = cblk[rowe + ihi];
  }
  if (a < s0) a = s0;
  if (a > s1) a = s1;
  if (b < a) b = a;
  if (b > s1) b = s1;
  int32_t best = -1;
  float bchi = 0.0f;
  n_cand += b - a;
  // candidates in index order, two at a time (both loads of a pair in flight)
  for (uint32_t c0 = a + 2 * sub; c0 < b; c0 += 2 * G) {
    int2 q[2];
    if (c0 + 1 < b) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(buffer_of(cl.pos), (int)(c0 * 8u), 0, 0);
      q[0] = make_int2((int)v.x, (int)v.y);
      q[1] = make_int2((int)v.z, (int)v.w);
    } else {
      q[0] = cl.pos[c0];
      q[1] = make_int2(0, 0);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (c0 + j >= b) break;
      const float my = (float)q[j].x * (float)FX_SCALE;
      const float mz = (float)(q[j].y - anchor) * (float)FX_SCALE;
      const float x2 = chi2_of(k, my, mz, si);
      if (x2 <= chi2max && (best < 0 || x2 < bchi)) {
        best = (int32_t)(c0 + j);
        bchi = x2;
        bq = q[j];
      }
    }
  }
  // the least chi2 of the group, the lower index on ties
  if (G >= 2) better_of<0xB1>(best, bchi, bq);  // lanes 1 0 3 2 of each four
  if (G >= 4) better_of<0x4E>(best, bchi, bq);  // lanes 2 3 0 1
  return best;
}

// Per tracklet (by a walk of its cleaned up-links, unless the walk for the chain
// lengths has left them in pts): its middle and end clusters
// (0xFFFFFFFF for a tracklet that cannot be followed: broken chain or rows
// beyond the last), its start unit-row, and the sort key of the outward
// following pass: the rows above its start row (the most rows that pass can
// take), 0 if it cannot be followed.
__global__ __launch_bounds__(256) void k_tracklet_points(ClusterView cl, uint32_t n_ur,
                                                         const int32_t* __restrict__ upc,
                                                         const uint32_t* __restrict__ tl_start,
                                                         const uint16_t* __restrict__ tl_len,
                                                         const uint32_t* n_tl_dev, uint32_t tl_cap,
                                                         uint32_t* __restrict__ pts,
                                                         uint8_t* __restrict__ key,
                                                         uint32_t* __restrict__ qnext, int walked,
                                                         DevStatus* st) {
  // the counters of the fit stage and the queue counters of its following
  if (blockIdx.x == 0 && threadIdx.x < 2 * XCD_GROUPS) {
    if (threadIdx.x < 5) (&st->n_fallback)[threadIdx.x] = 0;
    qnext[threadIdx.x] = 0;
  }
  if (failed(st)) return;
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  const uint32_t n_cl = scan_count(cl.n_clusters, cl.capacity);
  uint32_t dt;
  for (uint32_t t = xcd_thread_item(n_tl, dt); t < n_tl; t += dt) {
    const uint32_t A = tl_start[t];
    const int L = tl_len[t];
    uint32_t M = 0xFFFFFFFFu, E = 0xFFFFFFFFu, urA = 0;
    uint8_t rows = 0;
    if (A < n_cl && L >= 3) {
      urA = cluster_ur(cl.crow, n_ur, A);
      const int r1 = (int)(urA % NROW);
      if (r1 + L <= NROW) {
        const int im = (L + 1) / 2 - 1;
        uint32_t c = A, m = A;
        bool bad = false;
        if (walked) {  // pts holds them, from the chains' lengths
          m = pts[(size_t)t * 3 + 0];
          c = pts[(size_t)t * 3 + 1];
        }
        for (int i = walked ? L : 1; i < L; ++i) {
          const int32_t nx = upc[c];
          if (nx < 0 || (uint32_t)nx >= n_cl) {
            bad = true;
            break;
          }
          c = (uint32_t)nx;
          if (i == im) m = c;
        }
        if (!bad) {
          M = m;
          E = c;
          rows = (uint8_t)(NROW - 1 - r1);
        }
      }
    }
    pts[(size_t)t * 3 + 0] = M;
    pts[(size_t)t * 3 + 1] = E;
    pts[(size_t)t * 3 + 2] = urA;
    key[t] = rows;
  }
}

// Stable counting sort of the tracklets by an 8-bit key, largest first.  The
// key is the most rows a following pass can take (rows above the start row
// outward; the row of the outermost pass-A hit inward): the passes that can
// run longest start first, and the lanes of a wave start on one row and step
// through the same rows, reading the same parts of the hit grid.  The sort
// can first split the tracklets into ngrp groups of consecutive blocks (so of
// consecutive units) and sort each group on its own: the following gives group
// g to the workgroups that the dispatcher places on XCD g, so each XCD's L2
// holds the hit data of its own units only.  Steps: k_sort_work<false>
// counts each block of SORT_BLOCK tracklets per key; k_sort_work<true> writes
// perm, ranking the elements of one key in index order, from the position of
// its block's first element of each key.  DIRECT (up to SORT_DIRECT blocks per
// group, by capacity): the counts are bins[block * 256 + key'], key' = 255 - key,
// and each block adds up its group's itself.  Beyond that they are
// bins[(g * 256 + key') * npg + block in group] (npg blocks per group) and an
// exclusive scan of bins in place, between the steps, leaves the positions (a sort
// on a central collision took 23 us in five launches, 19 in four, 10 with DIRECT;
// a 2 ms slice is as fast either way, which is where the line is drawn).
// Tracklets of equal estimate keep their order (unit, row, time), so neighbouring
// tracks share a wave.  Wave w of a workgroup takes the elements
// [256 w, 256 w + 256) of its block.  Launch at least
// ceil(capacity / SORT_BLOCK) + ngrp - 1 workgroups, over as many times 256 bins.
#define SORT_DIRECT 512
#define SORT_BLOCK 1024
__device__ __forceinline__ uint32_t sort_blocks_per_group(uint32_t n, uint32_t ngrp) {
  return ((n + SORT_BLOCK - 1) / SORT_BLOCK + ngrp - 1) / ngrp;
}

// Where group g of the sorted order of n items starts (n for g = ngrp).
__device__ __forceinline__ uint32_t sort_group_start(uint32_t n, uint32_t ngrp, uint32_t g) {
  const uint64_t s = (uint64_t)g * sort_blocks_per_group(n, ngrp) * SORT_BLOCK;
  return s < n ? (uint32_t)s : n;
}

// One item per thread over the sorted order of n items in ngrp groups:
// workgroup b takes group b % ngrp (gridDim.x is a multiple of ngrp), in the
// group's order; [i0, i1) with stride di are this thread's positions.
__device__ __forceinline__ void sorted_items(uint32_t ngrp, uint32_t n, uint32_t& i0, uint32_t& i1,
                                             uint32_t& di) {
  const uint32_t g = blockIdx.x % ngrp, j = blockIdx.x / ngrp, per = gridDim.x / ngrp;
  i1 = sort_group_start(n, ngrp, g + 1);
  i0 = j < per ? sort_group_start(n, ngrp, g) + j * blockDim.x + threadIdx.x : i1;
  di = per * blockDim.x;
}

template <bool SCATTER, bool DIRECT>
__global__ __launch_bounds__(256) void k_sort_work(const uint8_t* __restrict__ key,
                                                   const uint32_t* n_tl_dev, uint32_t tl_cap,
                                                   uint32_t ngrp, uint32_t* __restrict__ bins,
                                                   uint32_t* __restrict__ perm,
                                                   const DevStatus* st) {
  if (failed(st)) return;
  __shared__ uint32_t h[4][256];  // per wave: count per key, then next position per key
  const uint32_t n = scan_count(n_tl_dev, tl_cap);
  const uint32_t npg = sort_blocks_per_group(n, ngrp);
  if (blockIdx.x >= ngrp * npg) return;  // uniform per workgroup
  const uint32_t grp = blockIdx.x / npg, lb = blockIdx.x - grp * npg;
  const uint32_t b0 = blockIdx.x * SORT_BLOCK;
  const uint32_t m = b0 < n ? min((uint32_t)SORT_BLOCK, n - b0) : 0u;
  if (SCATTER && m == 0) return;  // uniform per workgroup
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j][threadIdx.x] = 0;
  __syncthreads();
  uint32_t bin[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t i = 256u * w + 64u * j + lane;
    bin[j] = i < m ? 255u - key[b0 + i] : 0u;
    if (i < m) atomicAdd(&h[w][bin[j]], 1u);
  }
  __syncthreads();
  const uint32_t k = threadIdx.x;
  const uint32_t c0 = h[0][k], c1 = h[1][k], c2 = h[2][k], c3 = h[3][k];
  const size_t bi = DIRECT ? (size_t)blockIdx.x * 256u + k : (size_t)(grp * 256u + k) * npg + lb;
  if (!SCATTER) {
    bins[bi] = c0 + c1 + c2 + c3;
    return;
  }
  uint32_t base;
  if (DIRECT) {
    // this key's counts in the group and in its blocks before this one
    __shared__ uint32_t lds[256 / 64 + 1];
    uint32_t all = 0, before = 0, total;
#pragma unroll 8
    for (uint32_t l = 0; l < npg; ++l) {
      const uint32_t v = bins[(size_t)(grp * npg + l) * 256u + k];
      all += v;
      before += l < lb ? v : 0u;
    }
    base = sort_group_start(n, ngrp, grp) + block_excl_scan<uint32_t, 256>(all, lds, total) + before;
  } else {
    base = bins[bi];
  }
  __syncthreads();
  h[0][k] = base;
  h[1][k] = base + c0;
  h[2][k] = base + c0 + c1;
  h[3][k] = base + c0 + c1 + c2;
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t i = 256u * w + 64u * j + lane;
    const bool v = i < m;
    uint64_t eq = __ballot(v);  // valid lanes with the same key
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool on = (bin[j] >> bit) & 1u;
      const uint64_t bb = __ballot(on);
      eq &= on ? bb : ~bb;
    }
    if (v) perm[h[w][bin[j]] + (uint32_t)__popcll(eq & below)] = b0 + i;
    // the highest lane of each key advances the key's position; the reads
    // above belong to an earlier instruction of this wave
    if (v && (eq >> lane) == 1ull) h[w][bin[j]] += (uint32_t)__popcll(eq);
  }
}

// Following of one tracklet per lane: seed and first update, pass A outward
// row by row, pass B inward from the outermost pass-A hit, result.

struct FollowLane {
  Trk<float> k;   // state at row r
  float sp[5];    // state after the last update (pass A, then pass B)
  uint32_t t;
  int32_t anchor;
  int32_t pre;    // candidate of the next row known before its helix step, or -1
  uint32_t ubase;
  int r, r1, L, nmiss, nh, hi, lo, rs;  // rs: row of sp
  i32x4 quad;   // hit-table entries of the four rows about row r
  i32x4 lower;  // pass B: of the four rows below them
  int pend;     // last row whose entry in quad is not stored yet, or -1
  uint32_t n_steps, n_cands, n_upds;      // work done (measurement)
};

// The hit table is read and written four rows at a time: a lane's tracklet has
// lines of its own, and with an entry at a time the lines of all the lanes in
// flight did not stay in the caches (the two passes of a 2 ms slice 1286 and 1142 us,
// with four at a time 969 and 986).
static_assert(NROW % 4 == 0, "whole quads");
__device__ __forceinline__ int32_t quad_get(i32x4 v, int row) {
  const int m = row & 3;
  return m < 2 ? (m == 0 ? v.x : v.y) : (m == 2 ? v.z : v.w);
}
__device__ __forceinline__ void quad_set(i32x4& v, int row, int32_t hit) {
  const int m = row & 3;
  v.x = m == 0 ? hit : v.x;
  v.y = m == 1 ? hit : v.y;
  v.z = m == 2 ? hit : v.z;
  v.w = m == 3 ? hit : v.w;
}
// The entries of the four rows below `row`'s four, if pass A wrote any of them.
__device__ __forceinline__ i32x4 quad_lower(const FollowLane& f, const FollowOut& fo, int row) {
  const int r0 = (row & ~3) - 4;
  if (r0 + 3 < f.r1) return i32x4{-1, -1, -1, -1};
  return *reinterpret_cast<const i32x4*>(fo.hits + (size_t)f.t * NROW + r0);
}

// Seed and first update of tracklet t; false if it cannot be followed.
__device__ __forceinline__ bool follow_init(FollowLane& f, uint32_t t, const ClusterView& cl,
                                            const uint32_t* tl_start, const uint16_t* tl_len,
                                            const int32_t* upc, const uint32_t* pts, FollowOut& fo,
                                            const DevParams32* P, const PV<float>& pv,
                                            bool lead = true) {
  if (lead) {
    fo.ok[t] = 0;
    fo.nhits[t] = 0;
    fo.range[t] = 0;
  }
  const uint32_t M = pts[(size_t)t * 3 + 0], E = pts[(size_t)t * 3 + 1];
  if (M == 0xFFFFFFFFu) return false;
  const uint32_t urA = pts[(size_t)t * 3 + 2];
  const uint32_t A = tl_start[t];
  const int L = tl_len[t];
  const int r1 = urA % NROW;
  f.t = t;
  f.L = L;
  f.r1 = r1;
  f.ubase = urA - r1;
  const int im = (L + 1) / 2 - 1;
  const int rM = r1 + im, rE = r1 + L - 1;
  const int2 qA = cl.pos[A], qM = cl.pos[M], qE = cl.pos[E];
  const int32_t anchor = qA.y;
  f.anchor = anchor;
  // ---- seed: circle through A, M, E; differences are exact integers
  const int64_t dxm = P->xfx[rM] - P->xfx[r1], dym = (int64_t)qM.x - qA.x;
  const int64_t dxe = P->xfx[rE] - P->xfx[r1], dye = (int64_t)qE.x - qA.x;
  const int64_t dxx = P->xfx[rE] - P->xfx[rM], dyy = (int64_t)qE.x - qM.x;
  const float cross = (float)(dxm * dye - dym * dxe) * (float)(FX_SCALE * FX_SCALE);
  const float fma_ = hypotf((float)dxm, (float)dym) * (float)FX_SCALE;
  const float fea = hypotf((float)dxe, (float)dye) * (float)FX_SCALE;
  const float fem = hypotf((float)dxx, (float)dyy) * (float)FX_SCALE;
  const float b = pv.b();
  float C = 2.0f * cross / (fma_ * fem * fea);
  float qpt = -C / b;
  qpt = fminf(fmaxf(qpt, -pv.qpt_clamp()), pv.qpt_clamp());
  C = -b * qpt;
  const float sarg = fminf(fmaxf(fea * C * 0.5f, -1.0f), 1.0f);
  const float phiA = atan2f((float)dye, (float)dxe) - asinf(sarg);
  const float h = fea * fabsf(C) * 0.5f;
  const float arc = h > 0.0f ? fea * asinf(fminf(h, 1.0f)) / h : fea;
  Trk<float>& k = f.k;
  k.p[0] = (float)qA.x * (float)FX_SCALE;
  k.p[1] = 0.0f;
  k.p[2] = sinf(phiA);
  k.p[3] = (float)(qE.y - anchor) * (float)FX_SCALE / arc;
  k.p[4] = qpt;
  if (!(fabsf(k.p[2]) < pv.snp_max())) return false;
  c0_reset(k, pv, r1);
  f.n_upds += 1;
  if (!update(k, k.p[0], 0.0f, s_inverse(k, pv.vy(r1), pv.vz(r1)))) return false;
  f.quad = (int32_t)A;  // (entries of rows that no pass visits are not read)
  f.pend = r1;
  f.nh = 1;
#pragma unroll
  for (int i = 0; i < 5; ++i) f.sp[i] = k.p[i];
  f.rs = r1;
  f.nmiss = 0;
  f.hi = r1;
  f.pre = L > 1 ? upc[A] : -1;  // the next row is on the tracklet's own chain
  f.r = r1;
  return true;
}

// Stores the hit-table entries about row r (QUAD), or that of row r (in quad.x).
template <bool QUAD>
__device__ __forceinline__ void follow_flush(FollowLane& f, const FollowOut& fo, bool lead) {
  int32_t* H = fo.hits + (size_t)f.t * NROW;
  if (f.pend >= 0 && lead) {
    if (QUAD) *reinterpret_cast<i32x4*>(H + (f.pend & ~3)) = f.quad;
    else H[f.pend] = f.quad.x;
  }
  f.pend = -1;
}

// Pass B start: the outermost pass-A hit (row rs) with a reset covariance;
// false if its update fails (the tracklet then ends with the pass-A state).
template <bool QUAD>
__device__ __forceinline__ bool follow_start_b(FollowLane& f, const ClusterView& cl,
                                               const FollowOut& fo, const PV<float>& pv) {
  Trk<float>& k = f.k;
#pragma unroll
  for (int i = 0; i < 5; ++i) k.p[i] = f.sp[i];
  c0_reset(k, pv, f.rs);
  f.lo = f.r1;
  const int32_t* H = fo.hits + (size_t)f.t * NROW;
  int32_t co;
  if (QUAD) {
    f.quad = *reinterpret_cast<const i32x4*>(H + (f.rs & ~3));
    f.lower = quad_lower(f, fo, f.rs);
    co = quad_get(f.quad, f.rs);
  } else {
    co = H[f.rs];
    f.pre = f.rs - 1 >= f.r1 ? H[f.rs - 1] : -1;
  }
  f.pend = -1;
  const int2 q = cl.pos[co];
  const float my = (float)q.x * (float)FX_SCALE;
  const float mz = (float)(q.y - f.anchor) * (float)FX_SCALE;
  ++f.n_upds;
  if (!update(k, my, mz, s_inverse(k, pv.vy(f.rs), pv.vz(f.rs)))) return false;
#pragma unroll
  for (int i = 0; i < 5; ++i) f.sp[i] = k.p[i];
  f.nmiss = 0;
  f.r = f.rs;
  return true;
}

__device__ __forceinline__ void follow_finish(const FollowLane& f, FollowOut& fo) {
  // six floats per tracklet at 8-byte alignment: three 8-byte stores
  float2* S = reinterpret_cast<float2*>(fo.state + (size_t)f.t * 6);
  S[0] = make_float2(f.sp[0], f.sp[1]);
  S[1] = make_float2(f.sp[2], f.sp[3]);
  S[2] = make_float2(f.sp[4], (float)f.rs);
  fo.nhits[f.t] = (uint16_t)f.nh;
  fo.range[f.t] = (uint16_t)(f.lo | (f.hi << 8));
  fo.ok[f.t] = 1;
}

// One row of pass A (outward, PA = 1) or pass B (inward, PA = 0).  Returns
// true when the pass has ended.  With a group of G lanes per tracklet, lane
// sub = 0 of the group writes.
template <int PA, bool QUAD = true>
__device__ __forceinline__ bool follow_step(FollowLane& f, const ClusterView& cl,
                                            const uint32_t* cblk, uint32_t nblk,
                                            const int32_t* upc, FollowOut& fo, const DevParams32* P,
                                            const PV<float>& pv, float chi2max, uint32_t G = 1,
                                            uint32_t sub = 0) {
  constexpr bool pa = PA == 1;
  const bool lead = sub == 0;
  const int rn = f.r + (pa ? 1 : -1);
  if (rn >= NROW || rn < 0) return true;
  if (QUAD && (rn & 3) == (pa ? 0 : 3)) {  // into the next four rows
    follow_flush<QUAD>(f, fo, lead);
    if (!pa) {
      f.quad = f.lower;
      f.lower = quad_lower(f, fo, rn);
    }
  }
  // Rows whose candidate is known before the helix step: the tracklet's own
  // chain (pass A) and the rows pass A covered (pass B: its hit, or -1 for a
  // row it missed, which is searched).  The candidate's position and the chain's
  // next candidate are loaded before the step, so their latency overlaps its
  // arithmetic.
  const bool known = pa ? rn < f.r1 + f.L : rn >= f.r1;
  int32_t cand = !known ? -1 : pa || !QUAD ? f.pre : quad_get(f.quad, rn);
  int2 q = make_int2(0, 0);
  if (cand >= 0) q = cl.pos[cand];
  const int rn2 = rn + (pa ? 1 : -1);
  int32_t pre2 = -1;
  if (pa ? (rn2 < f.r1 + f.L && cand >= 0) : (!QUAD && rn2 >= f.r1))
    pre2 = pa ? upc[cand] : fo.hits[(size_t)f.t * NROW + rn2];
  if (!QUAD) follow_flush<QUAD>(f, fo, lead);
  Trk<float>& k = f.k;
  // the row's constants in one round of LDS reads, before the step
  const float dx = row_dx<float>(P, f.r, rn);
  const float vy = pv.vy(rn), vz = pv.vz(rn), edge = pv.hw(rn) + pv.edge_margin();
  if (!propagate(k, dx, pv, true, pv.snp_max())) return true;
  ++f.n_steps;
  const SInv<float> si = s_inverse(k, vy, vz);
  bool fresh = false;
  if (!known || (!pa && cand < 0)) {
    if (fabsf(k.p[0]) > edge) return true;
    cand = search_row(cl, cblk, nblk, f.ubase + rn, k, f.anchor, vz, si, chi2max, f.n_cands, q, G,
                      sub);
    fresh = true;
  }
  if (pa || !QUAD) f.pre = pre2;
  f.r = rn;
  auto entry = [&](int32_t hit) {
    if (QUAD) quad_set(f.quad, rn, hit);
    else f.quad.x = hit;
    f.pend = rn;
  };
  // a row this pass visits first gets exactly one store: its hit, or -1
  const bool first = pa || (fresh && rn < f.lo);
  if (pa) f.hi = rn;
  else if (first) f.lo = rn;
  if (cand < 0) {
    if (first) entry(-1);
    if ((pa || rn < f.r1) && ++f.nmiss >= P->max_miss) return true;
    return false;
  }
  const float my = (float)q.x * (float)FX_SCALE;
  const float mz = (float)(q.y - f.anchor) * (float)FX_SCALE;
  ++f.n_upds;
  if (!update(k, my, mz, si)) {
    if (first) entry(-1);
    return true;
  }
  if (pa || fresh) {
    entry(cand);
    ++f.nh;
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) f.sp[i] = k.p[i];
  f.rs = rn;
  f.nmiss = 0;
  return false;
}

// Pass B start of tracklet t from what pass A left in the outputs: the
// state at the outermost pass-A hit, its row, the hit count and row range.
__device__ __forceinline__ void follow_resume(FollowLane& f, uint32_t t, const ClusterView& cl,
                                              const uint32_t* tl_start, const uint16_t* tl_len,
                                              const uint32_t* pts, const FollowOut& fo) {
  const uint32_t urA = pts[(size_t)t * 3 + 2];
  f.t = t;
  f.r1 = (int)(urA % NROW);
  f.ubase = urA - (uint32_t)f.r1;
  f.L = tl_len[t];
  f.anchor = cl.pos[tl_start[t]].y;
  const float2* S = reinterpret_cast<const float2*>(fo.state + (size_t)t * 6);
  const float2 s01 = S[0], s23 = S[1], s4r = S[2];
  f.sp[0] = s01.x;
  f.sp[1] = s01.y;
  f.sp[2] = s23.x;
  f.sp[3] = s23.y;
  f.sp[4] = s4r.x;
  f.rs = (int)s4r.y;
  f.nh = fo.nhits[t];
  f.hi = fo.range[t] >> 8;
  f.pre = -1;
}

enum { FP_A = 0, FP_B = 1, FP_AB = 2 };

// Following, one tracklet per lane.  FP_A: seed and pass A of the tracklets
// in the order perm gives, leaving the pass-A
// result in the outputs and the sort key of pass B (the row of the outermost
// pass-A hit) in key; FP_B: pass B of the tracklets that pass A
// followed, in the order perm gives; FP_AB: both passes per lane, tracklets in
// index order (perm unused).  Either way a tracklet's result is the same.
// COUNT: also count the work done (helix steps, candidates, updates) into
// per-wave counters, for measurement only.
template <int B, int PASS, bool COUNT>
__global__ __launch_bounds__(B) void k_follow(ClusterView cl, const uint32_t* __restrict__ cblk,
                                               uint32_t nblk, const int32_t* __restrict__ upc,
                                               const uint32_t* __restrict__ tl_start,
                                               const uint16_t* __restrict__ tl_len,
                                               const uint32_t* __restrict__ pts,
                                               const uint32_t* __restrict__ perm, uint32_t ngrp,
                                               uint8_t* __restrict__ key,
                                               const uint32_t* n_tl_dev, uint32_t tl_cap,
                                               FollowOut fo, ulonglong4* __restrict__ work,
                                               const DevParams* __restrict__ Pg, DevStatus* st) {
  const uint32_t wave = blockIdx.x * (B / 64) + (threadIdx.x >> 6);
  if (failed(st)) {
    if (COUNT && (threadIdx.x & 63) == 0) work[wave] = make_ulonglong4(0, 0, 0, 0);
    return;
  }
  // FP32 only: the parameter block without its FP64 copies
  __shared__ DevParams32 Ps;
  const DevParams32* P = params_to_lds(Pg, &Ps);
  const PV<float> pv{P};
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  const float chi2max = pv.chi2_max();
  uint32_t w_steps = 0, w_cands = 0, w_upds = 0;
  uint32_t i0 = blockIdx.x * blockDim.x + threadIdx.x, i1 = n_tl, di = gridDim.x * blockDim.x;
  if (PASS != FP_AB) sorted_items(ngrp, n_tl, i0, i1, di);
  for (uint32_t i = i0; i < i1; i += di) {
    const uint32_t t = PASS == FP_AB ? i : perm[i];
    FollowLane f;
    f.n_steps = f.n_cands = f.n_upds = 0;
    if (PASS == FP_B) {
      if (!fo.ok[t]) continue;
      follow_resume(f, t, cl, tl_start, tl_len, pts, fo);
    } else if (!follow_init(f, t, cl, tl_start, tl_len, upc, pts, fo, P, pv)) {
      if (PASS == FP_A) key[t] = 0;
      if (COUNT) w_upds += f.n_upds;
      continue;
    }
    if (PASS != FP_B) {
      while (!follow_step<1>(f, cl, cblk, nblk, upc, fo, P, pv, chi2max)) {
      }
      follow_flush<true>(f, fo, true);
    }
    if (PASS == FP_A) {
      f.lo = f.r1;
      follow_finish(f, fo);
      key[t] = (uint8_t)f.rs;
    } else if (follow_start_b<true>(f, cl, fo, pv)) {
      while (!follow_step<0>(f, cl, cblk, nblk, upc, fo, P, pv, chi2max)) {
      }
      follow_flush<true>(f, fo, true);
      follow_finish(f, fo);
    } else if (PASS == FP_AB) {
      follow_finish(f, fo);
    }
    if (COUNT) {
      w_steps += f.n_steps;
      w_cands += f.n_cands;
      w_upds += f.n_upds;
    }
  }
  if (!COUNT) return;
  // work counters: one plain store per wave, summed by k_work_sum (atomics
  // from every wave on one address would serialise at the end of the kernel)
  const unsigned long long s0 = wave_sum_u64(w_steps), s1 = wave_sum_u64(w_cands),
                           s2 = wave_sum_u64(w_upds);
  // lane slots: the wave runs as long as its busiest lane (exact when each
  // lane takes at most one tracklet, as with a grid that covers the capacity)
  const uint32_t mx = (uint32_t)wave_max_i32((int32_t)w_steps);
  if ((threadIdx.x & 63) == 0) work[wave] = make_ulonglong4(s0, s1, s2, 64ull * mx);
}

// Following with lane refill, one pass (FP_A or FP_B) over the tracklets in
// sorted order.  A lane holds one tracklet; when at least FOLLOW_REFILL lanes
// of a wave are free (or none is busy), the wave takes that many next
// tracklets of its workgroup's sort group with one atomic on the group's
// counter (refill = FOLLOW_REFILL), so the wave no longer runs as long as its longest tracklet with
// the other lanes idle.  Every tracklet is followed by exactly one lane, with
// the same arithmetic as k_follow, so the results do not depend on which lane
// or wave takes it.  The grid is sized to the resident waves, at most
// FOLLOW_Q_WAVES_PER_CU per compute unit (more would find the queues empty);
// qnext holds ngrp zeroed counters.
#define FOLLOW_REFILL 32
// Waves of the lane-refill grid per compute unit.  Each lane gathers lines of
// its own (hit grid, positions, hit table) that the L2 holds only while few
// lanes compete for it: on a 2 ms Pb-Pb slice the following stage took 2.76, 2.14,
// 1.92, 1.93 and 1.94 ms with 8, 12, 16, 20 and 24 waves per compute unit (and 1.97,
// 1.91, 1.92, 1.93 and 2.01 ms with refills of 16, 24, 32, 40 and 48 lanes).
#define FOLLOW_Q_WAVES_PER_CU 16
// Few tracklets: a sort group that fills at most the lanes of
// FOLLOW_SPREAD_WAVES waves (the resident grid of one group) has its tracklets
// dealt evenly over those waves, one round, and each tracklet is held by a
// group of up to FOLLOW_SPREAD_G lanes that search a row's candidates together.
// A lone wave issues an instruction every ~7 cycles whatever its lanes hold, so
// there the pass lasts as long as the instructions of the longest tracklet plus
// what the wave's other lanes add (other branches, more candidates per search):
// fewer tracklets per wave cost less per step, and idle SIMDs take the rest.
// Following stage (both passes, sorts included) from the queue and spread: 250
// tracklets 725 and 486 us, 5,457 732 and 576, 20,000 863 and 602, 67,000 953 and
// 669, 103,000 998 and 698, 141,000 1083 and 920, 179,000 1194 and 984, 240,000 1257
// and 1148.  Groups of at most 1, 2 and 4 lanes at 5,457: 549, 559 and 576 us, at
// 20,000: 648, 608 and 602, at 67,000: 739, 664 and 669 (wider groups have to agree
// through LDS and gained nothing); 128, 256 and 512 waves per group at 67,000: 944,
// 790 and 669 us.  Above 64 per wave (262,144 tracklets in all) lanes are refilled
// from the queue instead: a 2 ms slice's 730,000 take 1.92 ms there, and spreading
// them over more waves evicts lines (above).
#define FOLLOW_SPREAD_WAVES 512
#define FOLLOW_SPREAD_SLOTS 64
#define FOLLOW_SPREAD_G 4
template <int B, int PASS, bool COUNT>
__global__ __launch_bounds__(B) void k_follow_q(ClusterView cl, const uint32_t* __restrict__ cblk,
                                                 uint32_t nblk, const int32_t* __restrict__ upc,
                                                 const uint32_t* __restrict__ tl_start,
                                                 const uint16_t* __restrict__ tl_len,
                                                 const uint32_t* __restrict__ pts,
                                                 const uint32_t* __restrict__ perm, uint32_t ngrp,
                                                 uint32_t* __restrict__ qnext,
                                                 uint32_t refill,
                                                 uint8_t* __restrict__ key,
                                                 const uint32_t* n_tl_dev, uint32_t tl_cap,
                                                 FollowOut fo, ulonglong4* __restrict__ work,
                                                 const DevParams* __restrict__ Pg, DevStatus* st) {
  static_assert(PASS == FP_A || PASS == FP_B, "one pass per launch");
  const uint32_t wave = blockIdx.x * (B / 64) + (threadIdx.x >> 6);
  if (failed(st)) {
    if (COUNT && (threadIdx.x & 63) == 0) work[wave] = make_ulonglong4(0, 0, 0, 0);
    return;
  }
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  // this workgroup's sort group: positions [gs, ge) of perm
  const uint32_t g = blockIdx.x % ngrp;
  const uint32_t gs = sort_group_start(n_tl, ngrp, g), ge = sort_group_start(n_tl, ngrp, g + 1);
  // few tracklets: slots per wave and lanes per slot of the group's spread
  const uint32_t wpb = B / 64, gw = gridDim.x / ngrp * wpb;
  const uint32_t j0 = blockIdx.x / ngrp * wpb;
  const uint32_t sw = gw < FOLLOW_SPREAD_WAVES ? gw : FOLLOW_SPREAD_WAVES;
  const uint32_t per = (ge - gs + sw - 1) / sw;
  const bool spread = per <= FOLLOW_SPREAD_SLOTS;
  if (!COUNT && spread && j0 * per >= ge - gs) return;  // uniform per workgroup
  // FP32 only: the parameter block without its FP64 copies
  __shared__ DevParams32 Ps;
  const DevParams32* P = params_to_lds(Pg, &Ps);
  const PV<float> pv{P};
  const float chi2max = pv.chi2_max();
  const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
  uint32_t w_steps = 0, w_cands = 0, w_upds = 0, w_iter = 0;
  FollowLane f;
  if (spread) {
    uint32_t G = 1;
    while (G < FOLLOW_SPREAD_G && per * (2 * G) <= 64) G *= 2;
    const uint32_t lane = threadIdx.x & 63, sub = lane & (G - 1), slot = lane / G;
    const bool lead = sub == 0;
    const uint32_t i = gs + (j0 + (threadIdx.x >> 6)) * per + slot;
    if (slot < per && i < ge) {
      const uint32_t t = perm[i];
      f.n_steps = f.n_cands = f.n_upds = 0;
      bool busy = false;
      if (PASS == FP_B) {
        if (fo.ok[t]) {
          follow_resume(f, t, cl, tl_start, tl_len, pts, fo);
          busy = follow_start_b<false>(f, cl, fo, pv);
        }
      } else {
        busy = follow_init(f, t, cl, tl_start, tl_len, upc, pts, fo, P, pv, lead);
        if (!busy && lead) key[t] = 0;
      }
      if (busy) {
        // (few waves: the caches hold their lines, and an entry at a time takes
        // fewer instructions of the one long chain)
        constexpr bool quad = false;
        while (!follow_step<PASS == FP_A ? 1 : 0, quad>(f, cl, cblk, nblk, upc, fo, P, pv, chi2max, G,
                                                  sub)) {
          if (COUNT) ++w_iter;
        }
        if (COUNT) ++w_iter;
        follow_flush<quad>(f, fo, lead);
        if (PASS == FP_A) f.lo = f.r1;
        if (lead) {
          follow_finish(f, fo);
          if (PASS == FP_A) key[f.t] = (uint8_t)f.rs;
        }
      }
      if (COUNT && lead) {
        w_steps = f.n_steps;
        w_cands = f.n_cands;
        w_upds = f.n_upds;
      }
    }
    if (COUNT) w_iter = (uint32_t)wave_max_i32((int32_t)w_iter);
  }
  bool busy = false, retired = spread;
  for (;;) {
    const uint64_t want = __ballot(!busy && !retired);
    const uint32_t nwant = (uint32_t)__popcll(want);
    const bool any_busy = __ballot(busy) != 0ull;
    if (!any_busy && nwant == 0) break;
    if (nwant >= refill || (!any_busy && nwant > 0)) {
      const int lead = __ffsll((long long)want) - 1;
      uint32_t base = 0;
      if ((int)(threadIdx.x & 63) == lead) base = atomicAdd(&qnext[g], nwant);
      base = (uint32_t)__shfl((int)base, lead, 64);
      if (!busy && !retired) {
        const uint32_t i = gs + base + (uint32_t)__popcll(want & below);
        if (i >= ge) {
          retired = true;
        } else {
          const uint32_t t = perm[i];
          f.n_steps = f.n_cands = f.n_upds = 0;
          if (PASS == FP_B) {
            if (fo.ok[t]) {
              follow_resume(f, t, cl, tl_start, tl_len, pts, fo);
              busy = follow_start_b<true>(f, cl, fo, pv);
            }
          } else {
            busy = follow_init(f, t, cl, tl_start, tl_len, upc, pts, fo, P, pv);
            if (!busy) key[t] = 0;
          }
          if (COUNT && !busy) w_upds += f.n_upds;
        }
      }
    }
    if (COUNT) ++w_iter;
    if (busy && follow_step<PASS == FP_A ? 1 : 0>(f, cl, cblk, nblk, upc, fo, P, pv, chi2max)) {
      busy = false;
      follow_flush<true>(f, fo, true);
      if (PASS == FP_A) {
        f.lo = f.r1;
        follow_finish(f, fo);
        key[f.t] = (uint8_t)f.rs;
      } else {
        follow_finish(f, fo);
      }
      if (COUNT) {
        w_steps += f.n_steps;
        w_cands += f.n_cands;
        w_upds += f.n_upds;
      }
    }
  }
  if (!COUNT) return;
  const unsigned long long s0 = wave_sum_u64(w_steps), s1 = wave_sum_u64(w_cands),
                           s2 = wave_sum_u64(w_upds);
  // lane slots: 64 per loop round of the wave
  if ((threadIdx.x & 63) == 0) work[wave] = make_ulonglong4(s0, s1, s2, 64ull * w_iter);
}

// Sum of the following's per-wave work counters into the status block.
__global__ __launch_bounds__(1024) void k_work_sum(const ulonglong4* __restrict__ work,
                                                   uint32_t n, DevStatus* st) {
  __shared__ unsigned long long part[4][16];
  unsigned long long a = 0, b = 0, c = 0, e = 0;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    const ulonglong4 v = work[i];
    a += v.x;
    b += v.y;
    c += v.z;
    e += v.w;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    a += __shfl_xor(a, d, 64);
    b += __shfl_xor(b, d, 64);
    c += __shfl_xor(c, d, 64);
    e += __shfl_xor(e, d, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = a;
    part[1][threadIdx.x >> 6] = b;
    part[2][threadIdx.x >> 6] = c;
    part[3][threadIdx.x >> 6] = e;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long s[4] = {0, 0, 0, 0};
    for (int k = 0; k < 4; ++k)
      for (uint32_t w = 0; w < blockDim.x / 64; ++w) s[k] += part[k][w];
    st->f_steps = s[0];
    st->f_cands = s[1];
    st->f_upds = s[2];
    st->f_slots = s[3];
  }
}

// Claim priority of a track: more hits first, then the lower tracklet id
// (tracklet ids stay below 2^24, hit counts below 2^8).
__device__ __forceinline__ uint32_t track_key(uint32_t nh, uint32_t t) {
  return (nh << 24) | (0xFFFFFFu - t);
}

// Conflict resolution: a wave takes KEEP_GROUP consecutive tracklets and the rows
// of their hit tables one after the other, 64 to a chunk, KEEP_CHUNKS chunks at a
// time: their hits are loaded together, then the hits' owners.  Bound by the
// gathers of owners, a line each (on a 2 ms slice the kernels, with every claim
// stored and then looked at, took 745 us with a tracklet at a time, 64 rows to a
// load, 668 this way; 741 with 8 tracklets; a tracklet per lane, 64 of them over one
// row after the other, was slower, 880: the lanes' hits share few lines).
#define KEEP_GROUP 4
#define KEEP_CHUNKS 4
// The rows of a tracklet that a kernel takes: all from its first to its last, those
// of its chain, or the rest.
enum { ROWS_ALL = 0, ROWS_CHAIN = 1, ROWS_REST = 2 };
struct BidGroup {
  uint32_t info;  // lane k: 1 | hit count << 8 | row range << 16 of tracklet t0 + k if it
                  // bids (followed, at least min_track_hits hits), else 0
  uint32_t rows;  // lane k: its first row | rows before the gap << 8 | rows of the gap << 16
  uint32_t pre;   // lane k: rows of the tracklets before it
  uint32_t tot;   // rows of the group
  uint32_t end[KEEP_GROUP];  // rows up to and with the k-th (uniform)
};
// (pts and tl_len: the tracklets' start unit-rows and chain lengths, not read for
// ROWS_ALL)
template <int ROWS>
__device__ __forceinline__ BidGroup bid_group(const FollowOut& fo, const uint32_t* pts,
                                              const uint16_t* tl_len, uint32_t t0, uint32_t t1,
                                              int min_hits) {
  BidGroup g;
  const uint32_t t = t0 + (threadIdx.x & 63);
  g.info = 0;
  g.rows = 0;
  uint32_t len = 0;
  if (t < t1 && fo.ok[t]) {
    const uint32_t nh = fo.nhits[t];
    if ((int)nh >= min_hits) {
      g.info = 1u | (nh << 8) | ((uint32_t)fo.range[t] << 16);
      const uint32_t lo = (g.info >> 16) & 255, hi = g.info >> 24;
      g.rows = lo | 255u << 8;
      len = hi - lo + 1;
      if (ROWS != ROWS_ALL) {
        const uint32_t r1 = pts[(size_t)t * 3 + 2] % NROW;  // lo <= r1 <= hi
        const uint32_t n = min((uint32_t)tl_len[t], hi + 1 - r1);
        g.rows = ROWS == ROWS_CHAIN ? r1 | 255u << 8 : lo | (r1 - lo) << 8 | n << 16;
        len = ROWS == ROWS_CHAIN ? n : len - n;
      }
    }
  }
  const uint32_t end = wave_incl_scan(len);
  g.pre = end - len;
#pragma unroll
  for (int k = 0; k < KEEP_GROUP; ++k)
    g.end[k] = (uint32_t)__builtin_amdgcn_readlane((int)end, k);
  g.tot = g.end[KEEP_GROUP - 1];
  return g;
}

// A row of the group: its tracklet (t0 + k, what bid_group holds of it), the row
// and the hit there (-1: none, or past the group's rows).
struct BidRow {
  uint32_t k, info;
  int32_t r, c;
};
template <int ROWS>
__device__ __forceinline__ BidRow bid_row(const BidGroup& g, const FollowOut& fo, uint32_t t0,
                                          uint32_t e, uint32_t n_cl_cap) {
  BidRow x;
  x.k = 0;
#pragma unroll
  for (int k = 0; k + 1 < KEEP_GROUP; ++k) x.k += e >= g.end[k];
  x.info = (uint32_t)__shfl((int)g.info, (int)x.k);
  const uint32_t rows = (uint32_t)__shfl((int)g.rows, (int)x.k);
  const uint32_t i = e - (uint32_t)__shfl((int)g.pre, (int)x.k);
  x.r = (int32_t)((rows & 255) + i);
  if (ROWS == ROWS_REST && i >= ((rows >> 8) & 255)) x.r += (int32_t)(rows >> 16);
  x.c = e < g.tot ? fo.hits[(size_t)(t0 + x.k) * NROW + x.r] : -1;
  if ((uint32_t)x.c >= n_cl_cap) x.c = -1;
  return x;
}

// Every followed tracklet with enough hits bids for its clusters: the owner of a
// cluster is the largest key among its bidders.  The owners start at 0, below
// every key.
// The tracklets of stage_tracklets take two launches: ROWS_CHAIN stores the key of
// each at the clusters of its own chain; ROWS_REST looks at the owners of its other
// clusters and raises them by atomicMax where its key is larger.  A cluster lies in
// one chain at most (a cleaned link is its two clusters' choice of each other, so no
// cluster is the upper end of two, and a chain starts at a cluster that is the upper
// end of none): the first launch writes no word twice, and the second one reads and
// writes by atomics of the device's scope, so that the result is the maximum
// whichever workgroups run on whichever XCD.
// A caller's tracklets may overlap: ROWS_ALL, one atomicMax per hit, in one launch.
// Whole calls, with every key stored and then looked at by plain loads (which
// leaves open what a load finds where two XCDs have stored to one word), with the
// chains' keys stored, and with ROWS_ALL: 2 ms slice 6030, 6090 and 6439 us; 20
// stressed collisions 2472, 2509 and 2499; one central collision 1128, 1127 and
// 1128; fit of ten collisions 1078, 1086 and 1088.  With every key stored by
// device-scope atomics and looked at: 6334, 2558, 1136 and 1117.
template <int ROWS>
__global__ __launch_bounds__(256) void k_claim(FollowOut fo, const uint32_t* __restrict__ pts,
                                               const uint16_t* __restrict__ tl_len,
                                               const uint32_t* n_tl_dev, uint32_t tl_cap,
                                               uint32_t* __restrict__ owner,
                                               uint32_t n_cl_cap, const DevParams* __restrict__ P,
                                               const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t n_grp = (n_tl + KEEP_GROUP - 1) / KEEP_GROUP;
  uint32_t nw;
  for (uint32_t i = xcd_wave_item(n_grp, nw); i < n_grp; i += nw) {
    const uint32_t t0 = i * KEEP_GROUP, t1 = min(t0 + KEEP_GROUP, n_tl);
    const BidGroup g = bid_group<ROWS>(fo, pts, tl_len, t0, t1, P->min_track_hits);
    for (uint32_t e0 = lane; e0 - lane < g.tot; e0 += 64 * KEEP_CHUNKS) {
      BidRow x[KEEP_CHUNKS];
#pragma unroll
      for (int m = 0; m < KEEP_CHUNKS; ++m) x[m] = bid_row<ROWS>(g, fo, t0, e0 + 64 * m, n_cl_cap);
      uint32_t o[KEEP_CHUNKS];
#pragma unroll
      for (int m = 0; m < KEEP_CHUNKS; ++m) {
        o[m] = x[m].c >= 0 ? 0u : 0xFFFFFFFFu;  // (nothing to claim)
        if (ROWS == ROWS_REST && x[m].c >= 0)
          o[m] = __hip_atomic_load(&owner[x[m].c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int m = 0; m < KEEP_CHUNKS; ++m) {
        const uint32_t key = track_key((x[m].info >> 8) & 255, t0 + x[m].k);
        if (o[m] >= key) continue;
        if (ROWS == ROWS_CHAIN) owner[x[m].c] = key;
        else atomicMax(&owner[x[m].c], key);
      }
    }
  }
}

// Hits each track keeps after the claims; < min_track_hits drops the track.
// The kept count is also the refit's sort key: the refit takes the tracks
// sorted by it, so the lanes of a wave refit tracks of equal length.
__global__ __launch_bounds__(256) void k_keep(FollowOut fo, const uint32_t* n_tl_dev,
                                              uint32_t tl_cap,
                                              const uint32_t* __restrict__ owner,
                                              uint32_t n_cl_cap, uint16_t* __restrict__ nkept,
                                              uint8_t* __restrict__ key,
                                              const DevParams* __restrict__ P,
                                              const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  const uint32_t lane = threadIdx.x & 63;
  uint32_t nw;
  // a wave takes KEEP_GROUP consecutive tracklets; lane k collects the count
  // of the k-th, and the counts go out as one run per array
  const uint32_t n_grp = (n_tl + KEEP_GROUP - 1) / KEEP_GROUP;
  const uint64_t below = (1ull << lane) - 1ull;
  for (uint32_t i = xcd_wave_item(n_grp, nw); i < n_grp; i += nw) {
    const uint32_t t0 = i * KEEP_GROUP, t1 = min(t0 + KEEP_GROUP, n_tl);
    const BidGroup g = bid_group<ROWS_ALL>(fo, nullptr, nullptr, t0, t1, P->min_track_hits);
    uint32_t n[KEEP_GROUP] = {};  // kept so far (uniform)
    for (uint32_t e0 = lane; e0 - lane < g.tot; e0 += 64 * KEEP_CHUNKS) {
      BidRow x[KEEP_CHUNKS];
#pragma unroll
      for (int m = 0; m < KEEP_CHUNKS; ++m)
        x[m] = bid_row<ROWS_ALL>(g, fo, t0, e0 + 64 * m, n_cl_cap);
      uint32_t o[KEEP_CHUNKS];
#pragma unroll
      for (int m = 0; m < KEEP_CHUNKS; ++m) o[m] = x[m].c >= 0 ? owner[x[m].c] : 0u;
#pragma unroll
      for (int m = 0; m < KEEP_CHUNKS; ++m) {
        // (not by the owner alone: the key of tracklet 2^24 - 1 is 0 if it does not bid)
        const bool kept = x[m].c >= 0 && o[m] == track_key((x[m].info >> 8) & 255, t0 + x[m].k);
        uint32_t at = 0;
#pragma unroll
        for (int k = 0; k < KEEP_GROUP; ++k) {
          const uint64_t mask = __ballot(kept && x[m].k == (uint32_t)k);
          if (x[m].k == (uint32_t)k) at = n[k] + (uint32_t)__popcll(mask & below);
          n[k] += (uint32_t)__popcll(mask);
        }
        if (kept) fo.krow[(size_t)(t0 + x[m].k) * NROW + at] = (uint8_t)x[m].r;
      }
    }
    uint32_t mine = 0;  // lane k: kept by the k-th
#pragma unroll
    for (int k = 0; k < KEEP_GROUP; ++k)
      if (lane == (uint32_t)k && (int)n[k] >= P->min_track_hits) mine = n[k];
    if (t0 + lane < t1) {
      nkept[t0 + lane] = (uint16_t)mine;
      key[t0 + lane] = (uint8_t)mine;  // sort key of the refit (n <= NROW)
    }
  }
}

struct RefitOut {
  float* par;      // [cap*5]
  float* cov;      // [cap*15]
  float* chi2;     // [cap]
  uint8_t* row;    // [cap]
  uint8_t* flags;  // [cap]
};

__device__ __forceinline__ int32_t tl_anchor(const ClusterView& cl, const uint32_t* tl_start,
                                             uint32_t t) {
  return cl.z_fx[tl_start[t]];
}

// ------------------------------------------------------------------ refit
// The refit keeps its covariance as UD factors, C = U D U^T, with U unit
// upper triangular (u[i][j] for j > i; the rest is implied) and D diagonal.
// The helix Jacobian is unit upper triangular too and there is no process
// noise, so a propagation is U <- J U with D unchanged.  A (y, z)
// measurement with independent errors is two scalar updates in Bierman's
// form: each pivot d_j becomes d_j alpha_(j-1) / alpha_j with alpha a running
// sum of non-negative terms, so the covariance stays positive definite and
// keeps FP32 precision while the broad start variances collapse by orders
// of magnitude (the dense form loses it to cancellation there).
template <typename T>
struct UDCov {
  T u[5][5];  // strictly upper part only
  T d[5];
};

__device__ __forceinline__ float rcp_of(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_of(double x) { return 1.0 / x; }

// U <- J U (rows 0..2 change; row 2 is read before it is written)
template <typename T>
__device__ __forceinline__ void ud_propagate(UDCov<T>& c, const HJac<T>& J) {
  const T u23 = c.u[2][3], u24 = c.u[2][4], u34 = c.u[3][4];
  c.u[0][2] += J.j02;
  c.u[0][3] += J.j02 * u23;
  c.u[0][4] += J.j02 * u24 + J.j04;
  c.u[1][2] += J.j12;
  c.u[1][3] += J.j12 * u23 + J.j13;
  c.u[1][4] += J.j12 * u24 + J.j13 * u34 + J.j14;
  c.u[2][4] += J.j24;
}

// Scalar measurement of parameter M with variance r (Bierman): updates the
// factors, writes the gain K and returns the residual variance alpha.
template <int M, typename T>
__device__ __forceinline__ T ud_update(UDCov<T>& c, T r, T K[5]) {
  T f[5], v[5], b[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    f[j] = j < M ? (T)0 : (j == M ? (T)1 : c.u[M][j]);
    v[j] = c.d[j] * f[j];
    b[j] = 0;
  }
  T alpha = r, ia = rcp_of(r);
#pragma unroll
  for (int j = M; j < 5; ++j) {
    const T ap = alpha, iap = ia;
    alpha = ap + f[j] * v[j];
    ia = rcp_of(alpha);
    c.d[j] *= ap * ia;
    const T lam = -f[j] * iap;
#pragma unroll
    for (int i = 0; i < j; ++i) {
      const T uij = c.u[i][j];
      c.u[i][j] = uij + b[i] * lam;
      b[i] += uij * v[j];
    }
    b[j] = v[j];
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) K[i] = b[i] * ia;
  return alpha;
}

// C = U D U^T, packed upper triangle
template <typename T>
__device__ __forceinline__ void ud_to_cov(const UDCov<T>& c, T* out) {
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = i; j < 5; ++j) {
      T a = 0;
#pragma unroll
      for (int k = j; k < 5; ++k) {
        const T uik = k == i ? (T)1 : c.u[i][k];
        const T ujk = k == j ? (T)1 : c.u[j][k];
        a += uik * c.d[k] * ujk;
      }
      out[PI(i, j)] = a;
    }
}

// positive definite: every pivot of the factorisation > 0 (NaN fails)
template <typename T>
__device__ __forceinline__ bool ud_pd(const UDCov<T>& c) {
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 5; ++j) ok = ok && c.d[j] > (T)0;
  return ok;
}

// Kalman update of the refit with the (y, z) measurement, as a y update then
// a z update; the y residual includes the low-order part of y.  Returns false
// if |sin phi| >= 1 afterwards (the track then fails).
template <typename T>
__device__ __forceinline__ bool ud_measure(T p[5], UDCov<T>& c, LoParts<T>* lo, T my, T mz, T vy,
                                           T vz, T* chi2) {
  T K[5];
  const T ry = lo ? (my - p[0]) - lo->y : my - p[0];
  const T ay = ud_update<0>(c, vy, K);
  if (lo) {
    p[0] = two_sum_acc(p[0], K[0] * ry, &lo->y);
    p[2] = two_sum_acc(p[2], K[2] * ry, &lo->s);
  } else {
    p[0] += K[0] * ry;
    p[2] += K[2] * ry;
  }
  p[1] += K[1] * ry;
  p[3] += K[3] * ry;
  p[4] += K[4] * ry;
  const T rz = mz - p[1];
  const T az = ud_update<1>(c, vz, K);
  if (lo) {
    p[0] = two_sum_acc(p[0], K[0] * rz, &lo->y);
    p[2] = two_sum_acc(p[2], K[2] * rz, &lo->s);
  } else {
    p[0] += K[0] * rz;
    p[2] += K[2] * rz;
  }
  p[1] += K[1] * rz;
  p[3] += K[3] * rz;
  p[4] += K[4] * rz;
  *chi2 = ry * ry * rcp_of(ay) + rz * rz * rcp_of(az);
  return fabs(p[2]) < (T)1;
}

// Kalman steps of the refit over the kept hits i, i-1, ... (rows
// descending); the state sits at row r_state.  On return i is the next kept
// hit.  Returns 1 if the helix cannot reach a hit's row or an update fails;
// pd turns false if an update left a pivot that is not positive.
template <typename T>
__device__ int refit_run(uint32_t t, const ClusterView& cl, int32_t anchor, const FollowOut& fo,
                         const DevParams* P, T p[5], UDCov<T>& c, T& chi2s, int& r_state, int& i,
                         bool& pd, LoParts<T>* lp) {
  const PV<T> pv{P};
  const int32_t* H = fo.hits + (size_t)t * NROW;
  const uint8_t* KR = fo.krow + (size_t)t * NROW;
  if (i < 0) return 0;
  // a hit's row, cluster and position are dependent loads: they are read three,
  // two and one steps ahead, so that each has a whole step to arrive (a central
  // collision's refit 225 us with all of them one step ahead, 154 so)
  auto row = [&](int j) { return (int)KR[j < 0 ? 0 : j]; };
  int r = KR[i], r1 = row(i - 1), r2 = row(i - 2);
  int2 q = cl.pos[H[r]];
  int32_t c1 = H[r1];
  for (; i >= 0; --i) {
    const int2 q1 = cl.pos[c1];
    const int32_t c2 = H[r2];
    const int r3 = row(i - 3);
    if (r != r_state) {
      HJac<T> J;
      if (!helix_step(p, row_dx<T>(P, r_state, r), pv, pv.refit_snp_max(), lp, &J)) return 1;
      ud_propagate(c, J);
    }
    const T my = (T)q.x * (T)FX_SCALE;
    const T mz = (T)(q.y - anchor) * (T)FX_SCALE;
    T x2;
    if (!ud_measure(p, c, lp, my, mz, pv.vy(r), pv.vz(r), &x2)) return 1;
    chi2s += x2;
    if (!ud_pd(c)) pd = false;
    r_state = r;
    r = r1;
    r1 = r2;
    r2 = r3;
    c1 = c2;
    q = q1;
  }
  return 0;
}

// Start of the refit: the circle through the innermost, middle and outermost
// kept clusters, evaluated at the outermost one (fixed-point differences are
// exact integers), and the broad refit prior as UD factors (U = I).  Returns
// the outermost kept row, or -1 if the track has fewer than 3 kept hits.
template <typename T>
__device__ int refit_seed(uint32_t t, const ClusterView& cl, int32_t anchor, const FollowOut& fo,
                          int n, const DevParams* P, T p[5], UDCov<T>& c) {
  const PV<T> pv{P};
  if (n < 3) return -1;
  const int32_t* H = fo.hits + (size_t)t * NROW;
  const uint8_t* KR = fo.krow + (size_t)t * NROW;
  const int im = (n + 1) / 2 - 1;  // middle, counted from the innermost
  const int rA = KR[0], rM = KR[im], rE = KR[n - 1];
  const int32_t cA = H[rA], cM = H[rM], cE = H[rE];
  const int2 qA = cl.pos[cA], qM = cl.pos[cM], qE = cl.pos[cE];
  const int64_t dxm = P->xfx[rM] - P->xfx[rA], dym = (int64_t)qM.x - qA.x;
  const int64_t dxe = P->xfx[rE] - P->xfx[rA], dye = (int64_t)qE.x - qA.x;
  const int64_t dxx = P->xfx[rE] - P->xfx[rM], dyy = (int64_t)qE.x - qM.x;
  const T S = (T)FX_SCALE;
  const T cross = (T)(dxm * dye - dym * dxe) * S * S;
  const T dma = hypot((T)dxm, (T)dym) * S, dea = hypot((T)dxe, (T)dye) * S;
  const T dem = hypot((T)dxx, (T)dyy) * S;
  const T b = pv.b();
  T C = (T)2 * cross / (dma * dem * dea);
  T qpt = -C / b;
  qpt = fmin(fmax(qpt, -pv.qpt_clamp()), pv.qpt_clamp());
  C = -b * qpt;
  const T sarg = fmin(fmax(dea * C * (T)0.5, (T)-1), (T)1);
  const T h = dea * fabs(C) * (T)0.5;
  const T arc = h > (T)0 ? dea * asin(fmin(h, (T)1)) / h : dea;
  p[0] = (T)qE.x * S;
  p[1] = (T)(qE.y - anchor) * S;
  p[2] = sin(atan2((T)dye, (T)dxe) + asin(sarg));  // tangent at the far end of the chord
  p[3] = (T)(qE.y - qA.y) * S / arc;
  p[4] = qpt;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
#pragma unroll
    for (int j = 0; j < 5; ++j) c.u[i][j] = 0;
    c.d[i] = pv.c0r(i);
  }
  return rE;
}

// The refit of each kept track, tracks taken in the order perm gives (sorted
// by kept hits): in FP32 from the circle seed, with y and sin phi carried
// with their rounding errors.  A low-pT track (|q/pT| >= lowpt_qpt at the
// seed) whose FP32 covariance loses positive definiteness is refit again in
// FP64 from its seed by the same lane (TF_TO_FP64 marks it; the mark is
// internal, the count an atomic per wave); force_fallback sends every track
// there (a test hook).
__global__ __launch_bounds__(64) void k_refit(ClusterView cl, const uint32_t* __restrict__ tl_start,
                                              FollowOut fo, const uint32_t* n_tl_dev,
                                              uint32_t tl_cap, const uint16_t* __restrict__ nkept,
                                              const uint32_t* __restrict__ perm, uint32_t ngrp,
                                              RefitOut ro,
                                              const DevParams* __restrict__ Pg, DevStatus* st) {
  if (failed(st)) return;
  __shared__ DevParams Ps;
  const DevParams* P = params_to_lds(Pg, &Ps);
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  uint32_t j0, j1, dj;
  sorted_items(ngrp, n_tl, j0, j1, dj);
  for (uint32_t j = j0; j < j1; j += dj) {
    const uint32_t t = perm[j];
    ro.flags[t] = 0;
    const int n = nkept[t];
    if (n == 0) continue;
    const int32_t anchor = tl_anchor(cl, tl_start, t);
    if (!P->force_fallback) {
      float p[5];
      UDCov<float> c;
      int rs = refit_seed<float>(t, cl, anchor, fo, n, P, p, c);
      const bool lowpt = rs >= 0 && fabsf(p[4]) >= (float)P->lowpt_qpt;
      int r = n - 1;
      bool pd = true;
      float chi2s = 0.0f;
      LoParts<float> lo{0.0f, 0.0f};
      if (rs < 0 || refit_run<float>(t, cl, anchor, fo, P, p, c, chi2s, rs, r, pd, &lo)) {
        ro.flags[t] = TF_REFIT_FAIL;
        atomicAdd(&st->n_refit_fail, 1u);
        continue;
      }
      if (pd || !lowpt) {
        p[0] += lo.y;
        p[2] += lo.s;
        float cv[15];
        ud_to_cov(c, cv);
#pragma unroll
        for (int i = 0; i < 5; ++i) ro.par[(size_t)t * 5 + i] = p[i];
#pragma unroll
        for (int i = 0; i < 15; ++i) ro.cov[(size_t)t * 15 + i] = cv[i];
        ro.chi2[t] = chi2s;
        ro.row[t] = (uint8_t)rs;
        if (!pd) {
          ro.flags[t] = TF_NOT_PD;
          atomicAdd(&st->n_not_pd, 1u);
        }
        continue;
      }
    }
    // the whole refit again in FP64 (an FP32 result is discarded), counted for
    // the status: one atomic for the lanes that get here together
    const uint64_t redo = __ballot(true);
    if ((threadIdx.x & 63) == (uint32_t)__builtin_ctzll(redo))
      atomicAdd(&st->n_fp64_redo, (uint32_t)__popcll(redo));
    double p[5];
    UDCov<double> c;
    double c2 = 0;
    int rs = refit_seed<double>(t, cl, anchor, fo, n, P, p, c);
    int r = n - 1;
    bool pd = true;
    const bool fail = rs < 0 || refit_run<double>(t, cl, anchor, fo, P, p, c, c2, rs, r, pd,
                                                  (LoParts<double>*)nullptr) != 0;
    if (fail || !pd) {
      ro.flags[t] = TF_TO_FP64 | (fail ? TF_REFIT_FAIL : TF_FP64_FAIL);
      atomicAdd(fail ? &st->n_refit_fail : &st->n_fallback_fail, 1u);
      continue;
    }
    double cv[15];
    ud_to_cov(c, cv);
#pragma unroll
    for (int i = 0; i < 5; ++i) ro.par[(size_t)t * 5 + i] = (float)p[i];
#pragma unroll
    for (int i = 0; i < 15; ++i) ro.cov[(size_t)t * 15 + i] = (float)cv[i];
    ro.chi2[t] = (float)c2;
    ro.row[t] = (uint8_t)rs;
    ro.flags[t] = TF_TO_FP64 | TF_FP64;
  }
}

// final keep flag of a tracklet slot
__device__ __forceinline__ bool final_kept(const uint16_t* nkept, const RefitOut& ro, uint32_t t) {
  return nkept[t] != 0 && (ro.flags[t] & (TF_REFIT_FAIL | TF_FP64_FAIL)) == 0;
}

struct GetTrackPair {
  const uint16_t* nkept;
  RefitOut ro;
  __device__ unsigned long long operator()(uint32_t t) const {
    return final_kept(nkept, ro, t) ? ((1ull << 32) | nkept[t]) : 0ull;
  }
};

struct EmitTrackPair {
  uint32_t* trk_index;  // [cap] track index or 0xFFFFFFFF
  uint32_t* hit_off;    // [cap]
  uint32_t* tlist;      // [cap] tracklet of each track
  uint32_t cap;
  __device__ void operator()(uint32_t t, unsigned long long pre, unsigned long long v) const {
    const uint32_t j = (uint32_t)(pre >> 32);
    trk_index[t] = v ? j : 0xFFFFFFFFu;
    hit_off[t] = (uint32_t)pre;
    if (v && j < cap) tlist[j] = t;
  }
};

struct TrackOut {
  uint32_t capacity, hit_capacity;
  uint32_t* tracklet;
  float *par, *cov, *chi2;
  uint16_t* ndf;
  uint8_t *row, *flags;
  int32_t* z_anchor;
  uint32_t* hit_start;
  uint32_t* hits;
  int32_t* cluster_track;
};

struct FinTracks {
  TrackOut to;
  uint32_t *n_tracks, *n_hits;
  DevStatus* st;
  __device__ void operator()(unsigned long long v) const {
    const uint32_t nt = (uint32_t)(v >> 32), nh = (uint32_t)v;
    st->n_tracks = nt;
    st->n_hits = nh;
    st->n_fallback = st->n_fp64_redo;
    if (n_tracks) *n_tracks = nt;
    if (n_hits) *n_hits = nh;
    if (nt > to.capacity) latch_capacity(st, OVF_TRACKS, nt);
    if (nh > to.hit_capacity) latch_capacity(st, OVF_HITS, nh);
    if (nt <= to.capacity) to.hit_start[nt] = nh;
  }
};

// A wave per run of consecutive tracks (the tracklets that became tracks,
// listed in order; up to 64, fewer where that gives every wave of the nw some),
// so that every output array is written in contiguous runs: lane i writes the
// fields of track j0 + i, the wave writes the parameters and covariances of its
// tracks as one run each, then the kept hits of all its tracks (one output run,
// in track order, each track's hits in ascending row order), lane e taking
// element e of the run: its track is the last one whose first hit is at or
// before e.  Bound by its chains of dependent loads: on a central collision 47 us
// with 64 tracks per wave, 10 spread (with the clusters' outputs, 51 before).
#define EMIT_MIN 4      // tracks per wave at least
#define EMIT_TRACKS 32  // tracklets per wave of the grid
__device__ __forceinline__ void track_emit(
    ClusterView cl, const uint32_t* __restrict__ tl_start, FollowOut fo,
    const uint32_t* __restrict__ tlist, const uint16_t* __restrict__ nkept, RefitOut ro,
    const uint32_t* __restrict__ hit_off, const TrackOut& to, uint32_t n_trk, uint32_t nw) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t per = min(64u, max((uint32_t)EMIT_MIN, (n_trk + nw - 1) / nw));
  for (uint32_t w = uni(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); w * per < n_trk;
       w += nw) {
    const uint32_t j0 = w * per, m = min(per, n_trk - j0);
    const uint32_t j = j0 + lane;
    uint32_t t = 0, o = 0, n = 0;
    if (lane < m) {
      t = tlist[j];
      o = hit_off[t];
      n = nkept[t];
      to.tracklet[j] = t;
      to.chi2[j] = ro.chi2[t];
      to.ndf[j] = (uint16_t)(2 * n - 5);
      to.row[j] = ro.row[t];
      to.flags[j] = ro.flags[t] & ~TF_TO_FP64;
      to.z_anchor[j] = cl.z_fx[tl_start[t]];
      to.hit_start[j] = o;
    }
    // every lane takes part in each shuffle (the loops are uniform)
    for (uint32_t e0 = 0; e0 < m * 5; e0 += 64) {
      const uint32_t e = e0 + lane, k = min(e / 5, 63u);
      const uint32_t tk = (uint32_t)__shfl((int)t, (int)k);
      if (e < m * 5) to.par[(size_t)j0 * 5 + e] = ro.par[(size_t)tk * 5 + (e - k * 5)];
    }
    for (uint32_t e0 = 0; e0 < m * 15; e0 += 64) {
      const uint32_t e = e0 + lane, k = min(e / 15, 63u);
      const uint32_t tk = (uint32_t)__shfl((int)t, (int)k);
      if (e < m * 15) to.cov[(size_t)j0 * 15 + e] = ro.cov[(size_t)tk * 15 + (e - k * 15)];
    }
    // the wave's hits: offsets relative to its first track's (lanes past the
    // last track hold the end, so no element maps to them)
    const uint32_t o0 = uni((uint32_t)__shfl((int)o, 0));
    const uint32_t last = m - 1;
    const uint32_t end = uni((uint32_t)__shfl((int)(o + n), (int)last)) - o0;
    const uint32_t rel = lane < m ? o - o0 : end;
    for (uint32_t e0 = 0; e0 < end; e0 += 64) {
      const uint32_t e = e0 + lane;
      uint32_t k = 0;
#pragma unroll
      for (uint32_t step = 32; step > 0; step >>= 1) {
        const uint32_t rk = (uint32_t)__shfl((int)rel, (int)(k + step));
        if (k + step < m && rk <= e) k += step;
      }
      const uint32_t tk = (uint32_t)__shfl((int)t, (int)k);
      const uint32_t rk = (uint32_t)__shfl((int)rel, (int)k);
      if (e < end && o0 + e < to.hit_capacity) {
        const uint32_t i = e - rk;
        to.hits[o0 + e] = (uint32_t)fo.hits[(size_t)tk * NROW + fo.krow[(size_t)tk * NROW + i]];
      }
    }
  }
}

__device__ __forceinline__ void cluster_track(const uint32_t* __restrict__ owner,
                                              const uint32_t* __restrict__ trk_index, uint32_t n,
                                              uint32_t tl_cap, int32_t* __restrict__ out,
                                              uint32_t first, uint32_t stride) {
  for (uint32_t c = first; c < n; c += stride) {
    const uint32_t key = owner[c];
    int32_t v = -1;
    if (key) {
      const uint32_t t = 0xFFFFFFu - (key & 0xFFFFFFu);
      if (t < tl_cap) {
        const uint32_t j = trk_index[t];
        if (j != 0xFFFFFFFFu) v = (int32_t)j;
      }
    }
    out[c] = v;
  }
}

// The tracks' outputs by the first nwg workgroups, the clusters' by the others.
__global__ __launch_bounds__(256) void k_track_output(
    ClusterView cl, const uint32_t* __restrict__ tl_start, FollowOut fo,
    const uint32_t* __restrict__ tlist, const uint16_t* __restrict__ nkept, RefitOut ro,
    const uint32_t* __restrict__ hit_off, TrackOut to, uint32_t nwg,
    const uint32_t* __restrict__ owner, const uint32_t* __restrict__ trk_index, uint32_t tl_cap,
    const DevStatus* st) {
  if (failed(st)) return;
  if (blockIdx.x < nwg)
    track_emit(cl, tl_start, fo, tlist, nkept, ro, hit_off, to, min(st->n_tracks, to.capacity),
               nwg * (blockDim.x >> 6));
  else
    cluster_track(owner, trk_index, scan_count(cl.n_clusters, cl.capacity), tl_cap,
                  to.cluster_track, (blockIdx.x - nwg) * blockDim.x + threadIdx.x,
                  (gridDim.x - nwg) * blockDim.x);
}

// Per-tracklet following result as full rows (debug output).
__global__ void k_follow_export(FollowOut fo, const uint32_t* n_tl_dev, uint32_t tl_cap,
                                int32_t* __restrict__ out, const DevStatus* st) {
  if (failed(st)) return;
  const uint32_t n_tl = scan_count(n_tl_dev, tl_cap);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_tl * NROW;
       i += gridDim.x * blockDim.x) {
    const uint32_t t = i / NROW;
    const int r = i % NROW;
    const int lo = fo.range[t] & 255, hi = fo.range[t] >> 8;
    out[i] = (fo.ok[t] && r >= lo && r <= hi) ? fo.hits[i] : -1;
  }
}
