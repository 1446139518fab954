// Quality-control histograms of one reconstruction: cluster total and peak
// charge, hits per track, and clusters on / off a track.  Each workgroup
// fills its own histograms in LDS (LDS atomics only), writes them out whole,
// and a second kernel sums the workgroups' histograms bin by bin, so no
// device-scope atomic is involved.
#pragma once

#include "common.hpp"

#define QC_QTOT 0      // 256 bins: min(qtot >> 3, 255)
#define QC_QMAX 256    // 256 bins: min(qmax >> 2, 255)
#define QC_NHITS 512   // 153 bins: hits per track, 0..152
#define QC_ATTACH 665  // 2 bins: cluster not on a track / on a track
#define QC_BINS 667
#define QC_WG 1024     // workgroups of the fill kernel (4 per CU)

__global__ __launch_bounds__(256) void k_qc_fill(const uint16_t* __restrict__ qtot,
                                                 const uint16_t* __restrict__ qmax,
                                                 const int32_t* __restrict__ cluster_track,
                                                 const uint32_t* n_cl_dev, uint32_t cl_cap,
                                                 const uint32_t* __restrict__ hit_start,
                                                 const uint32_t* n_trk_dev, uint32_t trk_cap,
                                                 uint32_t* __restrict__ part, const DevStatus* st) {
  // one histogram per wave (fewer lanes contend for a hot bin); the two
  // on/off-track bins are counted in registers and added once per wave
  __shared__ uint32_t h[4][QC_BINS];
  const uint32_t w = threadIdx.x >> 6;
  for (uint32_t i = threadIdx.x; i < 4 * QC_BINS; i += blockDim.x) (&h[0][0])[i] = 0;
  __syncthreads();
  // after a latched error the outputs are not valid: empty histograms (no
  // status word, st == nullptr: the caller vouches for the outputs)
  const bool ok = st == nullptr || !failed(st);
  const uint32_t n_cl = ok ? scan_count(n_cl_dev, cl_cap) : 0u;
  const uint32_t n_trk = ok ? scan_count(n_trk_dev, trk_cap) : 0u;
  const uint32_t stride = gridDim.x * blockDim.x;
  uint32_t on = 0, off = 0;
  auto count = [&](uint32_t qt, uint32_t qm, int32_t ct) {
    atomicAdd(&h[w][QC_QTOT + min(qt >> 3, 255u)], 1u);
    atomicAdd(&h[w][QC_QMAX + min(qm >> 2, 255u)], 1u);
    if (ct >= 0) ++on;
    else ++off;
  };
  // eight clusters per thread and step in four 16-byte loads, where the arrays
  // allow them (the caller may pass views).  Bound by the bytes in flight: on
  // 1.7e7 clusters (1.4e8 bytes) from HBM the call took 99 us with a cluster per
  // thread and step, 41 us with eight (512 or 2048 workgroups: 40 and 44)
  uint32_t done = 0;
  if ((((uintptr_t)qtot | (uintptr_t)qmax | (uintptr_t)cluster_track) & 15) == 0) {
    const uint4* qt8 = reinterpret_cast<const uint4*>(qtot);
    const uint4* qm8 = reinterpret_cast<const uint4*>(qmax);
    const int4* ct4 = reinterpret_cast<const int4*>(cluster_track);
    const uint32_t n8 = n_cl / 8;
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < n8; g += stride) {
      const uint4 a = qt8[g], b = qm8[g];
      const int4 c0 = ct4[2 * (size_t)g], c1 = ct4[2 * (size_t)g + 1];
      count(a.x & 0xFFFFu, b.x & 0xFFFFu, c0.x);
      count(a.x >> 16, b.x >> 16, c0.y);
      count(a.y & 0xFFFFu, b.y & 0xFFFFu, c0.z);
      count(a.y >> 16, b.y >> 16, c0.w);
      count(a.z & 0xFFFFu, b.z & 0xFFFFu, c1.x);
      count(a.z >> 16, b.z >> 16, c1.y);
      count(a.w & 0xFFFFu, b.w & 0xFFFFu, c1.z);
      count(a.w >> 16, b.w >> 16, c1.w);
    }
    done = n8 * 8;
  }
  for (uint32_t c = done + blockIdx.x * blockDim.x + threadIdx.x; c < n_cl; c += stride)
    count(qtot[c], qmax[c], cluster_track[c]);
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n_trk; j += stride) {
    const uint32_t n = hit_start[j + 1] - hit_start[j];
    atomicAdd(&h[w][QC_NHITS + min(n, (uint32_t)NROW)], 1u);
  }
  const unsigned long long son = wave_sum_u64(on), soff = wave_sum_u64(off);
  if ((threadIdx.x & 63) == 0) {
    h[w][QC_ATTACH] += (uint32_t)soff;
    h[w][QC_ATTACH + 1] += (uint32_t)son;
  }
  __syncthreads();
  uint32_t* mine = part + (size_t)blockIdx.x * QC_BINS;
  for (uint32_t i = threadIdx.x; i < QC_BINS; i += blockDim.x)
    mine[i] = h[0][i] + h[1][i] + h[2][i] + h[3][i];
}

// hist[i] = sum over the nwg workgroup histograms of bin i: one workgroup
// per bin, its threads taking every 256th workgroup histogram
__global__ __launch_bounds__(256) void k_qc_sum(const uint32_t* __restrict__ part, uint32_t nwg,
                                                uint32_t* __restrict__ hist) {
  __shared__ unsigned long long ws[4];
  const uint32_t i = blockIdx.x;
  uint32_t s = 0;
  for (uint32_t w = threadIdx.x; w < nwg; w += blockDim.x) s += part[(size_t)w * QC_BINS + i];
  const unsigned long long t = wave_sum_u64(s);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) hist[i] = (uint32_t)(ws[0] + ws[1] + ws[2] + ws[3]);
}
