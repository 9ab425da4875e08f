// Wavefront helpers shared by the device sources.
#pragma once

#include "tfg_internal.h"

namespace tfg {

// A value the compiler cannot prove wave-uniform, made scalar.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Inclusive scan over the wavefront (all lanes active) with DPP moves: shifts
// inside each row of 16 lanes, then the row totals carried to the rows after.
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15, rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31, rows 2 and 3
  return v;
}

// Exclusive scan of one value per thread over a block of NW waves.
template <int NW>
__device__ __forceinline__ int block_excl_scan(int v, int* tmp, int* total) {
  const int wave = threadIdx.x / kWave;
  int incl = wave_incl_scan(v);
  if (lane_id() == kWave - 1) tmp[wave] = incl;
  __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    int t = tmp[w];
    if (w < wave) off += t;
    tot += t;
  }
  __syncthreads();
  if (total) *total = tot;
  return off + incl - v;
}

// K exclusive scans at once (one value per list per thread) over a block of
// NW <= 64 waves: the lists share the barriers (three in all), and one wave per
// list scans its wave totals. tmp: (NW + 1) * K ints.
template <int NW, int K>
__device__ __forceinline__ void block_excl_scan_lists(const int (&v)[K], int (&ex)[K],
                                                      int (&total)[K], int* tmp) {
  const int wave = threadIdx.x / kWave;
  int incl[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    incl[i] = wave_incl_scan(v[i]);
    if (lane_id() == kWave - 1) tmp[i * NW + wave] = incl[i];
  }
  __syncthreads();
  for (int i = wave; i < K; i += NW) {  // uniform per wave
    const int t = lane_id() < NW ? tmp[i * NW + lane_id()] : 0;
    const int s = wave_incl_scan(t);
    if (lane_id() < NW) tmp[i * NW + lane_id()] = s - t;
    if (lane_id() == NW - 1) tmp[K * NW + i] = s;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < K; ++i) {
    ex[i] = tmp[i * NW + wave] + incl[i] - v[i];
    total[i] = tmp[K * NW + i];
  }
  __syncthreads();  // tmp may be written again
}

}  // namespace tfg
