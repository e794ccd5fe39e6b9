// Dot products on v_mfma_f32_16x16x4_f32 whose rounding is that of short sums.  One accumulator for all D products rounds
// each against the whole sum so far, which at D = 128 doubles or triples the error of a score against 64 bits; here four
// accumulators take 16 products each and are added up every 64 dims (3 to 6 % of the attention kernels' time; one accumulator
// added up every 16 dims took 8 to 13 %, as its instructions wait for one another).
#pragma once
#include "common.h"

struct FoldSum {
  f32x4_t part[4], total;
  __device__ __forceinline__ FoldSum() : total{0.f, 0.f, 0.f, 0.f} { clear(); }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int t = 0; t < 4; ++t) part[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void add(int t, float a, float b) { part[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, part[t], 0, 0, 0); }
  // behind the four instructions of the u-th 16 dims
  __device__ __forceinline__ void fold(int u) {
    if (u % 4 != 3) return;
    total += (part[0] + part[1]) + (part[2] + part[3]);
    clear();
  }
};
