// Causal attention by input type (bf16: attn_mfma.hip, fp32: attn_fp32.hip), and the small kernels around it: row sums
// dO . O, casts of the gradient accumulators, fills.
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "common.h"

namespace {


// Bound by the rows: 16 bytes per lane, D sizeof(T) / 16 lanes per row, kDeltaRows rows of a lane requested together.  (A wave per
// row and a value per lane took 160 us at 16 heads of 64k, 57 at 32 heads of 8k with D = 128; 46 and 20 now, 22 -> 7 at 8 heads of 16k.)
// A row's sum is added up within the lane first: another order of the fp32 sums than a wave per row had (differences of a last bit,
// which flip the rounding of a bf16 dS now and then; against 64 bits both are equally far).
// O may lie anywhere (no other kernel reads it): WIDE is for 16-byte boundaries, the other form loads value by value, same sums.
constexpr int kDeltaRows = 4;
template <typename T, int D, bool WIDE>
__global__ void __launch_bounds__(256) k_delta(const T* __restrict__ O, const T* __restrict__ dO,
                                                float* __restrict__ delta, size_t rows) {
  constexpr int E = 16 / (int)sizeof(T), LPR = D / E, RPB = 256 / LPR;  // values per lane, lanes per row, rows side by side
  const int c = threadIdx.x % LPR;
  const size_t r0 = (size_t)blockIdx.x * (RPB * kDeltaRows) + threadIdx.x / LPR;
  float o[kDeltaRows][E], g[kDeltaRows][E];
#pragma unroll
  for (int u = 0; u < kDeltaRows; ++u) {
    const size_t at = min(r0 + (size_t)RPB * u, rows - 1) * D + E * c;
#pragma unroll
    for (int e = 0; e < E; e += 4) {
      if constexpr (WIDE) {
        ld4(O, at + e, &o[u][e]);
        ld4(dO, at + e, &g[u][e]);
      } else {
#pragma unroll
        for (int x = e; x < e + 4; ++x) { o[u][x] = Elem<T>::ld(O, at + x); g[u][x] = Elem<T>::ld(dO, at + x); }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kDeltaRows; ++u) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) s = fmaf(o[u][e], g[u][e], s);
    s = group_sum<(LPR < 16 ? LPR : 16)>(s);
    if (LPR == 32) s += __shfl_xor(s, 16, 64);
    const size_t row = r0 + (size_t)RPB * u;
    if (c == 0 && row < rows) delta[row] = s;
  }
}

template <typename T>
__global__ void k_cast(const float* __restrict__ src, T* __restrict__ dst, size_t n, float mul) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) Elem<T>::st(dst, i, src[i] * mul);
}
// The same for bf16 results at a 16-byte boundary, eight values per lane, several tensors in one launch: 85 -> 52 us for the three
// gradients of 32 heads of 8k, D = 128.  Results anywhere else keep the kernel above.
__global__ void __launch_bounds__(256) k_cast8(CastRanges c, float mul) {
  const size_t first = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  for (int r = 0; r < c.n; ++r) {
    const float4* src = reinterpret_cast<const float4*>(c.r[r].src);
    uint4* dst = reinterpret_cast<uint4*>(c.r[r].dst);
    for (size_t i = first; i < c.r[r].n / 8; i += stride) {
      const float4 a = src[2 * i], b = src[2 * i + 1];
      dst[i] = make_uint4(pack_bf16x2(a.x * mul, a.y * mul), pack_bf16x2(a.z * mul, a.w * mul), pack_bf16x2(b.x * mul, b.y * mul),
                          pack_bf16x2(b.z * mul, b.w * mul));
    }
  }
}

// Several arrays of 32-bit words, each with a value of its own, in one launch (a small call pays 5 us for every launch); 16
// bytes per lane where an array begins on such a boundary.
__global__ void __launch_bounds__(256) k_fill(FillRanges f) {
  const size_t first = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  for (int r = 0; r < f.n; ++r) {
    uint32_t* p = reinterpret_cast<uint32_t*>(f.r[r].p);
    const uint32_t v = f.r[r].v;
    const size_t n4 = ((uintptr_t)p & 15) == 0 ? f.r[r].n / 4 : 0;
    for (size_t i = first; i < n4; i += stride) reinterpret_cast<uint4*>(p)[i] = make_uint4(v, v, v, v);
    for (size_t i = 4 * n4 + first; i < f.r[r].n; i += stride) p[i] = v;
  }
}

}  // namespace

// implemented in attn_fp32.hip
int muse_launch_attn_fwd_f32(const MuseDims& d, int Bs, const float* Q, const float* K, const float* V, const float* ff,
                             float* O, float* LSE, hipStream_t st);
int muse_launch_attn_bwd_f32(const MuseDims& d, int Bs, const float* Q, const float* K, const float* V, const float* dO,
                             const float* LSE, const float* delta, float* dQ, float* dK, float* dV, hipStream_t st);

// implemented in attn_mfma.hip
int muse_launch_attn_fwd_mfma(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V,
                              const float* ff, void* O, float* LSE, hipStream_t st);
int muse_launch_attn_bwd_mfma(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V,
                              const void* dO, const float* LSE, const float* delta, float* dQacc,
                              float* dKacc, float* dVacc, hipStream_t st);

int muse_launch_attn_fwd(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V,
                         const float* ff, void* O, float* LSE, hipStream_t st) {
  if (d.dtype == MUSE_DTYPE_BF16) return muse_launch_attn_fwd_mfma(d, Bs, Q, K, V, ff, O, LSE, st);
  return muse_launch_attn_fwd_f32(d, Bs, (const float*)Q, (const float*)K, (const float*)V, ff, (float*)O, LSE, st);
}

int muse_launch_delta(const MuseDims& d, const void* O, const void* dO, float* delta, hipStream_t st) {
  const size_t rows = (size_t)d.B * d.Hq * d.N;
  MuseProf prof_("k_delta", st);
  auto go = [&](auto* kernel, auto* o, auto* g) {
    const size_t per = 256 * kDeltaRows * 16 / (d.D * sizeof(*o));  // rows of a workgroup
    hipLaunchKernelGGL(kernel, dim3((unsigned)((rows + per - 1) / per)), dim3(256), 0, st, o, g, delta, rows);
  };
  const bool wide = ((uintptr_t)O | (uintptr_t)dO) % 16 == 0;
  auto of = [&](auto* o, auto* g) {
    using T = std::remove_cv_t<std::remove_pointer_t<decltype(o)>>;
    if (d.D == 64) wide ? go(k_delta<T, 64, true>, o, g) : go(k_delta<T, 64, false>, o, g);
    else wide ? go(k_delta<T, 128, true>, o, g) : go(k_delta<T, 128, false>, o, g);
  };
  if (d.dtype == MUSE_DTYPE_BF16) of((const bf16_t*)O, (const bf16_t*)dO);
  else of((const float*)O, (const float*)dO);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_attn_bwd(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V,
                         const void* dO, const float* LSE, const float* delta, float* dQacc,
                         float* dKacc, float* dVacc, hipStream_t st) {
  if (d.dtype == MUSE_DTYPE_BF16)
    return muse_launch_attn_bwd_mfma(d, Bs, Q, K, V, dO, LSE, delta, dQacc, dKacc, dVacc, st);
  return muse_launch_attn_bwd_f32(d, Bs, (const float*)Q, (const float*)K, (const float*)V, (const float*)dO, LSE, delta,
                                  dQacc, dKacc, dVacc, st);
}

int muse_launch_casts(const CastRanges& c, int dst_dtype, float mul, hipStream_t st) {
  CastRanges wide;
  size_t most = 0;
  for (int r = 0; r < c.n; ++r) {
    const float* src = c.r[r].src;
    void* dst = c.r[r].dst;
    const size_t n = c.r[r].n, blocks = std::min<size_t>((n + 1023) / 1024, 65535 * 16);
    if (n == 0) continue;
    if (dst_dtype == MUSE_DTYPE_BF16 && (((uintptr_t)src | (uintptr_t)dst) & 15) == 0 && n % 8 == 0) {
      wide.add(src, dst, n);
      most = std::max(most, n);
      continue;
    }
    MuseProf prof_("k_cast", st);
    if (dst_dtype == MUSE_DTYPE_BF16) hipLaunchKernelGGL(k_cast<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, st, src, (bf16_t*)dst, n, mul);
    else hipLaunchKernelGGL(k_cast<float>, dim3((unsigned)blocks), dim3(256), 0, st, src, (float*)dst, n, mul);
  }
  if (most > 0) {
    MuseProf prof_("k_cast", st);
    hipLaunchKernelGGL(k_cast8, dim3((unsigned)std::min<size_t>((most / 8 + 255) / 256, 1 << 20)), dim3(256), 0, st, wide, mul);
  }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_fills(const FillRanges& f, hipStream_t st) {
  size_t most = 0;
  for (int r = 0; r < f.n; ++r) most = std::max(most, f.r[r].n);
  if (most == 0) return MUSE_OK;
  {
    MuseProf prof_("k_fill", st);
    hipLaunchKernelGGL(k_fill, dim3((unsigned)std::min<size_t>((most + 1023) / 1024, 1 << 20)), dim3(256), 0, st, f);
  }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
