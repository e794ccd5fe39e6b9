// Causal attention by input type (bf16: attn_mfma.hip, fp32: attn_fp32.hip), and the small kernels around it: row sums
// dO . O, casts of the gradient accumulators, fills.
#include "common.h"

namespace {


template <typename T, int D>
__global__ void __launch_bounds__(256) k_delta(const T* __restrict__ O, const T* __restrict__ dO,
                                                float* __restrict__ delta, size_t rows) {
  size_t row = (size_t)blockIdx.x * 4 + threadIdx.x / 64;
  if (row >= rows) return;
  int lane = threadIdx.x % 64;
  float s = 0.f;
  for (int d = lane; d < D; d += 64) s += Elem<T>::ld(O, row * D + d) * Elem<T>::ld(dO, row * D + d);
  s = wave_sum(s);
  if (lane == 0) delta[row] = s;
}

template <typename T>
__global__ void k_cast(const float* __restrict__ src, T* __restrict__ dst, size_t n, float mul) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) Elem<T>::st(dst, i, src[i] * mul);
}

__global__ void k_fill_i32(int32_t* __restrict__ dst, size_t n, int32_t v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) dst[i] = v;
}

__global__ void k_fill(float* __restrict__ dst, size_t n, float v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) dst[i] = v;
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
  size_t rows = (size_t)d.B * d.Hq * d.N;
  dim3 g((unsigned)((rows + 3) / 4));
  if (d.dtype == MUSE_DTYPE_BF16) {
    if (d.D == 64) { MuseProf prof_("k_delta", st); hipLaunchKernelGGL((k_delta<bf16_t, 64>), g, dim3(256), 0, st, (const bf16_t*)O, (const bf16_t*)dO, delta, rows); }
    else { MuseProf prof_("k_delta", st); hipLaunchKernelGGL((k_delta<bf16_t, 128>), g, dim3(256), 0, st, (const bf16_t*)O, (const bf16_t*)dO, delta, rows); }
  } else {
    if (d.D == 64) { MuseProf prof_("k_delta", st); hipLaunchKernelGGL((k_delta<float, 64>), g, dim3(256), 0, st, (const float*)O, (const float*)dO, delta, rows); }
    else { MuseProf prof_("k_delta", st); hipLaunchKernelGGL((k_delta<float, 128>), g, dim3(256), 0, st, (const float*)O, (const float*)dO, delta, rows); }
  }
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

int muse_launch_cast(const float* src, void* dst, size_t n, int dst_dtype, float mul, hipStream_t st) {
  unsigned blocks = (unsigned)((n + 1023) / 1024 > 65535 * 16 ? 65535 * 16 : (n + 1023) / 1024);
  if (blocks == 0) return MUSE_OK;
  if (dst_dtype == MUSE_DTYPE_BF16) { MuseProf prof_("k_cast", st); hipLaunchKernelGGL(k_cast<bf16_t>, dim3(blocks), dim3(256), 0, st, src, (bf16_t*)dst, n, mul); }
  else { MuseProf prof_("k_cast", st); hipLaunchKernelGGL(k_cast<float>, dim3(blocks), dim3(256), 0, st, src, (float*)dst, n, mul); }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_fill(float* dst, size_t n, float v, hipStream_t st) {
  unsigned blocks = (unsigned)((n + 1023) / 1024 > 65535 * 16 ? 65535 * 16 : (n + 1023) / 1024);
  if (blocks == 0) return MUSE_OK;
  { MuseProf prof_("k_fill", st); hipLaunchKernelGGL(k_fill, dim3(blocks), dim3(256), 0, st, dst, n, v); }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_fill_i32(int32_t* dst, size_t n, int32_t v, hipStream_t st) {
  unsigned blocks = (unsigned)((n + 1023) / 1024 > 65535 * 16 ? 65535 * 16 : (n + 1023) / 1024);
  if (blocks == 0) return MUSE_OK;
  { MuseProf prof_("k_fill_i32", st); hipLaunchKernelGGL(k_fill_i32, dim3(blocks), dim3(256), 0, st, dst, n, v); }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
