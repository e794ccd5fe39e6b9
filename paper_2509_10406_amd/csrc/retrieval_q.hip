// Exact retrieval (Sec. 3.3) on the query side for bf16 inputs: per (query, slot) the partial softmax state over the keys
// of the retrieved pair (forward), and the partial query gradient (backward).
#include "ff_common.h"
#include "lds_tile.h"

namespace {

// Both kernels: a workgroup of kRunTiles waves per work item, a run of up to kRunTiles tiles of 32 hits of one retrieved
// pair; a wave's hits are the MFMA columns (rows read straight from Q and dO), the pair's keys the rows.
//   hit = n | g << 22, slot * k2e + u  (query position and head inside the KV group; where the result goes)
// The keys and values are staged once for all four tiles, row-major, 64 at a time, and serve both operand forms
// (lds_tile.h); a heavy pair is many items, a light one a single item, so nothing waits for a long one.
// Bound by the scattered rows: a hit is one row of Q (and dO) and one result row of 4 D bytes.
// One wave per item, which staged a pair of more than 32 keys anew for every tile (transposed, in 2-byte stores) and wrote
// 32 bytes of 32 rows per instruction, took (forward / backward) 1.47 / 2.14 ms at 16 heads of 64k tokens with 128 x 128
// clusters, now 0.79 / 0.87; 0.89 / 1.04 with 256 x 1024, now 0.71 / 0.83; 3.02 / 3.14 at 32 heads of 32k with D = 128, now
// 2.15 / 2.71 (7.5 GB of result rows each).  Streaming stores need the rows whole lines: with (max, sum) behind each row
// instead of in an array of their own they took 1.24 against 0.71 ms.
constexpr int kKeys = 64;  // keys staged at a time

struct PairItem {
  int klo, khi, h0, hhi;  // bucketed key range of the pair; first hit of the wave's tile, end of the item's hits
  size_t hqbase;          // first query head of the KV group
};

// keys k0 .. of X into LDS (the pair's last key again past its end, up to a whole tile of 32)
template <int D>
__device__ __forceinline__ void stage_keys(const bf16_t* __restrict__ Ks, const bf16_t* __restrict__ Vs, size_t base, int k0, int khi,
                                           bf16_t* ks, bf16_t* vs) {
  constexpr int CPR = D / 8, RPI = 256 / CPR, NI = kKeys / RPI;
  const int r0 = threadIdx.x / CPR, cc = threadIdx.x % CPR, need = (min(khi - k0, kKeys) + 31) / 32 * 32;
  uint4 a[NI], b[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const size_t at = (base + min(k0 + r0 + RPI * i, khi - 1)) * D + 8 * cc;
    if (RPI * i < need) {
      a[i] = *reinterpret_cast<const uint4*>(Ks + at);
      b[i] = *reinterpret_cast<const uint4*>(Vs + at);
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i)
    if (RPI * i < need) {
      *reinterpret_cast<uint4*>(ks + tile_at<D>(r0 + RPI * i, cc)) = a[i];
      *reinterpret_cast<uint4*>(vs + tile_at<D>(r0 + RPI * i, cc)) = b[i];
    }
}

// The wave's 32 result rows (accumulator columns) to dst + idx * D, idx the lane's own row number: through 4 KB of LDS
// per 32 dims, so that a store instruction writes whole 128-byte lines of 8 rows and not 32 bytes of 32.
template <int D>
__device__ __forceinline__ void store_rows(const f32x16_t (&acc)[D / 32], float mul, float* lds, float* __restrict__ dst, size_t idx,
                                           int nrows, int lane) {
  const int col = lane % 32, half = lane / 32, r8 = lane / 8, c8 = lane % 8;
  float* out[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned lo = __shfl((unsigned)idx, 8 * i + r8, 64), hi = __shfl((unsigned)(idx >> 32), 8 * i + r8, 64);
    out[i] = dst + (((size_t)hi << 32) | lo) * D + 4 * c8;
  }
#pragma unroll
  for (int t = 0; t < D / 32; ++t) {
    wave_lds_fence();
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(lds + 32 * col + 4 * ((2 * g + half) ^ ((col >> 1) & 7))) =
          make_float4(mul * acc[t][4 * g], mul * acc[t][4 * g + 1], mul * acc[t][4 * g + 2], mul * acc[t][4 * g + 3]);
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 8 * i + r8;
      const float4 v = *reinterpret_cast<const float4*>(lds + 32 * row + 4 * (c8 ^ ((row >> 1) & 7)));
      const float x[4] = {v.x, v.y, v.z, v.w};
      if (row < nrows) st4_stream(out[i], 32 * t, x);  // read by a later kernel, when nothing of it is cached
    }
  }
}

__device__ __forceinline__ bool pair_item(PairItem& it, const int32_t* __restrict__ off_k, const int32_t* __restrict__ run_off,
                                          const int4* __restrict__ run_map, size_t run_cap, int nb, int Ck, int Hq, int Hkv) {
  const int hk = blockIdx.y, NBm = nb - 1, G_ = Hq / Hkv;
  if ((int)blockIdx.x >= run_off[(size_t)hk * ((size_t)NBm * Ck + 1) + (size_t)NBm * Ck]) return false;  // past the last item
  const int4 item = run_map[(size_t)hk * run_cap + blockIdx.x];  // (pair, first hit, end)
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  it.klo = ok[item.x];  // pair = b' Ck + j indexes the segment table directly
  it.khi = ok[item.x + 1];
  it.h0 = item.y + 32 * __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  it.hhi = item.z;
  it.hqbase = (size_t)(hk / Hkv) * Hq + (size_t)(hk % Hkv) * G_;
  return it.klo < it.khi;
}

//   part[(qn*R2 + su)][D] = sum_m exp(l_m - max) v_m,  part_ml[..][2] = max (natural log units), sum
template <int D>
__global__ void __launch_bounds__(64 * kRunTiles) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 3, 4))) k_ret_fwd_pairs(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ Ks, const bf16_t* __restrict__ Vs, const int32_t* __restrict__ off_k,
    const int32_t* __restrict__ run_off, const int4* __restrict__ run_map, const uint2* __restrict__ hits, float* __restrict__ part,
    float* __restrict__ part_ml,
    size_t run_cap, size_t hit_cap, int N, int nb, int Ck, int Hq, int Hkv, int R2, float scale_log2e) {
  constexpr int KS = D / 16, DT = D / 32;
  __shared__ __attribute__((aligned(16))) bf16_t ks[kKeys * D];
  __shared__ __attribute__((aligned(16))) bf16_t vs[kKeys * D];
  PairItem it;
  if (!pair_item(it, off_k, run_off, run_map, run_cap, nb, Ck, Hq, Hkv)) return;
  const int hk = blockIdx.y, lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const bool mine = it.h0 < it.hhi;
  const uint2 hit = hits[(size_t)hk * hit_cap + min(it.h0 + col, it.hhi - 1)];
  const size_t qn = (it.hqbase + (hit.x >> 22)) * N + (hit.x & 0x3fffffu);
  bf16x8_t qf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const bf16x8_t*>(Q + qn * D + 16 * s + 8 * half);
  f32x16_t o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) o[t] = zero16();
  float m = MUSE_NEG_INF, l = 0.f;
  for (int k0 = it.klo; k0 < it.khi; k0 += kKeys) {
    if (k0 > it.klo) __syncthreads();
    stage_keys<D>(Ks, Vs, (size_t)hk * N, k0, it.khi, ks, vs);
    __syncthreads();
    if (!mine) continue;
#pragma unroll 1
    for (int u = 0; u < kKeys && k0 + u < it.khi; u += 32) {
      f32x16_t s = zero16();
#pragma unroll
      for (int x = 0; x < KS; ++x) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(ks, u + col, 2 * x + half), qf[x], s, 0, 0, 0);
      if (k0 + u + 32 > it.khi) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (k0 + u + 8 * (e / 4) + 4 * half + (e % 4) >= it.khi) s[e] = MUSE_NEG_INF;
      }
      float tmax = MUSE_NEG_INF;
#pragma unroll
      for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, s[e]);
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      const float mn = fmaxf(m, tmax * scale_log2e);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);  // every tile holds at least one key, so mn is finite
      float psum = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -mn));
        psum += s[e];
      }
      l = l * alpha + psum;
      m = mn;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[t][e] *= alpha;
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        const bf16x8_t pf = pack8(s, 2 * G, 2 * G + 1);
#pragma unroll
        for (int t = 0; t < DT; ++t) o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_cols<D>(vs, u + 16 * G, t, lane), pf, o[t], 0, 0, 0);
      }
    }
  }
  l += __shfl_xor(l, 32, 64);
  if (it.h0 + col < it.hhi) {
    if (half == 0) *reinterpret_cast<float2*>(part_ml + 2 * (qn * R2 + hit.y)) = make_float2(m * 0.6931471805599453f, l);
  }
  __syncthreads();  // the staged keys are done with
  float* lds = reinterpret_cast<float*>(threadIdx.x < 128 ? ks : vs) + 1024 * ((threadIdx.x / 64) % 2);
  if (mine) store_rows<D>(o, 1.f, lds, part, qn * R2 + hit.y, it.hhi - it.h0, lane);
}

//   dqpart[(qn*R2 + su)][0..D) = scale * sum_m dl_m k_m over the keys of the pair
template <int D>
__global__ void __launch_bounds__(64 * kRunTiles) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2, 4))) k_ret_bwd_dq_pairs(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ dO, const bf16_t* __restrict__ Ks, const bf16_t* __restrict__ Vs,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ off_k,
    const int32_t* __restrict__ run_off, const int4* __restrict__ run_map, const uint2* __restrict__ hits,
    float* __restrict__ dqpart, size_t run_cap, size_t hit_cap, int N, int nb, int Ck, int Hq, int Hkv, int R2, float scale,
    float scale_log2e) {
  constexpr int KS = D / 16, DT = D / 32;
  __shared__ __attribute__((aligned(16))) bf16_t ks[kKeys * D];
  __shared__ __attribute__((aligned(16))) bf16_t vs[kKeys * D];
  PairItem it;
  if (!pair_item(it, off_k, run_off, run_map, run_cap, nb, Ck, Hq, Hkv)) return;
  const int hk = blockIdx.y, lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const bool mine = it.h0 < it.hhi;
  const uint2 hit = hits[(size_t)hk * hit_cap + min(it.h0 + col, it.hhi - 1)];
  const size_t qn = (it.hqbase + (hit.x >> 22)) * N + (hit.x & 0x3fffffu);
  bf16x8_t qf[KS], gf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    qf[s] = *reinterpret_cast<const bf16x8_t*>(Q + qn * D + 16 * s + 8 * half);
    gf[s] = *reinterpret_cast<const bf16x8_t*>(dO + qn * D + 16 * s + 8 * half);
  }
  const float lse2 = LSE[qn] * 1.4426950408889634f, dl = delta[qn];
  f32x16_t dq[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) dq[t] = zero16();
  for (int k0 = it.klo; k0 < it.khi; k0 += kKeys) {
    if (k0 > it.klo) __syncthreads();
    stage_keys<D>(Ks, Vs, (size_t)hk * N, k0, it.khi, ks, vs);
    __syncthreads();
    if (!mine) continue;
#pragma unroll 1
    for (int u = 0; u < kKeys && k0 + u < it.khi; u += 32) {
      f32x16_t s = zero16(), dp = zero16();
#pragma unroll
      for (int x = 0; x < KS; ++x) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(ks, u + col, 2 * x + half), qf[x], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(vs, u + col, 2 * x + half), gf[x], dp, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -lse2)) * (dp[e] - dl);
      if (k0 + u + 32 > it.khi) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (k0 + u + 8 * (e / 4) + 4 * half + (e % 4) >= it.khi) s[e] = 0.f;
      }
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        const bf16x8_t df = pack8(s, 2 * G, 2 * G + 1);
#pragma unroll
        for (int t = 0; t < DT; ++t) dq[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_cols<D>(ks, u + 16 * G, t, lane), df, dq[t], 0, 0, 0);
      }
    }
  }
  __syncthreads();  // the staged keys are done with
  float* lds = reinterpret_cast<float*>(threadIdx.x < 128 ? ks : vs) + 1024 * ((threadIdx.x / 64) % 2);
  if (mine) store_rows<D>(dq, scale, lds, dqpart, qn * R2 + hit.y, it.hhi - it.h0, lane);
}

}  // namespace

int muse_launch_ret_fwd_pairs(const MuseDims& d, const void* Q, const void* Ks, const void* Vs, const int32_t* off_k,
                              const int32_t* run_off, const int4* run_map, size_t run_cap, const uint2* hits,
                              size_t hit_cap, float* part, hipStream_t st) {
  // one workgroup per work item (a run of hit tiles inside one pair); the grid covers the most there can be
  const dim3 g((unsigned)run_cap, d.B * d.Hkv);
  const float sl = d.scale * 1.4426950408889634f;
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_ret_fwd_pairs", st);
    hipLaunchKernelGGL(kernel, g, dim3(64 * kRunTiles), 0, st, (const bf16_t*)Q, (const bf16_t*)Ks, (const bf16_t*)Vs, off_k, run_off,
                       run_map, hits, part, part + (size_t)d.B * d.Hq * d.N * d.r * d.k2e * d.D, run_cap, hit_cap, d.N, d.nb, d.Ck, d.Hq, d.Hkv, d.r * d.k2e, sl);
  };
  if (d.D == 64) go(k_ret_fwd_pairs<64>);
  else go(k_ret_fwd_pairs<128>);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_ret_bwd_dq_pairs(const MuseDims& d, const void* Q, const void* dO, const void* Ks, const void* Vs,
                                 const float* LSE, const float* delta, const int32_t* off_k, const int32_t* run_off,
                                 const int4* run_map, size_t run_cap, const uint2* hits, size_t hit_cap, float* dqpart,
                                 hipStream_t st) {
  const dim3 g((unsigned)run_cap, d.B * d.Hkv);
  const float sl = d.scale * 1.4426950408889634f;
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_ret_bwd_dq_pairs", st);
    hipLaunchKernelGGL(kernel, g, dim3(64 * kRunTiles), 0, st, (const bf16_t*)Q, (const bf16_t*)dO, (const bf16_t*)Ks, (const bf16_t*)Vs,
                       LSE, delta, off_k, run_off, run_map, hits, dqpart, run_cap, hit_cap, d.N, d.nb, d.Ck, d.Hq, d.Hkv, d.r * d.k2e,
                       d.scale, sl);
  };
  if (d.D == 64) go(k_ret_bwd_dq_pairs<64>);
  else go(k_ret_bwd_dq_pairs<128>);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
