// Retrieval backward for fp32 inputs (Sec. 3.3 "Exact retrieval", gradient w.r.t. keys and values) on fp32 MFMA: one wave
// per (retrieved pair, hit slice) item of the inverse index, as the bf16 kernel k_c3_pairs; the pair is a dense
// attention-backward block, 16 queries that retrieved it against 16 of its keys at a time (v_mfma_f32_16x16x4_f32:
// operand lanes hold four consecutive dims of a row, accumulator element t of lane l is row 4 (l / 16) + t, column l % 16).
//
// Bound by the latency of the gathered query rows.  A wave per (key block, 32 key clusters) that walked a bit matrix of
// the selections, as this was before, had a hundred waves at work: 5.1 -> 0.065 ms at 4 heads of 8k tokens with 128 key
// clusters and r = 4, 9.6 -> 0.16 ms at 4 heads of 4.7k with 12 key clusters.
#include "ff_common.h"

namespace {

template <int D>
__global__ void __launch_bounds__(64) k_c3_pairs_f32(
    const float* __restrict__ Q, const float* __restrict__ dO, const float* __restrict__ Ks, const float* __restrict__ Vs,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ off_k,
    const int32_t* __restrict__ pair_off, const int32_t* __restrict__ c3_off, const int2* __restrict__ c3_map,
    const uint2* __restrict__ hits, float* __restrict__ dKs, float* __restrict__ dVs, float* __restrict__ part,
    size_t run_cap, size_t hit_cap, int N, int nb, int Ck, int Hq, int Hkv, int HK, int tps, float scale) {
  constexpr int MT = D / 16;
  __shared__ __attribute__((aligned(16))) float qrow[16][D + 4];
  __shared__ __attribute__((aligned(16))) float grow[16][D + 4];
  __shared__ __attribute__((aligned(16))) float2 tsc[16];  // (LSE, delta) of a tile's queries
  const int hk = blockIdx.y, NBm = nb - 1;
  if ((int)blockIdx.x >= c3_off[(size_t)hk * ((size_t)NBm * Ck + 1) + (size_t)NBm * Ck]) return;  // past the last item
  const int2 item = c3_map[(size_t)hk * run_cap + blockIdx.x];  // (pair, slice)
  const int sl = item.y, G_ = Hq / Hkv;
  const size_t hqbase = (size_t)(hk / Hkv) * Hq + (size_t)(hk % Hkv) * G_;
  const int lane = threadIdx.x, c16 = lane % 16, g = lane / 16;
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const int klo = ok[item.x], khi = ok[item.x + 1];  // pair = b' Ck + j indexes the segment table directly
  const int32_t* po = pair_off + (size_t)hk * ((size_t)NBm * Ck + 1) + item.x;
  const int hlo = po[0], hhi = po[1];
  if (klo == khi) return;
  const int step = 32 * c3_slices(hhi - hlo, tps);  // the slice's tiles of 32 hits, two tiles of 16 here
  const uint2* hh = hits + (size_t)hk * hit_cap;
  for (int k0 = klo; k0 < khi; k0 += 16) {
    const bool kvalid = k0 + c16 < khi;
    const size_t krow = ((size_t)hk * N + (kvalid ? k0 + c16 : klo)) * D;
    float4 kf[MT], vf[MT];
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      kf[u] = *reinterpret_cast<const float4*>(Ks + krow + 16 * u + 4 * g);
      vf[u] = *reinterpret_cast<const float4*>(Vs + krow + 16 * u + 4 * g);
    }
    f32x4_t dk[MT], dv[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < 4; ++t) { dk[m][t] = 0.f; dv[m][t] = 0.f; }
    float4 qn_[MT], gn_[MT];
    float2 scn;
    auto gather = [&](int h0) {  // rows of the 16 hits from h0, past the end the last hit with p = 0
      const bool hv = h0 + c16 < hhi;
      const uint32_t hit = hh[hv ? h0 + c16 : hhi - 1].x;
      const size_t qn = (hqbase + (hit >> 22)) * N + (hit & 0x3fffffu);
#pragma unroll
      for (int u = 0; u < MT; ++u) {
        qn_[u] = *reinterpret_cast<const float4*>(Q + qn * D + 16 * u + 4 * g);
        gn_[u] = *reinterpret_cast<const float4*>(dO + qn * D + 16 * u + 4 * g);
      }
      scn = make_float2(hv ? LSE[qn] : __builtin_huge_valf(), delta[qn]);
    };
    gather(hlo + 32 * sl);
    for (int h0 = hlo + 32 * sl; h0 < hhi; h0 += (h0 - hlo) % 32 == 0 ? 16 : step - 16) {
      f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
      wave_lds_fence();  // the previous tile's rows are read
#pragma unroll
      for (int u = 0; u < MT; ++u) {
        const float4 q4 = make_float4(scale * qn_[u].x, scale * qn_[u].y, scale * qn_[u].z, scale * qn_[u].w);
        const float qv[4] = {q4.x, q4.y, q4.z, q4.w}, gv[4] = {gn_[u].x, gn_[u].y, gn_[u].z, gn_[u].w};
        const float kv[4] = {kf[u].x, kf[u].y, kf[u].z, kf[u].w}, vv[4] = {vf[u].x, vf[u].y, vf[u].z, vf[u].w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          s = __builtin_amdgcn_mfma_f32_16x16x4f32(qv[t], kv[t], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_16x16x4f32(gv[t], vv[t], dp, 0, 0, 0);
        }
        *reinterpret_cast<float4*>(&qrow[c16][16 * u + 4 * g]) = q4;
        *reinterpret_cast<float4*>(&grow[c16][16 * u + 4 * g]) = gn_[u];
      }
      if (lane < 16) tsc[lane] = scn;
      wave_lds_fence();
      const int next = h0 + ((h0 - hlo) % 32 == 0 ? 16 : step - 16);
      if (next < hhi) gather(next);
      const float4 a4 = *reinterpret_cast<const float4*>(&tsc[4 * g]), b4 = *reinterpret_cast<const float4*>(&tsc[4 * g + 2]);
      const float ls[4] = {a4.x, a4.z, b4.x, b4.z}, de[4] = {a4.y, a4.w, b4.y, b4.w};
      float pr[4], dl[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        pr[t] = kvalid ? __expf(s[t] - ls[t]) : 0.f;
        dl[t] = pr[t] * (dp[t] - de[t]);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          dk[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(qrow[4 * g + t][16 * m + c16], dl[t], dk[m], 0, 0, 0);
          dv[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(grow[4 * g + t][16 * m + c16], pr[t], dv[m], 0, 0, 0);
        }
    }
    if (kvalid) {
      // slice 0 owns the gradient rows (cleared by the caller); a later slice leaves its share in its partial rows [dK | dV]
      const size_t mk = k0 + c16;
      float* pk = sl == 0 ? dKs + ((size_t)hk * N + mk) * D : part + ((((size_t)(sl - 1) * HK + hk) * N + mk) * 2) * D;
      float* pv = sl == 0 ? dVs + ((size_t)hk * N + mk) * D : pk + D;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int o = 16 * m + 4 * g;
        float4 a = make_float4(dk[m][0], dk[m][1], dk[m][2], dk[m][3]), c = make_float4(dv[m][0], dv[m][1], dv[m][2], dv[m][3]);
        if (sl == 0) {
          const float4 x = *reinterpret_cast<const float4*>(pk + o), y = *reinterpret_cast<const float4*>(pv + o);
          a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
          c.x += y.x; c.y += y.y; c.z += y.z; c.w += y.w;
        }
        *reinterpret_cast<float4*>(pk + o) = a;
        *reinterpret_cast<float4*>(pv + o) = c;
      }
    }
  }
}

}  // namespace

int muse_launch_c3_pairs_f32(const MuseDims& d, const float* Q, const float* dO, const float* LSE, FFWorkspace& w, hipStream_t st) {
  const int HK = d.B * d.Hkv;
  const dim3 g((unsigned)w.run_cap, HK);
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_c3_pairs_f32", st);
    hipLaunchKernelGGL(kernel, g, dim3(64), 0, st, Q, dO, (const float*)w.Ks, (const float*)w.Vs, LSE, w.delta, w.off_k, w.pair_off,
                       w.c3_off, w.c3_map, w.hits, w.dKs, w.dVs, w.c3_part, w.run_cap, w.hit_cap, d.N, d.nb, d.Ck, d.Hq, d.Hkv, HK, ff_c3_tiles(d), d.scale);
  };
  if (d.D == 64) go(k_c3_pairs_f32<64>);
  else go(k_c3_pairs_f32<128>);
  MUSE_LAUNCH_CHECK();
  return muse_launch_c3_reduce(d, w, st);
}
