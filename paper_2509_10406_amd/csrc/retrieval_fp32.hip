// Retrieval backward for fp32 inputs (Sec. 3.3 "Exact retrieval", gradient w.r.t. keys and values) on fp32 MFMA: a workgroup
// of four waves per (retrieved pair, hit slice) item of the inverse index; the pair is a dense attention-backward block, 16
// queries that retrieved it against 16 of its keys at a time (v_mfma_f32_16x16x4_f32: operand lanes hold four consecutive dims
// of a row, accumulator element t of lane l is row 4 (l / 16) + t, column l % 16).  The tiles of 16 hits go round the waves of
// all slices; the waves of a workgroup add up through LDS in wave order, the slices through partial rows (k_c3_reduce).
//
// Bound by the matrix instructions of the heavy pairs (64 of 32 cycles per tile at D = 64), which therefore go to several
// CUs; partial rows are what a CU more costs in memory, and ff_c3_cut says how many there is room for.  At 4 heads of 8k
// tokens with 128 key clusters and r = 4, 65 us and 10 for the reduction (three slices at most); one wave per slice and up to
// eight slices 71 + 10, a workgroup of eight waves per pair and no slices 112, a wave per (key block, 32 key clusters) that
// walked a bit matrix of the selections 5100.  D = 128 (there 156 us) keeps one wave per SIMD: with two, 73 registers spilled
// take 228.
#include "ff_common.h"
#include "fp32_sum.h"

namespace {

constexpr int W = 4;  // waves per workgroup, one per SIMD

template <int D>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1, 4))) k_c3_pairs_f32(
    const float* __restrict__ Q, const float* __restrict__ dO, const float* __restrict__ Ks, const float* __restrict__ Vs,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ off_k,
    const int32_t* __restrict__ pair_off, const int32_t* __restrict__ c3_off, const int2* __restrict__ c3_map,
    const uint2* __restrict__ hits, float* __restrict__ dKs, float* __restrict__ dVs, float* __restrict__ part,
    size_t run_cap, size_t hit_cap, int N, int nb, int Ck, int Hq, int Hkv, int HK, C3Cut cut, float scale) {
  constexpr int MT = D / 16;
  __shared__ __attribute__((aligned(16))) float rows[W][2][16][D + 4];  // q~ and dO of a wave's tile; at the end its sums
  __shared__ __attribute__((aligned(16))) float2 sc[W][16];             // (LSE, delta) of the tile's queries
  static_assert(sizeof(rows[0]) >= 2 * MT * 64 * 16, "a wave's sums fit its tiles");
  const int hk = blockIdx.y, NBm = nb - 1;
  if ((int)blockIdx.x >= c3_off[(size_t)hk * ((size_t)NBm * Ck + 1) + (size_t)NBm * Ck]) return;  // past the last item
  const int2 item = c3_map[(size_t)hk * run_cap + blockIdx.x];  // (pair, slice)
  const int sl = item.y, G_ = Hq / Hkv;
  const size_t hqbase = (size_t)(hk / Hkv) * Hq + (size_t)(hk % Hkv) * G_;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, c16 = lane % 16, g = lane / 16;
  float (*qrow)[D + 4] = rows[wave][0];
  float (*grow)[D + 4] = rows[wave][1];
  float2* tsc = sc[wave];
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const int klo = ok[item.x], khi = ok[item.x + 1];  // pair = b' Ck + j indexes the segment table directly
  const int32_t* po = pair_off + (size_t)hk * ((size_t)NBm * Ck + 1) + item.x;
  const int hlo = po[0], hhi = po[1];
  if (klo == khi) return;
  const int hfirst = hlo + 16 * (W * sl + wave), step = 16 * W * c3_slices(hhi - hlo, cut);  // the wave's tiles of 16 hits
  const int nw = min(W, (hhi - hlo + 15) / 16 - W * sl);  // waves of the slice that have hits
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
    if (wave < nw) gather(hfirst);
    for (int h0 = hfirst; h0 < hhi; h0 += step) {
      FoldSum ss, dps;
      wave_lds_fence();  // the previous tile's rows are read
#pragma unroll
      for (int u = 0; u < MT; ++u) {
        const float4 q4 = make_float4(scale * qn_[u].x, scale * qn_[u].y, scale * qn_[u].z, scale * qn_[u].w);
        const float qv[4] = {q4.x, q4.y, q4.z, q4.w}, gv[4] = {gn_[u].x, gn_[u].y, gn_[u].z, gn_[u].w};
        const float kv[4] = {kf[u].x, kf[u].y, kf[u].z, kf[u].w}, vv[4] = {vf[u].x, vf[u].y, vf[u].z, vf[u].w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          ss.add(t, qv[t], kv[t]);
          dps.add(t, gv[t], vv[t]);
        }
        ss.fold(u);
        dps.fold(u);
        *reinterpret_cast<float4*>(&qrow[c16][16 * u + 4 * g]) = q4;
        *reinterpret_cast<float4*>(&grow[c16][16 * u + 4 * g]) = gn_[u];
      }
      const f32x4_t s = ss.total, dp = dps.total;
      if (lane < 16) tsc[lane] = scn;
      wave_lds_fence();
      if (h0 + step < hhi) gather(h0 + step);
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
    // the waves' sums, 2 MT pieces of 16 bytes per lane: each wave adds up its share of the pieces
    float4* mine = reinterpret_cast<float4*>(&rows[wave][0][0][0]) + lane;
    wave_lds_fence();
    if (wave < nw)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        mine[64 * m] = make_float4(dk[m][0], dk[m][1], dk[m][2], dk[m][3]);
        mine[64 * (MT + m)] = make_float4(dv[m][0], dv[m][1], dv[m][2], dv[m][3]);
      }
    __syncthreads();
    if (kvalid)
#pragma unroll
      for (int z = 0; z < 2 * MT / W; ++z) {
        const int piece = wave + W * z;
        // slice 0 owns the gradient rows (cleared by the caller); a later slice leaves its share in its partial rows [dK | dV]
        float* row = sl == 0 ? (piece < MT ? dKs : dVs) + krow : part + 2 * ((size_t)(sl - 1) * HK * N * D + krow) + (piece < MT ? 0 : D);
        float4* dst = reinterpret_cast<float4*>(row + 16 * (piece % MT) + 4 * g);
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (sl == 0) a = *dst;
        for (int w = 0; w < nw; ++w) {
          const float4 x = reinterpret_cast<const float4*>(&rows[w][0][0][0])[64 * piece + lane];
          a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
        }
        *dst = a;
      }
    __syncthreads();
  }
}

}  // namespace

int muse_launch_c3_pairs_f32(const MuseDims& d, const float* Q, const float* dO, const float* LSE, FFWorkspace& w, hipStream_t st) {
  const int HK = d.B * d.Hkv;
  const dim3 g((unsigned)w.run_cap, HK);
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_c3_pairs_f32", st);
    hipLaunchKernelGGL(kernel, g, dim3(64 * W), 0, st, Q, dO, (const float*)w.Ks, (const float*)w.Vs, LSE, w.delta, w.off_k, w.pair_off,
                       w.c3_off, w.c3_map, w.hits, w.dKs, w.dVs, w.c3_part, w.run_cap, w.hit_cap, d.N, d.nb, d.Ck, d.Hq, d.Hkv, HK, ff_c3_cut(d), d.scale);
  };
  if (d.D == 64) go(k_c3_pairs_f32<64>);
  else go(k_c3_pairs_f32<128>);
  MUSE_LAUNCH_CHECK();
  if (ff_c3_cut(d).most == 1) return MUSE_OK;
  return muse_launch_c3_reduce(d, w, st);
}
