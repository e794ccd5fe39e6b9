// Gradients of the accumulated cells (component 1) for bf16 inputs: the queries of a (block b, query cluster i) group
// against the accumulated summaries they saw are a dense attention-backward block with the summaries in the role of
// keys and values:
//   g_A_k = sum dl q~,  g_A_v = sum p dO,  g_A_c = sum [dl (1 - q~.kbar) - p dO.vbar]
// Operands are rounded to bf16 for the matrix cores (gradients only; no selection depends on them).
//
// One workgroup per group: its queries (up to 96 at a time, nearly always all of them) are staged in LDS once, row-major;
// a wave walks the units of 16 key clusters (v_mfma_f32_16x16x32_bf16, the clusters being the columns) with the next
// unit's summaries in flight.  The rows serve S and dP as they lie and G_k, G_v through transposed reads.  A group with
// more than 96 queries takes further passes that add to the rows of the first.
//
// Bound by streaming the summaries in and the gradients out.  Units of 16 clusters halve a wave's accumulators against
// 32: at D = 128 that is two waves per SIMD and 96 staged queries in place of one wave and 32, whose second passes read
// and wrote everything again (10.2 -> 2.9 ms at 32 heads of 32k tokens, 128 x 512 clusters); at D = 64 three waves per
// SIMD in place of two (3.43 -> 3.24 ms at 16 heads of 64k, 256 x 1024; 0.63 -> 0.45 ms with 128 x 128).
#include "ff_common.h"
#include "lds_tile.h"

namespace {

constexpr int kQR = 96;  // queries staged at a time

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, D == 64 ? 3 : 2))) k_ff_bwd_cells_mx(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ dO, const float* __restrict__ qc,
    const float* __restrict__ A_mu, const bf16_t* __restrict__ A_kb, const bf16_t* __restrict__ A_v,
    const int32_t* __restrict__ perm_q, const int32_t* __restrict__ off_q, const float* __restrict__ LSE,
    const float* __restrict__ delta, const uint32_t* __restrict__ selmask, float* __restrict__ g_A_c,
    bf16_t* __restrict__ g_A_k, bf16_t* __restrict__ g_A_v, int h0, int N, int nb, int Cq, int Ck, float scale) {
  constexpr int KX = D / 32, MT = D / 16, CPR = D / 8;
  __shared__ __attribute__((aligned(16))) bf16_t qs[kQR * D];
  __shared__ __attribute__((aligned(16))) bf16_t gs[kQR * D];
  __shared__ __attribute__((aligned(16))) float ls[kQR];
  __shared__ __attribute__((aligned(16))) float ds[kQR];
  __shared__ __attribute__((aligned(16))) uint32_t mws[4][kQR];
  __shared__ __attribute__((aligned(16))) bf16_t tw[4][16][D + 8];
  const int hl = blockIdx.z, hq = h0 + hl;
  const int NBm = nb - 1, W = (Ck + 31) / 32, nunit = (Ck + 15) / 16;
  const int b = blockIdx.y / Cq + 1, i = blockIdx.y % Cq;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, c16 = lane % 16, g = lane / 16;
  const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1);
  const int qlo = oq[b * Cq + i], qhi = oq[b * Cq + i + 1];
  const size_t acell = (((size_t)hl * NBm + (b - 1)) * Cq + i) * Ck;
  const float* qci = qc + ((size_t)hq * Cq + i) * D;
  struct CT {  // one unit of 16 accumulated summaries as this lane's operands (cluster c16, dims 32 x + 8 g ..)
    bf16x8_t kf[KX], vf[KX];
    float amu;       // raw: any arithmetic on a prefetched value would wait for the whole prefetch at once
    uint32_t mw[2];  // selection-mask words of the staged queries lane and 64 + lane
  };
  auto load_ct = [&](int unit, int q0, CT& c) {
    const int jc = unit * 16 + c16 < Ck ? unit * 16 + c16 : Ck - 1;
#pragma unroll
    for (int x = 0; x < KX; ++x) {
      c.kf[x] = *reinterpret_cast<const bf16x8_t*>(A_kb + (acell + jc) * D + 32 * x + 8 * g);
      c.vf[x] = *reinterpret_cast<const bf16x8_t*>(A_v + (acell + jc) * D + 32 * x + 8 * g);
    }
    c.amu = A_mu[acell + jc];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const int pq = q0 + 64 * z + lane;
      c.mw[z] = selmask[((size_t)hq * W + unit / 2) * N + (pq < qhi ? pq : q0)];
    }
  };
  for (int q0 = qlo; q0 < qhi || q0 == qlo; q0 += kQR) {  // an empty group still writes its (zero) cells
    const bool first = q0 == qlo;
    const int ntl = q0 < qhi ? min((qhi - q0 + 31) / 32, kQR / 32) : 0;  // staged tiles of 32 queries
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kQR * CPR / 256; ++u) {
      const int c = threadIdx.x + 256 * u, row = c / CPR, cc = c % CPR;
      if (row < 32 * ntl) {
        const int pos = q0 + row < qhi ? q0 + row : q0;
        const size_t qn = (size_t)hq * N + perm_q[(size_t)hq * N + pos];
        const uint4 qv = *reinterpret_cast<const uint4*>(Q + qn * D + cc * 8);
        const uint4 gvv = *reinterpret_cast<const uint4*>(dO + qn * D + cc * 8);
        const float4 c0 = *reinterpret_cast<const float4*>(qci + cc * 8), c1 = *reinterpret_cast<const float4*>(qci + cc * 8 + 4);
        auto two = [&](uint32_t w, float a, float b2) {
          return pack_bf16x2(scale * (__uint_as_float(w << 16) - a), scale * (__uint_as_float(w & 0xffff0000u) - b2));
        };
        *reinterpret_cast<uint4*>(qs + tile_at<D>(row, cc)) = make_uint4(two(qv.x, c0.x, c0.y), two(qv.y, c0.z, c0.w), two(qv.z, c1.x, c1.y), two(qv.w, c1.z, c1.w));
        *reinterpret_cast<uint4*>(gs + tile_at<D>(row, cc)) = gvv;
      }
    }
    if (threadIdx.x < 32 * ntl) {
      const int row = threadIdx.x;
      const bool ok = q0 + row < qhi;
      const size_t qn = (size_t)hq * N + perm_q[(size_t)hq * N + (ok ? q0 + row : q0)];
      ls[row] = ok ? LSE[qn] * 1.4426950408889634f : __builtin_huge_valf();  // +inf -> p = 0 for padding rows
      ds[row] = delta[qn];
    }
    __syncthreads();
    CT cur, nxt;
    const int qm = q0 < qhi ? q0 : 0;
    if (wave < nunit) load_ct(wave, qm, cur);
    for (int unit = wave; unit < nunit; unit += 4) {
      // always issued (the last unit again at the end): with the same number of loads in flight on every path the wait
      // for this unit's operands can leave the next unit's loads outstanding
      load_ct(unit + 4 < nunit ? unit + 4 : unit, qm, nxt);
      wave_lds_fence();
      mws[wave][lane] = cur.mw[0];
      if (lane < kQR - 64) mws[wave][64 + lane] = cur.mw[1];
      wave_lds_fence();
      const int jc = unit * 16 + c16, bit = 16 * (unit & 1) + c16;
      const bool jvalid = jc < Ck;
      const float amu2 = jvalid ? cur.amu * 1.4426950408889634f : MUSE_NEG_INF;
      f32x4_t gk[MT], gv[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) { gk[m][t] = 0.f; gv[m][t] = 0.f; }
      float csum = 0.f;
      for (int qt = 0; qt < ntl; ++qt) {
        bf16x8_t pf, df;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int r0 = 32 * qt + 16 * u;
          f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int x = 0; x < KX; ++x) {
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_row<D>(qs, r0 + c16, 4 * x + g), cur.kf[x], s, 0, 0, 0);
            dp = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_row<D>(gs, r0 + c16, 4 * x + g), cur.vf[x], dp, 0, 0, 0);
          }
          const float4 l4 = *reinterpret_cast<const float4*>(&ls[r0 + 4 * g]), d4 = *reinterpret_cast<const float4*>(&ds[r0 + 4 * g]);
          const uint4 w4 = *reinterpret_cast<const uint4*>(&mws[wave][r0 + 4 * g]);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv4[4] = {d4.x, d4.y, d4.z, d4.w};
          const uint32_t mv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            float p = __builtin_amdgcn_exp2f(fmaf(s[t], 1.4426950408889634f, amu2 - lv[t]));
            p = ((mv[t] >> bit) & 1u) ? 0.f : p;
            const float dlg = p * (dp[t] - dv4[t]);
            csum += p > 0.f ? dlg * (1.f - s[t]) - p * dp[t] : 0.f;
            pf[4 * u + t] = (__bf16)p;
            df[4 * u + t] = (__bf16)dlg;
          }
        }
        // k-slots of lane group g: rows 4 g .. and 16 + 4 g .. of the 32, as in pf and df
        const int rr = 32 * qt + 4 * g + c16 / 4, cc = 4 * (c16 % 4);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const bf16x8_t ag = tr_join(tile_tr4<D>(gs, rr, 16 * m + cc), tile_tr4<D>(gs, rr + 16, 16 * m + cc));
          gv[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag, pf, gv[m], 0, 0, 0);
          const bf16x8_t aq = tr_join(tile_tr4<D>(qs, rr, 16 * m + cc), tile_tr4<D>(qs, rr + 16, 16 * m + cc));
          gk[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, df, gk[m], 0, 0, 0);
        }
      }
      csum += __shfl_xor(csum, 16, 64);
      csum += __shfl_xor(csum, 32, 64);
      // rows go out through a per-wave LDS tile: a store instruction then writes 64 / (D/8) whole rows of consecutive
      // clusters (contiguous memory)
#pragma unroll
      for (int arr = 0; arr < 2; ++arr) {
        wave_lds_fence();
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const f32x4_t& a = arr == 0 ? gk[m] : gv[m];
          *reinterpret_cast<uint2*>(&tw[wave][c16][16 * m + 4 * g]) = make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
        }
        wave_lds_fence();
        bf16_t* dst = arr == 0 ? g_A_k : g_A_v;
#pragma unroll
        for (int it = 0; it < 16 * CPR / 64; ++it) {
          const int row = it * (64 / CPR) + lane / CPR, cc = lane % CPR;
          if (unit * 16 + row < Ck) {
            uint4 v = *reinterpret_cast<const uint4*>(&tw[wave][row][cc * 8]);
            uint4* o = reinterpret_cast<uint4*>(dst + (acell + unit * 16 + row) * D + cc * 8);
            if (!first) {  // further pass of a large group: add to what the earlier passes wrote
              const uint4 old = *o;
              auto add2 = [](uint32_t x, uint32_t y) {
                return pack_bf16x2(__uint_as_float(x << 16) + __uint_as_float(y << 16),
                                   __uint_as_float(x & 0xffff0000u) + __uint_as_float(y & 0xffff0000u));
              };
              v = make_uint4(add2(v.x, old.x), add2(v.y, old.y), add2(v.z, old.z), add2(v.w, old.w));
            }
            typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
            const u4_t vs = {v.x, v.y, v.z, v.w};
            __builtin_nontemporal_store(vs, reinterpret_cast<u4_t*>(o));  // written once, read by the next kernel much later
          }
        }
      }
      if (jvalid && g == 0) g_A_c[acell + jc] = first ? csum : g_A_c[acell + jc] + csum;
      cur = nxt;
    }
  }
}

}  // namespace

int muse_launch_ff_bwd_cells_mx(const MuseDims& d, const void* Q, const void* dO, const float* qc, const float* LSE,
                                FFWorkspace& w, int h0, int hn, hipStream_t st) {
  const dim3 g(1, (d.nb - 1) * d.Cq, hn);
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_ff_bwd_cells_mx", st);
    hipLaunchKernelGGL(kernel, g, dim3(256), 0, st, (const bf16_t*)Q, (const bf16_t*)dO, qc, w.A_mu, (const bf16_t*)w.A_kb,
                       (const bf16_t*)w.A_v, w.perm_q, w.off_q, LSE, w.delta, w.selmask, w.g_A_c, (bf16_t*)w.g_A_k,
                       (bf16_t*)w.g_A_v, h0, d.N, d.nb, d.Cq, d.Ck, d.scale);
  };
  if (d.D == 64) go(k_ff_bwd_cells_mx<64>);
  else go(k_ff_bwd_cells_mx<128>);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
