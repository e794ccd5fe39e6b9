// Retrieval backward, gradient w.r.t. keys and values (Sec. 3.3 "Exact retrieval") for bf16 inputs, and the reduction of
// the hit slices of a pair (also behind the fp32 kernel of retrieval_fp32.hip).
#include "ff_common.h"
#include "lds_tile.h"

namespace {

// A workgroup of two waves per (retrieved pair, hit slice): the queries that retrieved the pair are gathered, and the pair
// is a dense attention-backward block with its keys as the MFMA columns.
//   hit = n | g << 22  (query position, query head inside the KV group)
// Bound by the gathers: a hit is two rows of 2 D bytes from anywhere in Q and dO.  So
//   - a step's rows (64 hits at D = 64, 32 at D = 128) are requested whole rows at a time (8 or 16 lanes a row) while
//     the step before is computed, with the hits of the step after behind them: one round trip per step, none exposed;
//   - they are staged once, row-major, for both operand forms (lds_tile.h), instead of a transposed copy in 2-byte stores;
//   - at D = 64 the two waves take 32 keys each of the same hits (one gather for 64 keys), or, where at most 32 keys are
//     left, the two halves of the hits, added up through LDS at the end; at D = 128 they take half of the head dim of
//     dK and dV each, which keeps two waves per SIMD.
// One wave per (pair, slice) that gathered 16 bytes of 32 rows per instruction and stored them transposed took 2.30 ms at 16
// heads of 64k tokens with 128 x 128 clusters (now 1.22: 7.3 M hits, 1.9 GB of rows), 1.00 with 256 x 1024 (0.82), 2.54 at
// 32 heads of 32k, D = 128 (1.61).
// A pair with many hits (at 128 x 128 clusters of 64k tokens: 600 on average, 16k at most) is shared by c3_slices
// workgroups, each with an equal run of the hit tiles: slice 0 adds to the bucketed-order gradient rows of the pair's keys,
// the others write partial rows, which k_c3_reduce adds in slice order (fixed order, no atomics).  blockIdx.z deals the
// key groups of a pair out to as many workgroups as the average pair has use for.
template <int D>
__global__ void __launch_bounds__(128, 2) k_c3_pairs(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ dO, const bf16_t* __restrict__ Ks, const bf16_t* __restrict__ Vs,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ off_k,
    const int32_t* __restrict__ pair_off, const int32_t* __restrict__ c3_off, const int2* __restrict__ c3_map,
    const uint2* __restrict__ hits, float* __restrict__ dKs, float* __restrict__ dVs, float* __restrict__ part, size_t run_cap,
    size_t hit_cap, int N, int nb, int Ck, int Hq, int Hkv, int HK, C3Cut cut, float scale, float scale_log2e) {
  constexpr int KS = D / 16, CPR = D / 8;
  constexpr bool kSplitD = D == 128;              // the waves share one key tile and split the head dim of the results
  constexpr int DT = 2;                           // 32-dim tiles of dK and dV per wave
  constexpr int R = 4096 / D, KG = kSplitD ? 32 : 64;  // hits per step, keys per group
  constexpr int RPI = 128 / CPR;                  // rows per load instruction of the workgroup
  __shared__ __attribute__((aligned(16))) bf16_t st_[2 * R * D];
  __shared__ __attribute__((aligned(16))) float lse_s[R];
  __shared__ __attribute__((aligned(16))) float dl_s[R];
  bf16_t* qs = st_;
  bf16_t* gs = st_ + R * D;
  const int hk = blockIdx.y, NBm = nb - 1;
  if ((int)blockIdx.x >= c3_off[(size_t)hk * ((size_t)NBm * Ck + 1) + (size_t)NBm * Ck]) return;  // past the last item
  const int2 item = c3_map[(size_t)hk * run_cap + blockIdx.x];  // (pair, slice)
  const int sl = item.y;
  const int G_ = Hq / Hkv;
  const size_t hqbase = (size_t)(hk / Hkv) * Hq + (size_t)(hk % Hkv) * G_;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, col = lane % 32, half = lane / 32;
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const int klo = ok[item.x], khi = ok[item.x + 1];  // pair = b' Ck + j indexes the segment table directly
  const int kbeg = klo + KG * (int)blockIdx.z;
  if (kbeg >= khi) return;
  const int32_t* po = pair_off + (size_t)hk * ((size_t)NBm * Ck + 1) + item.x;
  const int plo = po[0], phi = po[1], nt = (phi - plo + 31) / 32, S = c3_slices(phi - plo, cut);
  const int hlo = plo + 32 * (nt * sl / S), hhi = min(phi, plo + 32 * (nt * (sl + 1) / S));  // this slice's hits, never empty
  const uint2* hh = hits + (size_t)hk * hit_cap;
  const int row0 = tid / CPR, chunk = tid % CPR;
  const int d0 = kSplitD ? 64 * w : 0;
  for (int k0 = kbeg; k0 < khi; k0 += KG * (int)gridDim.z) {
    const bool two = !kSplitD && khi - k0 > 32;  // two key tiles, one per wave
    const int mk = k0 + (two ? 32 * w : 0) + col;
    const bool kvalid = mk < khi;
    const size_t krow = ((size_t)hk * N + (kvalid ? mk : klo)) * D;
    bf16x8_t kf[KS], vf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      kf[s] = *reinterpret_cast<const bf16x8_t*>(Ks + krow + 16 * s + 8 * half);
      vf[s] = *reinterpret_cast<const bf16x8_t*>(Vs + krow + 16 * s + 8 * half);
    }
    f32x16_t dk[DT], dv[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) { dk[t][e] = 0.f; dv[t][e] = 0.f; }
    // a thread's hits of a step (row row0 + RPI it, as row indices of Q), its 16 bytes of their rows, and for the first
    // R threads LSE and delta of hit tid; past the end the last hit again
    uint32_t hn[4], hm;
    uint4 q0, q1, q2, q3, g0, g1, g2, g3;
    float lse, dl;
    auto load_hits = [&](int h0) {
#pragma unroll
      for (int it = 0; it < 4; ++it) hn[it] = hh[min(h0 + row0 + RPI * it, hhi - 1)].x;
      hm = hh[min(h0 + tid % R, hhi - 1)].x;
    };
    auto qrow = [&](uint32_t h) { return (hqbase + (h >> 22)) * N + (h & 0x3fffffu); };
    auto gather = [&]() {
      const size_t o0 = qrow(hn[0]) * D + 8 * chunk, o1 = qrow(hn[1]) * D + 8 * chunk, o2 = qrow(hn[2]) * D + 8 * chunk,
                   o3 = qrow(hn[3]) * D + 8 * chunk;
      q0 = *reinterpret_cast<const uint4*>(Q + o0); g0 = *reinterpret_cast<const uint4*>(dO + o0);
      q1 = *reinterpret_cast<const uint4*>(Q + o1); g1 = *reinterpret_cast<const uint4*>(dO + o1);
      q2 = *reinterpret_cast<const uint4*>(Q + o2); g2 = *reinterpret_cast<const uint4*>(dO + o2);
      q3 = *reinterpret_cast<const uint4*>(Q + o3); g3 = *reinterpret_cast<const uint4*>(dO + o3);
      const size_t qm = qrow(hm);
      lse = LSE[qm];
      dl = delta[qm];
    };
    auto put = [&](int it, const uint4& q, const uint4& g) {
      const int at = tile_at<D>(row0 + RPI * it, chunk);
      *reinterpret_cast<uint4*>(qs + at) = q;
      *reinterpret_cast<uint4*>(gs + at) = g;
    };
    load_hits(hlo);
    gather();
    load_hits(hlo + R);
    for (int h0 = hlo; h0 < hhi; h0 += R) {
      __syncthreads();
      put(0, q0, g0); put(1, q1, g1); put(2, q2, g2); put(3, q3, g3);
      if (tid < R) {
        lse_s[tid] = h0 + tid < hhi ? lse * 1.4426950408889634f : __builtin_huge_valf();  // +inf -> p = 0
        dl_s[tid] = dl;
      }
      __syncthreads();
      gather();
      load_hits(h0 + 2 * R);
#pragma unroll 1
      for (int u = (kSplitD || two) ? 0 : w; u < (kSplitD ? 1 : 2); u += two ? 1 : 2) {
        if (h0 + 32 * u >= hhi) break;
        f32x16_t s, dp;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
        for (int x = 0; x < KS; ++x) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(qs, 32 * u + col, 2 * x + half), kf[x], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(gs, 32 * u + col, 2 * x + half), vf[x], dp, 0, 0, 0);
        }
        f32x16_t pr;
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const float4 l4 = *reinterpret_cast<const float4*>(&lse_s[32 * u + 8 * gq + 4 * half]);
          const float4 d4 = *reinterpret_cast<const float4*>(&dl_s[32 * u + 8 * gq + 4 * half]);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            const int e = 4 * gq + y;
            pr[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -lv[y]));
            s[e] = pr[e] * (dp[e] - dv4[y]);
          }
        }
        // transposed operands: this lane group's 16 columns (dims), rows 4 half .. and 8 + 4 half .. of 16 hits
        const int rr = 32 * u + 4 * half + (lane % 16) / 4, cc = d0 + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
#pragma unroll
        for (int G = 0; G < 2; ++G) {
          const bf16x8_t pf = pack8(pr, 2 * G, 2 * G + 1), df = pack8(s, 2 * G, 2 * G + 1);
#pragma unroll
          for (int t = 0; t < DT; ++t) {
            const bf16x8_t ag = tr_join(tile_tr4<D>(gs, rr + 16 * G, 32 * t + cc), tile_tr4<D>(gs, rr + 16 * G + 8, 32 * t + cc));
            dv[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ag, pf, dv[t], 0, 0, 0);
            const bf16x8_t aq = tr_join(tile_tr4<D>(qs, rr + 16 * G, 32 * t + cc), tile_tr4<D>(qs, rr + 16 * G + 8, 32 * t + cc));
            dk[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq, df, dk[t], 0, 0, 0);
          }
        }
      }
    }
    if (!kSplitD && !two) {  // both waves hold sums of the same keys: wave 1 hands its own over, 8 KB of dK and of dV in turn
      float* x = reinterpret_cast<float*>(st_);
      static_assert(kSplitD || sizeof(st_) >= 4 * 64 * DT * 16, "one result of a wave fits the staged rows");
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        __syncthreads();
        if (w == 1) {
#pragma unroll
          for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) x[(16 * t + e) * 64 + lane] = z ? dv[t][e] : dk[t][e];
        }
        __syncthreads();
        if (w == 0) {
#pragma unroll
          for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) (z ? dv : dk)[t][e] += x[(16 * t + e) * 64 + lane];
        }
      }
    }
    if (kvalid && (kSplitD || two || w == 0)) {
      // slice 0 owns the gradient rows; a later slice leaves its share in its own partial rows [dK | dV]
      float* pk = (sl == 0 ? dKs + ((size_t)hk * N + mk) * D : part + ((((size_t)(sl - 1) * HK + hk) * N + mk) * 2) * D) + d0;
      float* pv = sl == 0 ? dVs + ((size_t)hk * N + mk) * D + d0 : pk + D;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int o = 32 * t + 8 * g + 4 * half;
          float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
          if (sl == 0) { a = *reinterpret_cast<float4*>(pk + o); c = *reinterpret_cast<float4*>(pv + o); }
          a.x += scale * dk[t][4 * g + 0]; a.y += scale * dk[t][4 * g + 1];
          a.z += scale * dk[t][4 * g + 2]; a.w += scale * dk[t][4 * g + 3];
          c.x += dv[t][4 * g + 0]; c.y += dv[t][4 * g + 1]; c.z += dv[t][4 * g + 2]; c.w += dv[t][4 * g + 3];
          *reinterpret_cast<float4*>(pk + o) = a;
          *reinterpret_cast<float4*>(pv + o) = c;
        }
    }
  }
}

// adds the partial rows of the hit slices 1 .. S-1 of every pair to the rows slice 0 owns, in slice order: one workgroup
// per pair, 16 lanes per key row, a row's slices requested together (16 heads of 64k tokens with 128 x 128
// clusters: 0.16 ms, the rows themselves)
template <int D>
__global__ void __launch_bounds__(256) k_c3_reduce(const int32_t* __restrict__ off_k, const int32_t* __restrict__ pair_off,
                                                   const int32_t* __restrict__ c3_off, const int2* __restrict__ c3_map,
                                                   const float* __restrict__ part, float* __restrict__ dKs,
                                                   float* __restrict__ dVs, size_t run_cap, int N, int nb, int Ck, int HK, C3Cut cut) {
  // walks the same item list as k_c3_pairs: the item (pair, slice 1) exists exactly for the pairs with partial rows
  const int hk = blockIdx.y, NBm = nb - 1;
  if ((int)blockIdx.x >= c3_off[(size_t)hk * ((size_t)NBm * Ck + 1) + (size_t)NBm * Ck]) return;
  const int2 item = c3_map[(size_t)hk * run_cap + blockIdx.x];
  if (item.y != 1) return;
  const int32_t* po = pair_off + (size_t)hk * ((size_t)NBm * Ck + 1) + item.x;
  const int S = c3_slices(po[1] - po[0], cut);  // every slice has hits
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const int klo = ok[item.x], khi = ok[item.x + 1];
  const int sub = threadIdx.x / 16, l16 = threadIdx.x % 16;
  for (int m = klo + sub; m < khi; m += 16)
#pragma unroll
    for (int d0 = 0; d0 < 2 * D; d0 += 64) {  // the row pair [dK | dV] as 2 D floats
      const int d = d0 + 4 * l16;
      float* dst = (d0 < D ? dKs : dVs - D) + ((size_t)hk * N + m) * D + d;
      float4 a = *reinterpret_cast<float4*>(dst), x[kC3Slices - 1];
#pragma unroll
      for (int s = 1; s < kC3Slices; ++s)
        x[s - 1] = *reinterpret_cast<const float4*>(part + ((((size_t)((s < S ? s : 1) - 1) * HK + hk) * N + m) * 2) * D + d);
#pragma unroll
      for (int s = 1; s < kC3Slices; ++s)
        if (s < S) { a.x += x[s - 1].x; a.y += x[s - 1].y; a.z += x[s - 1].z; a.w += x[s - 1].w; }
      *reinterpret_cast<float4*>(dst) = a;
    }
}

}  // namespace

int muse_launch_c3_reduce(const MuseDims& d, FFWorkspace& w, hipStream_t st) {
  const int HK = d.B * d.Hkv;
  const dim3 g((unsigned)w.run_cap, HK);
  MuseProf prof_("k_c3_reduce", st);
  if (d.D == 64) hipLaunchKernelGGL(k_c3_reduce<64>, g, dim3(256), 0, st, w.off_k, w.pair_off, w.c3_off, w.c3_map, w.c3_part, w.dKs, w.dVs, w.run_cap, d.N, d.nb, d.Ck, HK, ff_c3_cut(d));
  else hipLaunchKernelGGL(k_c3_reduce<128>, g, dim3(256), 0, st, w.off_k, w.pair_off, w.c3_off, w.c3_map, w.c3_part, w.dKs, w.dVs, w.run_cap, d.N, d.nb, d.Ck, HK, ff_c3_cut(d));
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_c3_pairs(const MuseDims& d, const void* Q, const void* dO, const float* LSE, FFWorkspace& w, hipStream_t st) {
  const int HK = d.B * d.Hkv;
  // A pair has N / (nb Ck) keys on average and a few times that at most: 1, 2 or 4 workgroups share its groups of keys, each
  // of which gathers the hits anew.  Kernel us with 1 / 2 / 4, by keys of the average pair: 16 heads of 64k tokens, r = 8,
  //   8: 722 797 894   16: 759 802 854   32: 949 963 1023   64: 1234 1221 1250   128: 1713 1641 1632;
  // 8 heads of 16k   8: 75 77 88   16: 103 93 94   32: 112 103 113   64: 149 132 132   128: 240 181 168;
  // 32 heads of 32k, D = 128   8: 962 1024 1025   16: 1341 1256 1258   32: 1785 1543 1651   64: 2820 2509 2340.
  const int keys = d.N / (d.nb * d.Ck), z = keys <= 16 ? 1 : keys <= 32 ? 2 : 4;
  const dim3 g((unsigned)w.run_cap, HK, z);
  const float sl = d.scale * 1.4426950408889634f;
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_c3_pairs", st);
    hipLaunchKernelGGL(kernel, g, dim3(128), 0, st, (const bf16_t*)Q, (const bf16_t*)dO, (const bf16_t*)w.Ks, (const bf16_t*)w.Vs, LSE,
                       w.delta, w.off_k, w.pair_off, w.c3_off, w.c3_map, w.hits, w.dKs, w.dVs, w.c3_part, w.run_cap, w.hit_cap, d.N,
                       d.nb, d.Ck, d.Hq, d.Hkv, HK, ff_c3_cut(d), d.scale, sl);
  };
  if (d.D == 64) go(k_c3_pairs<64>);
  else go(k_c3_pairs<128>);
  MUSE_LAUNCH_CHECK();
  return muse_launch_c3_reduce(d, w, st);
}
