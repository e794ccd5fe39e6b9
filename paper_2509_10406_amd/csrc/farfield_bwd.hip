// Far-field backward: gradient of the forward of Sec. 3.1-3.3 with the assignments, the selections
// and the query centroids held fixed (App. C "Centroid Gradient Flow"); gradient flows into K and
// V through the tilted aggregation weights (App. C "Aggregation Weight Gradient Flow", default).
//
// With p_u = exp(logit_u - LSE), delta = dO.O, dl_u = p_u (dO.value_u - delta) per virtual key:
//   summary keys (component 1 on accumulated cells, component 2 on per-block cells):
//     dq~ += dl kappa,  g_k[cell] += dl q~,  g_v[cell] += p dO,  g_mu[cell] += dl
//   a cell in unnormalised form (S = e^mu, Ksum = S kappa, Vsum = S vbar) receives
//     dKsum = g_k/S, dVsum = g_v/S, dS = c/S with c = g_mu - g_k.kappa - g_v.vbar,
//   accumulated cells are plain sums of per-block (S, Ksum, Vsum), and for a key m of a per-block
//   cell with w = exp(qbar.k_m - mu):  dv_m += w G_v,  dk_m += w G_k + w (G_c + G_k.k_m + G_v.v_m) qbar,
//   where G = own gradient + sum over later accumulated cells a of exp(mu - Amu[a]) gA[a].
// Every reduction has one owner (no float atomics): cells by (query cluster, key-cluster tile),
// keys by (key block, key-cluster tile).
#include <algorithm>
#include <type_traits>

#include "ff_common.h"
#include "lds_tile.h"

namespace {

// The exported selections, re-indexed by bucketed query position p (consecutive p = one (block, cluster)
// group, so that every later read is coalesced):
//   slotinfo[hq][p][t] = j | (bitmask of the retrieved key blocks) << 16 for slot t, -1 when the slot is empty
//   selmask[hq][j/32][p]: bit j%32 set when query p retrieved key cluster j
// R >= r: a query's slots are held in registers, so that all its loads are requested together (a loop over the slots beyond
// eight took 1.02 ms at 32 heads of 32k with r = 16, this 0.21).
template <int R>
__global__ void __launch_bounds__(256) k_selinfo(const int32_t* __restrict__ selc, const int32_t* __restrict__ selb,
                                                  const int32_t* __restrict__ perm_q, uint32_t* __restrict__ mask,
                                                  int32_t* __restrict__ slotinfo, int N, int r, int k2e, int W) {
  const size_t hq = blockIdx.y;
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= N) return;
  const size_t q = hq * N + perm_q[hq * N + p];
  int32_t* si = slotinfo + (hq * N + p) * r;
  int jj[R];
  uint32_t bm[R];
#pragma unroll
  for (int t = 0; t < R; ++t) {
    jj[t] = t < r ? selc[q * r + t] : -1;
    bm[t] = 0;
  }
  for (int u = 0; u < k2e; ++u) {
    int bb[R];
#pragma unroll
    for (int t = 0; t < R; ++t) bb[t] = t < r ? selb[(q * r + t) * k2e + u] : -1;
#pragma unroll
    for (int t = 0; t < R; ++t) bm[t] |= bb[t] >= 0 ? 1u << bb[t] : 0u;
  }
#pragma unroll
  for (int t = 0; t < R; ++t)
    if (t < r) si[t] = jj[t] >= 0 ? (int)((uint32_t)jj[t] | (bm[t] << 16)) : -1;
  for (int w = 0; w < W; ++w) {
    uint32_t m = 0;
#pragma unroll
    for (int t = 0; t < R; ++t) m |= (jj[t] >> 5) == w ? 1u << (jj[t] & 31) : 0u;
    mask[(hq * W + w) * N + p] = m;
  }
}

// ------------------------------------------------------------------------------------------
// dQ of component 1, one wave per query tile (same tiling as the forward kernel)
// ------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1, 2))) k_ff_bwd_dq(
    const T* __restrict__ Q, const T* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ A_mu,
    const float* __restrict__ A_k, const T* __restrict__ A_v, const bf16_t* __restrict__ A_kb,
    const int32_t* __restrict__ perm_q, const int32_t* __restrict__ off_q, const int32_t* __restrict__ tile_off,
    const float* __restrict__ LSE, const float* __restrict__ delta, const uint32_t* __restrict__ selmask,
    float* __restrict__ dQ, bool add, int h0, int N, int nb, int Cq, int Ck, float scale) {
  constexpr int U = D / 8, DT = D / 32;
  const int hl = blockIdx.z, hq = h0 + hl;
  const int b = blockIdx.y + 1, NBm = nb - 1;
  const int lane = threadIdx.x, col = lane % 32, half = lane / 32;
  const int W = (Ck + 31) / 32;

  const int32_t* to = tile_off + ((size_t)hq * nb + b) * (Cq + 1);
  // x % 8 is the XCD (grid x extent a multiple of 8): each XCD takes a contiguous run of the tiles, so the
  // tiles of one (block, query cluster) group share its L2
  const int ntl = to[Cq], run = (ntl + 7) / 8;
  const int tile = (blockIdx.x % 8) * run + blockIdx.x / 8;
  if ((int)blockIdx.x / 8 >= run || tile >= ntl) return;
  int lo_ = 0, hi_ = Cq;
  while (hi_ - lo_ > 1) {
    int mid = (lo_ + hi_) >> 1;
    if (to[mid] <= tile) lo_ = mid; else hi_ = mid;
  }
  const int i = lo_, tt = tile - to[lo_];
  const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1);
  const int qlo = oq[b * Cq + i], qhi = oq[b * Cq + i + 1];
  int pos = qlo + 32 * tt + col;
  const bool valid = pos < qhi;
  pos = valid ? pos : qlo + 32 * tt;
  const int n = perm_q[(size_t)hq * N + pos];
  const size_t qn = (size_t)hq * N + n;

  float qt[U][4], gt[U][4];  // fp32 inputs
  if constexpr (sizeof(T) == 4) {
    const float* qci = qc + ((size_t)hq * Cq + i) * D;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[4];
      ld4(Q, qn * D + 8 * u + 4 * half, x);
      float4 c = *reinterpret_cast<const float4*>(qci + 8 * u + 4 * half);
      qt[u][0] = scale * (x[0] - c.x); qt[u][1] = scale * (x[1] - c.y);
      qt[u][2] = scale * (x[2] - c.z); qt[u][3] = scale * (x[3] - c.w);
      ld4(dO, qn * D + 8 * u + 4 * half, gt[u]);
    }
  }
  const float lse = LSE[qn], dl = delta[qn];
  const size_t acell = (((size_t)hl * NBm + (b - 1)) * Cq + i) * Ck;
  const float* Amu = A_mu + acell;
  const float* Ak = A_k + acell * D;
  const float* Avf = reinterpret_cast<const float*>(A_v) + acell * D;   // fp32 inputs
  const bf16_t* Akh = A_kb + acell * D;                                  // bf16 inputs
  const bf16_t* Avh = reinterpret_cast<const bf16_t*>(A_v) + acell * D;
  const int ntile = (Ck + 31) / 32;

  f32x16_t dq[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) dq[t] = zero16();
  // component 1
  if constexpr (sizeof(T) == 2) {
    // bf16 inputs: operands rounded to bf16 for the matrix cores (gradients only)
    constexpr int KS = D / 16, CPR = D / 8, NIT = 32 * CPR / 64;
    __shared__ __attribute__((aligned(16))) bf16_t kt[32 * D];
    __shared__ __attribute__((aligned(16))) bf16_t vt[32 * D];
    __shared__ __attribute__((aligned(16))) float mus[32];
    bf16x8_t qb[KS], gb[KS];
    // the bf16 operand order (8 consecutive dims per lane half) differs from the fp32 row pattern of qt/gt
    {
      const float* qci = qc + ((size_t)hq * Cq + i) * D;
#pragma unroll
      for (int x = 0; x < KS; ++x) {
        float q8[8], g8[8];
        ld4(Q, qn * D + 16 * x + 8 * half, q8); ld4(Q, qn * D + 16 * x + 8 * half + 4, q8 + 4);
        ld4(dO, qn * D + 16 * x + 8 * half, g8); ld4(dO, qn * D + 16 * x + 8 * half + 4, g8 + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          qb[x][e] = (__bf16)(scale * (q8[e] - qci[16 * x + 8 * half + e]));
          gb[x][e] = (__bf16)g8[e];
        }
      }
    }
    // A tile: the k-bar and v-bar rows of 32 clusters, whole rows per load instruction (a lane that reads its own operand
    // touches 32 rows with every instruction), their mu-bar (lane col) and the retrieved-cluster mask of the lane's query.
    // Two buffers in registers: the next tile's loads are in flight while this one is used; loads are unconditional (a
    // tile index past the end repeats the last tile) and the values stay raw until they are used.  Through LDS, row-major,
    // the rows serve S and dP as they lie and the dq contraction through transposed reads.
    struct BT {
      bf16x8_t k[NIT], v[NIT];
      float mu;
      uint32_t mw;
    };
    auto load_bt = [&](BT& t, int jt) {
      jt = jt < ntile ? jt : ntile - 1;
      const int j0 = jt * 32;
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const uint32_t o = (uint32_t)(min(j0 + it * (64 / CPR) + lane / CPR, Ck - 1) * D + lane % CPR * 8);
        t.k[it] = *reinterpret_cast<const bf16x8_t*>(Akh + o);
        t.v[it] = *reinterpret_cast<const bf16x8_t*>(Avh + o);
      }
      t.mu = Amu[min(j0 + col, Ck - 1)];
      t.mw = selmask[((size_t)hq * W + jt) * N + pos];
    };
    auto process = [&](const BT& t, int jt) {
      const int j0 = jt * 32;
      wave_lds_fence();
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int at = tile_at<D>(it * (64 / CPR) + lane / CPR, lane % CPR);
        *reinterpret_cast<bf16x8_t*>(kt + at) = t.k[it];
        *reinterpret_cast<bf16x8_t*>(vt + at) = t.v[it];
      }
      if (half == 0) mus[col] = t.mu;
      wave_lds_fence();
      f32x16_t s, dp = zero16();
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 m4 = *reinterpret_cast<const float4*>(&mus[8 * g + 4 * half]);
        s[4 * g] = m4.x; s[4 * g + 1] = m4.y; s[4 * g + 2] = m4.z; s[4 * g + 3] = m4.w;
      }
#pragma unroll
      for (int x = 0; x < KS; ++x) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(kt, col, 2 * x + half), qb[x], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(vt, col, 2 * x + half), gb[x], dp, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = 8 * (e / 4) + 4 * half + (e % 4);
        const bool off_ = ((t.mw >> row) & 1u) || j0 + row >= Ck;  // retrieved, or past the last cluster
        const float p = off_ ? 0.f : __expf(s[e] - lse);
        s[e] = p * (dp[e] - dl);
      }
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        const bf16x8_t df = pack8(s, 2 * G, 2 * G + 1);
#pragma unroll
        for (int x = 0; x < DT; ++x)
          dq[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_cols<D>(kt, 16 * G, x, lane), df, dq[x], 0, 0, 0);
      }
    };
    BT ta, tb;
    load_bt(ta, 0);
    for (int jt = 0; jt < ntile; jt += 2) {
      load_bt(tb, jt + 1);
      process(ta, jt);
      if (jt + 1 < ntile) {
        load_bt(ta, jt + 2);
        process(tb, jt + 1);
      }
    }
  } else
  for (int jt = 0; jt < ntile; ++jt) {
    const int j0 = jt * 32;
    f32x16_t s = score_tile<D>(Amu, Ak, j0, Ck, qt, col, half);
    int c = j0 + col;
    c = c < Ck ? c : Ck - 1;
    f32x16_t dp = mfma_rows<D>(zero16(), Avf + (size_t)c * D + 4 * half, gt);
    const uint32_t mw = selmask[((size_t)hq * W + jt) * N + pos];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      int row = 8 * (e / 4) + 4 * half + (e % 4);
      float p = ((mw >> row) & 1u) ? 0.f : __expf(s[e] - lse);
      s[e] = p * (dp[e] - dl);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        int jr = j0 + 8 * g + 4 * half + t;
        jr = jr < Ck ? jr : Ck - 1;
        const float* krow = Ak + (size_t)jr * D + col;
#pragma unroll
        for (int x = 0; x < DT; ++x) dq[x] = mfma32(krow[32 * x], s[4 * g + t], dq[x]);
      }
  }
  if (!valid) return;
  float res[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int x = 0; x < 4; ++x) res[u][x] = scale * dq[u / 4][4 * (u % 4) + x];
  float* out = dQ + qn * D + 4 * half;
  if (add) {  // to what the block-diagonal kernel left
    float4 o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) o[u] = *reinterpret_cast<const float4*>(out + 8 * u);
#pragma unroll
    for (int u = 0; u < U; ++u) { res[u][0] += o[u].x; res[u][1] += o[u].y; res[u][2] += o[u].z; res[u][3] += o[u].w; }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    *reinterpret_cast<float4*>(out + 8 * u) = make_float4(res[u][0], res[u][1], res[u][2], res[u][3]);
}

// ------------------------------------------------------------------------------------------
// dQ of component 2, per query (16 lanes, dims 64 x + 4 l16 + t, in the order of far_position): for every
// retrieved cluster, the summaries of the preceding blocks that were NOT retrieved contribute  dl k-bar  with
// dl = p (dO.v-bar - delta),  p = exp(q~.k-bar + mu-bar - LSE).  The retrieval's share is added here too: bf16 inputs
// have per-pair dq partials, fp32 inputs walk the retrieved keys, kKeys of them requested together.  The sum of
// this and the tile kernel's row (dQff) is added to what the block-diagonal kernel left in dQ.  us, every lane summing every block's product and without far_position's order / now: 4498 / 3996
// at 32 heads of 32k with D = 128, 1235 / 1121 at 16 heads of 64k, 1103 / 981 with 128 x 128 clusters, 111 / 73 at 12 heads of
// 6k, 162 / 120 at 4 fp32 heads of 8k.  (fp32 inputs had both in the tile kernel, a lane pair per query and a key per round trip:
// 384 us at 4 heads of 8k, r = 4, against 44 + 120 for the two kernels now.)
// ------------------------------------------------------------------------------------------
template <typename T, int D, int NBC>
__global__ void __launch_bounds__(256) k_comp2_bwd_dq(
    const T* __restrict__ Q, const T* __restrict__ dO, const float* __restrict__ qc, const T* __restrict__ Ks,
    const T* __restrict__ Vs, const float* __restrict__ L, const int32_t* __restrict__ off_k,
    const float* __restrict__ s_mu, const float* __restrict__ s_k, const T* __restrict__ s_v,
    const int32_t* __restrict__ perm_q, const int32_t* __restrict__ aq,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ slotinfo, const float* __restrict__ dqpart,
    const float* __restrict__ dQff, float* __restrict__ dQ, int h0, int N, int nb, int Bs, int Cq, int Ck, int r, int k2e, int Hq, int Hkv, float scale) {
  constexpr int NG = D / 64;
  constexpr bool kF32 = sizeof(T) == 4;
  const int hl = blockIdx.y, hq = h0 + hl;
  const int l16 = threadIdx.x % 16;
  const int pos = far_position(Bs, nb);
  if (pos < 0) return;
  const int n = perm_q[(size_t)hq * N + pos];
  const size_t qn = (size_t)hq * N + n;
  const int b = pos / Bs, i = aq[qn], NBm = nb - 1;
  const float lse = LSE[qn], dl = delta[qn];
  float qt[NG][4], gt[NG][4], dq[NG][4];
#pragma unroll
  for (int x = 0; x < NG; ++x) {
    float q4[4];
    ld4(Q, qn * D + 64 * x + 4 * l16, q4);
    ld4(dO, qn * D + 64 * x + 4 * l16, gt[x]);
    const float4 c4 = *reinterpret_cast<const float4*>(qc + ((size_t)hq * Cq + i) * D + 64 * x + 4 * l16);
    qt[x][0] = scale * (q4[0] - c4.x); qt[x][1] = scale * (q4[1] - c4.y);
    qt[x][2] = scale * (q4[2] - c4.z); qt[x][3] = scale * (q4[3] - c4.w);
#pragma unroll
    for (int t = 0; t < 4; ++t) dq[x][t] = 0.f;
  }
  const int32_t* si = slotinfo + ((size_t)hq * N + pos) * r;
  const int hk = (hq / Hq) * Hkv + (hq % Hq) / (Hq / Hkv);  // fp32 inputs: the retrieved keys
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const T *Kh = Ks + (size_t)hk * N * D + 4 * l16, *Vh = Vs + (size_t)hk * N * D + 4 * l16;
  const float* Li = L + ((size_t)hl * Cq + i) * N;
  // the tile kernel's row is requested now and used at the end
  float4 oldq[NG];
#pragma unroll
  for (int x = 0; x < NG; ++x) oldq[x] = *reinterpret_cast<const float4*>(dQff + qn * D + 64 * x + 4 * l16);
  // the four queries of a wave are of one block, which bounds the block loops
  // (the bound is a template constant of the loop body below: one straight-line body per value, loads batched)
  const int bwv = __builtin_amdgcn_readfirstlane(b);
  // places in the head's summaries, in units of the lane's share of a row (16 bytes of s_k); 32 bits hold them
  using F4 = Frag<T, 4>;
  const int u8 = l16 & 7;  // the key block (of eight) whose scalars this lane has
  const uint32_t cells = (uint32_t)Cq * Ck, stride = cells * (D / 4);
  const float* kbase = s_k + (size_t)hl * NBm * cells * D;
  const T* vbase = s_v + (size_t)hl * NBm * cells * D;
  const float* mubase = s_mu + (size_t)hl * NBm * cells;
  auto run = [&](auto bw_c) {
  constexpr int bw = decltype(bw_c)::value;
  int next = si[0];  // a slot is read a step ahead of its rows: one round trip per slot
  for (int t = 0; t < r; ++t) {
    const int info = next;
    next = si[t + 1 < r ? t + 1 : t];
    if (info < 0) continue;
    const int j = info & 0xffff;
    const unsigned selbits = (unsigned)info >> 16;
    if constexpr (kF32) {  // component 3: the keys of the retrieved (cluster, block) pairs, with the full query
      for (int bp = 0; bp < b; ++bp) {
        if (!((selbits >> bp) & 1u)) continue;
        const int klo = ok[bp * Ck + j], khi = ok[bp * Ck + j + 1];
        for (int p0 = klo; p0 < khi; p0 += kKeys) {
          float k4[kKeys][NG][4], v4[kKeys][NG][4], lg[kKeys], part[kKeys], dpp[kKeys];
#pragma unroll
          for (int u = 0; u < kKeys; ++u) {
            const int p = min(p0 + u, khi - 1);
            lg[u] = Li[p];
#pragma unroll
            for (int x = 0; x < NG; ++x) {
              ld4(Kh, (size_t)p * D + 64 * x, k4[u][x]);
              ld4(Vh, (size_t)p * D + 64 * x, v4[u][x]);
            }
          }
#pragma unroll
          for (int u = 0; u < kKeys; ++u) {
            part[u] = dpp[u] = 0.f;
#pragma unroll
            for (int x = 0; x < NG; ++x)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                part[u] = fmaf(qt[x][e], k4[u][x][e], part[u]);
                dpp[u] = fmaf(gt[x][e], v4[u][x][e], dpp[u]);
              }
            part[u] = group_sum<16>(part[u]);
            dpp[u] = group_sum<16>(dpp[u]);
          }
#pragma unroll
          for (int u = 0; u < kKeys; ++u) {
            if (p0 + u >= khi) continue;
            const float dlg = __expf(part[u] + lg[u] - lse) * (dpp[u] - dl);  // q.k = q~.k + q-bar.k
#pragma unroll
            for (int x = 0; x < NG; ++x)
#pragma unroll
              for (int e = 0; e < 4; ++e) dq[x][e] = fmaf(dlg, k4[u][x][e], dq[x][e]);
          }
        }
      }
    }
    const unsigned used = ((1u << b) - 1u) & ~selbits;
    if (used == 0u) continue;  // every preceding block is retrieved
    const uint32_t cell0 = (uint32_t)i * Ck + j, at = cell0 * (D / 4) + l16;
#pragma unroll
    for (int c0 = 0; c0 < 8 * NBC; c0 += 8) {
      if (c0 >= bw) break;
      float part[8], dpp[8];
      float4 kr[8][NG];
      typename F4::raw vr[8][NG];
      const float mu = mubase[cell0 + (uint32_t)min(c0 + u8, b - 1) * cells];
      // a retrieved block's rows are not used: rows that are requested anyway, instead of its own (the rows
      // come from the L2, whose rate is half of what bounds this kernel)
      uint32_t pl = at + (uint32_t)(c0 == 0 ? ((used & 1u) || b == 1 ? 0 : 1) : min(c0, b - 1)) * stride;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (c0 + u >= bw) break;
        if (u > 0 && ((used >> (c0 + u)) & 1u)) pl = at + (uint32_t)(c0 + u) * stride;
#pragma unroll
        for (int x = 0; x < NG; ++x) {
          kr[u][x] = *reinterpret_cast<const float4*>(kbase + (size_t)pl * 4 + 64 * x);
          vr[u][x] = F4::ld(vbase + (size_t)pl * 4, 64 * x);
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        part[u] = dpp[u] = 0.f;
        if (c0 + u >= bw) continue;
#pragma unroll
        for (int x = 0; x < NG; ++x) {
          part[u] = fmaf(qt[x][0], kr[u][x].x, part[u]); part[u] = fmaf(qt[x][1], kr[u][x].y, part[u]);
          part[u] = fmaf(qt[x][2], kr[u][x].z, part[u]); part[u] = fmaf(qt[x][3], kr[u][x].w, part[u]);
#pragma unroll
          for (int e = 0; e < 4; ++e) dpp[u] = fmaf(gt[x][e], F4::get(vr[u][x], e), dpp[u]);
        }
      }
      const float sum = sums_to_lanes(part), dp = sums_to_lanes(dpp);
      const bool use = mu > MUSE_NEG_INF && ((used >> (c0 + u8)) & 1u);
      const float dlg = use ? __expf(sum + mu - lse) * (dp - dl) : 0.f;
      [[maybe_unused]] const unsigned uses = kF32 ? lanes_of_8(use) : 0u;
      each_lane<(bw < 8 ? bw : 8)>(dlg, [&](int u, float du) {
        if (kF32 && !((uses >> u) & 1u)) return;
#pragma unroll
        for (int x = 0; x < NG; ++x) {
          dq[x][0] = fmaf(du, kr[u][x].x, dq[x][0]); dq[x][1] = fmaf(du, kr[u][x].y, dq[x][1]);
          dq[x][2] = fmaf(du, kr[u][x].z, dq[x][2]); dq[x][3] = fmaf(du, kr[u][x].w, dq[x][3]);
        }
      });
    }
  }
  };
  if (NBC == 1) {
    switch (bwv) {
      case 1: run(std::integral_constant<int, 1>{}); break;
      case 2: run(std::integral_constant<int, 2>{}); break;
      case 3: run(std::integral_constant<int, 3>{}); break;
      case 4: run(std::integral_constant<int, 4>{}); break;
      case 5: run(std::integral_constant<int, 5>{}); break;
      case 6: run(std::integral_constant<int, 6>{}); break;
      case 7: run(std::integral_constant<int, 7>{}); break;
      default: run(std::integral_constant<int, 8>{}); break;
    }
  } else {
    run(std::integral_constant<int, 8 * NBC>{});
  }
#pragma unroll
  for (int x = 0; x < NG; ++x)
#pragma unroll
    for (int t = 0; t < 4; ++t) dq[x][t] *= scale;
  float4 base[NG];  // what the block-diagonal kernel left
#pragma unroll
  for (int x = 0; x < NG; ++x) base[x] = *reinterpret_cast<const float4*>(dQ + qn * D + 64 * x + 4 * l16);
  // retrieval part, computed per retrieved pair (already scaled); a slot's pair u exists iff its block bit is set
  if (kF32) {
  } else if (k2e == 1) {
    // the usual shape: the partial rows of eight slots are requested together and added in slot order
    for (int t0 = 0; t0 < r; t0 += 8) {
      int inf[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) inf[t] = t0 + t < r ? si[t0 + t] : -1;
      float4 v[8][NG];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const bool ok = inf[t] >= 0 && ((unsigned)inf[t] >> 16) != 0u;
#pragma unroll
        for (int x = 0; x < NG; ++x)
          v[t][x] = ok ? *reinterpret_cast<const float4*>(dqpart + (qn * r + t0 + t) * D + 64 * x + 4 * l16) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int x = 0; x < NG; ++x) { dq[x][0] += v[t][x].x; dq[x][1] += v[t][x].y; dq[x][2] += v[t][x].z; dq[x][3] += v[t][x].w; }
    }
  } else {
    for (int t = 0; t < r; ++t) {
      const int info = si[t];
      if (info < 0 || ((unsigned)info >> 16) == 0u) continue;
      for (int u = 0; u < k2e; ++u) {
        const float* pp = dqpart + (qn * r * k2e + t * k2e + u) * D;
        if (u < (int)__popc((unsigned)info >> 16)) {
#pragma unroll
          for (int x = 0; x < NG; ++x) {
            const float4 v = *reinterpret_cast<const float4*>(pp + 64 * x + 4 * l16);
            dq[x][0] += v.x; dq[x][1] += v.y; dq[x][2] += v.z; dq[x][3] += v.w;
          }
        }
      }
    }
  }
#pragma unroll
  for (int x = 0; x < NG; ++x) {
    float4 o = oldq[x];
    o.x += dq[x][0]; o.y += dq[x][1]; o.z += dq[x][2]; o.w += dq[x][3];
    o.x += base[x].x; o.y += base[x].y; o.z += base[x].z; o.w += base[x].w;
    *reinterpret_cast<float4*>(dQ + qn * D + 64 * x + 4 * l16) = o;
  }
}

// ------------------------------------------------------------------------------------------
// gradients of the accumulated cells (component 1): one wave per (query block b, query cluster i,
// tile of 32 key clusters); loops over the queries of the group.  Writes every cell it owns:
//   g_A_k = sum dl q~,  g_A_v = sum p dO,  g_A_c = sum [dl (1 - q~.kappa) - p dO.vbar]
// ------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(64) k_ff_bwd_cells(
    const T* __restrict__ Q, const T* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ A_mu,
    const float* __restrict__ A_k, const float* __restrict__ A_v, const int32_t* __restrict__ perm_q,
    const int32_t* __restrict__ off_q, const float* __restrict__ LSE, const float* __restrict__ delta,
    const uint32_t* __restrict__ selmask, float* __restrict__ g_A_c, float* __restrict__ g_A_k,
    float* __restrict__ g_A_v, int h0, int N, int nb, int Cq, int Ck, float scale) {
  constexpr int U = D / 8, DT = D / 32;
  __shared__ int ns[32];
  __shared__ float ls[32], ds[32];
  __shared__ uint32_t mws[32];
  const int hl = blockIdx.z, hq = h0 + hl;
  const int NBm = nb - 1;
  const int b = blockIdx.y / Cq + 1, i = blockIdx.y % Cq;
  const int jt = blockIdx.x, j0 = jt * 32;
  const int lane = threadIdx.x, col = lane % 32, half = lane / 32;
  const int W = (Ck + 31) / 32;
  const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1);
  const int qlo = oq[b * Cq + i], qhi = oq[b * Cq + i + 1];
  const size_t acell = (((size_t)hl * NBm + (b - 1)) * Cq + i) * Ck;
  const int jc = j0 + col;
  const bool jvalid = jc < Ck;
  const int jcc = jvalid ? jc : Ck - 1;
  // B operands: this lane's key cluster
  float kt[U][4], vt[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float4 a = *reinterpret_cast<const float4*>(A_k + (acell + jcc) * D + 8 * u + 4 * half);
    float4 c = *reinterpret_cast<const float4*>(A_v + (acell + jcc) * D + 8 * u + 4 * half);
    kt[u][0] = a.x; kt[u][1] = a.y; kt[u][2] = a.z; kt[u][3] = a.w;
    vt[u][0] = c.x; vt[u][1] = c.y; vt[u][2] = c.z; vt[u][3] = c.w;
  }
  const float amu = jvalid ? A_mu[acell + jcc] : MUSE_NEG_INF;
  const float* qci = qc + ((size_t)hq * Cq + i) * D;
  f32x16_t gk[DT], gv[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) { gk[t] = zero16(); gv[t] = zero16(); }
  float csum = 0.f;
  for (int q0 = qlo; q0 < qhi; q0 += 32) {
    __syncthreads();
    if (half == 0) {
      int pos = q0 + col;
      bool ok_ = pos < qhi;
      int n = perm_q[(size_t)hq * N + (ok_ ? pos : q0)];
      ns[col] = n;
      ls[col] = ok_ ? LSE[(size_t)hq * N + n] : __builtin_huge_valf();  // +inf -> p = 0 for padding rows
      ds[col] = delta[(size_t)hq * N + n];
      mws[col] = selmask[((size_t)hq * W + jt) * N + (ok_ ? pos : q0)];
    }
    __syncthreads();
    // A operands (row pattern): this lane's query row
    const size_t qn = (size_t)hq * N + ns[col];
    f32x16_t s = zero16(), dp = zero16();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[4], g[4];
      ld4(Q, qn * D + 8 * u + 4 * half, x);
      ld4(dO, qn * D + 8 * u + 4 * half, g);
      float4 c = *reinterpret_cast<const float4*>(qci + 8 * u + 4 * half);
      s = mfma32(scale * (x[0] - c.x), kt[u][0], s); s = mfma32(scale * (x[1] - c.y), kt[u][1], s);
      s = mfma32(scale * (x[2] - c.z), kt[u][2], s); s = mfma32(scale * (x[3] - c.w), kt[u][3], s);
      dp = mfma32(g[0], vt[u][0], dp); dp = mfma32(g[1], vt[u][1], dp);
      dp = mfma32(g[2], vt[u][2], dp); dp = mfma32(g[3], vt[u][3], dp);
    }
    f32x16_t pr;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      int row = 8 * (e / 4) + 4 * half + (e % 4);
      float p = __expf(s[e] + amu - ls[row]);   // amu = -inf or lse = +inf -> 0
      p = ((mws[row] >> col) & 1u) ? 0.f : p;
      float dlg = p * (dp[e] - ds[row]);
      csum += p > 0.f ? dlg * (1.f - s[e]) - p * dp[e] : 0.f;
      pr[e] = p;
      s[e] = dlg;
    }
    // g_k^T [D x clusters] += q~^T dl,  g_v^T += dO^T p  (column pattern over the query rows)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const size_t rn = (size_t)hq * N + ns[8 * g + 4 * half + t];
#pragma unroll
        for (int x = 0; x < DT; ++x) {
          float qv = scale * (Elem<T>::ld(Q, rn * D + 32 * x + col) - qci[32 * x + col]);
          float gvv = Elem<T>::ld(dO, rn * D + 32 * x + col);
          gk[x] = mfma32(qv, s[4 * g + t], gk[x]);
          gv[x] = mfma32(gvv, pr[4 * g + t], gv[x]);
        }
      }
  }
  csum += __shfl_xor(csum, 32, 64);
  if (!jvalid) return;
  float* ok_ = g_A_k + (acell + jc) * D;
  float* ov_ = g_A_v + (acell + jc) * D;
#pragma unroll
  for (int x = 0; x < DT; ++x)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      int d = 32 * x + 8 * g + 4 * half;
      *reinterpret_cast<float4*>(ok_ + d) = make_float4(gk[x][4 * g], gk[x][4 * g + 1], gk[x][4 * g + 2], gk[x][4 * g + 3]);
      *reinterpret_cast<float4*>(ov_ + d) = make_float4(gv[x][4 * g], gv[x][4 * g + 1], gv[x][4 * g + 2], gv[x][4 * g + 3]);
    }
  if (half == 0) g_A_c[acell + jc] = csum;
}

// ------------------------------------------------------------------------------------------
// Gradients of the per-block cells from those of the accumulated cells, fp32 inputs (bf16: cell_grads.hip): one block of
// 256 threads per (query cluster i, tile of 32 key clusters); wave w owns the 8 chains (i, j, all blocks), j = 32 jt + 8 w + c.  A
// wave is 8 groups of 8 lanes; a lane holds D/8 elements of a row (d = 32 x + 4 l8 + t); group c owns chain c.
// Reverse accumulation over the key blocks a = nb-2 .. 0, in registers:
//      R[a] = gA[a] + exp(Amu[a] - Amu[a+1]) R[a+1],   G[a] = exp(mu[a] - Amu[a]) R[a]   (written out)
// All factors are <= 1.  One owner per cell.  Component 2 is added afterwards by k_chain_grads.
// ------------------------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256) k_cell_grads(
    const float* __restrict__ s_mu, const float* __restrict__ A_mu, const float* __restrict__ g_A_c,
    const float* __restrict__ g_A_k, const float* __restrict__ g_A_v, float* __restrict__ G_c, float* __restrict__ G_k,
    float* __restrict__ G_v, int nb, int Cq, int Ck) {
  constexpr int NV = D / 32;
  using F4 = Frag<float, 4>;
  const int hl = blockIdx.z;
  const int i = blockIdx.y, jt = blockIdx.x;
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, s8 = lane / 8, l8 = lane % 8;
  const int NBm = nb - 1;

  const int jown = jt * 32 + 8 * wave + s8;
  const bool jok = jown < Ck;
  {
    float Rk[NV][4], Rv[NV][4], an = 0.f, rc = 0.f;
#pragma unroll
    for (int x = 0; x < NV; ++x)
#pragma unroll
      for (int t = 0; t < 4; ++t) { Rk[x][t] = 0.f; Rv[x][t] = 0.f; }
    struct Step {
      float Am, mu, gac;
      typename F4::raw gak[NV], gav[NV];
    };
    auto load_step = [&](int a, Step& st) {
      const size_t cell = (((size_t)hl * NBm + a) * Cq + i) * Ck + (jok ? jown : Ck - 1);
      st.Am = A_mu[cell]; st.mu = s_mu[cell]; st.gac = g_A_c[cell];
#pragma unroll
      for (int x = 0; x < NV; ++x) {
        st.gak[x] = F4::ld(g_A_k, cell * D + 32 * x + 4 * l8);
        st.gav[x] = F4::ld(g_A_v, cell * D + 32 * x + 4 * l8);
      }
    };
    // the loads of up to 8 steps are issued together: the recurrence itself is a few multiply-adds per step
    for (int a1 = NBm - 1; a1 >= 0; a1 -= 8) {
      Step st[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (a1 - u >= 0) load_step(a1 - u, st[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int a = a1 - u;
        if (a < 0 || !jok) continue;
        const Step& cur = st[u];
        const size_t cell = (((size_t)hl * NBm + a) * Cq + i) * Ck + jown;
        const float f = (a < NBm - 1 && cur.Am > MUSE_NEG_INF) ? __expf(cur.Am - an) : 0.f;
        const float wgt = cur.mu > MUSE_NEG_INF ? __expf(cur.mu - cur.Am) : 0.f;
        rc = cur.gac + f * rc;
        an = cur.Am;
        if (l8 == 0) G_c[cell] = wgt * rc;
#pragma unroll
        for (int x = 0; x < NV; ++x) {
          float ok4[4], ov4[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            Rk[x][t] = F4::get(cur.gak[x], t) + f * Rk[x][t];
            Rv[x][t] = F4::get(cur.gav[x], t) + f * Rv[x][t];
            ok4[t] = wgt * Rk[x][t];
            ov4[t] = wgt * Rv[x][t];
          }
          st4(G_k, cell * D + 32 * x + 4 * l8, ok4);
          st4(G_v, cell * D + 32 * x + 4 * l8, ov4);
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// summary gradients -> keys and values: one wave per (kv head, key block b', key cluster j); loops
// over the query heads of the group and over tiles of 32 query clusters.
//   W[i,m] = exp(L[i,m] - mu[i]),  T[i,m] = G_c[i] + G_k[i].k_m + G_v[i].v_m
//   dv_m += sum_i W G_v[i],  dk_m += sum_i W G_k[i] + (W T) qbar_i
// ------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(64) k_cells_to_keys(const T* __restrict__ Ks, const T* __restrict__ Vs,
                                                       const float* __restrict__ qc, const float* __restrict__ L,
                                                       const float* __restrict__ s_mu, const float* __restrict__ G_c,
                                                       const float* __restrict__ G_k, const float* __restrict__ G_v,
                                                       const int32_t* __restrict__ off_k, float* __restrict__ dKs,
                                                       float* __restrict__ dVs, int h0, int N, int nb, int Cq, int Ck,
                                                       int Hq, int Hkv, float scale, int frozen) {
  constexpr int U = D / 8, DT = D / 32;
  const int G_ = Hq / Hkv;
  const int hkl = blockIdx.z;                 // kv head inside the chunk
  const int hq0 = h0 + hkl * G_;              // first query head of the group (global flat index)
  const int hk = (hq0 / Hq) * Hkv + (hq0 % Hq) / G_;
  const int bp = blockIdx.y, j = blockIdx.x, NBm = nb - 1;
  const int lane = threadIdx.x, col = lane % 32, half = lane / 32;
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const int klo = ok[bp * Ck + j], khi = ok[bp * Ck + j + 1];
  for (int m0 = klo; m0 < khi; m0 += 32) {
    const int pm = m0 + col;
    const bool mvalid = pm < khi;
    const int pmc = mvalid ? pm : m0;
    // B operands (row pattern): this lane's key
    float kb[U][4], vb[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ld4(Ks, ((size_t)hk * N + pmc) * D + 8 * u + 4 * half, kb[u]);
      ld4(Vs, ((size_t)hk * N + pmc) * D + 8 * u + 4 * half, vb[u]);
    }
    f32x16_t dk[DT], dv[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) { dk[t] = zero16(); dv[t] = zero16(); }
    for (int g = 0; g < G_; ++g) {
      const int hl = hkl * G_ + g, hq = h0 + hl;
      for (int i0 = 0; i0 < Cq; i0 += 32) {
        const int ic = i0 + col < Cq ? i0 + col : Cq - 1;  // A-operand row of this lane
        const size_t cellA = (((size_t)hl * NBm + bp) * Cq + ic) * Ck + j;
        f32x16_t tacc, wv;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          int ir = i0 + 8 * (e / 4) + 4 * half + (e % 4);
          bool iv = ir < Cq;
          int irc = iv ? ir : Cq - 1;
          const size_t cell = (((size_t)hl * NBm + bp) * Cq + irc) * Ck + j;
          tacc[e] = G_c[cell];
          float w = __expf(L[((size_t)hl * Cq + irc) * N + pmc] - s_mu[cell]);
          wv[e] = (iv && mvalid) ? w : 0.f;
        }
        tacc = mfma_rows<D>(tacc, G_k + cellA * D + 4 * half, kb);
        tacc = mfma_rows<D>(tacc, G_v + cellA * D + 4 * half, vb);
        // frozen aggregation weights: nothing flows through W (the T term drops out)
#pragma unroll
        for (int e = 0; e < 16; ++e) tacc[e] = (wv[e] > 0.f && !frozen) ? wv[e] * tacc[e] : 0.f;
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            int ir = i0 + 8 * gg + 4 * half + t;
            ir = ir < Cq ? ir : Cq - 1;
            const size_t cell = (((size_t)hl * NBm + bp) * Cq + ir) * Ck + j;
#pragma unroll
            for (int x = 0; x < DT; ++x) {
              float gkv = G_k[cell * D + 32 * x + col];
              float gvv = G_v[cell * D + 32 * x + col];
              float qb = scale * qc[((size_t)hq * Cq + ir) * D + 32 * x + col];
              dv[x] = mfma32(gvv, wv[4 * gg + t], dv[x]);
              dk[x] = mfma32(gkv, wv[4 * gg + t], dk[x]);
              dk[x] = mfma32(qb, tacc[4 * gg + t], dk[x]);
            }
          }
      }
    }
    if (mvalid) {
      float *ok_ = dKs + ((size_t)hk * N + pm) * D, *ov_ = dVs + ((size_t)hk * N + pm) * D;
#pragma unroll
      for (int x = 0; x < DT; ++x)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          const int d = 32 * x + 8 * gg + 4 * half;
          float4 a = *reinterpret_cast<float4*>(ok_ + d), c = *reinterpret_cast<float4*>(ov_ + d);
          a.x += dk[x][4 * gg]; a.y += dk[x][4 * gg + 1]; a.z += dk[x][4 * gg + 2]; a.w += dk[x][4 * gg + 3];
          c.x += dv[x][4 * gg]; c.y += dv[x][4 * gg + 1]; c.z += dv[x][4 * gg + 2]; c.w += dv[x][4 * gg + 3];
          *reinterpret_cast<float4*>(ok_ + d) = a;
          *reinterpret_cast<float4*>(ov_ + d) = c;
        }
    }
  }
}

// Keys' and values' far-field rows (bucketed) of all blocks but the last, which has none, added to the block diagonal's (in the sequence's order)
__global__ void __launch_bounds__(256) k_scatter_rows(const float* __restrict__ dKs, const float* __restrict__ dVs, const int32_t* __restrict__ perm,
                                                       float* __restrict__ dK, float* __restrict__ dV, int N, int rows, int D) {
  const float* src = blockIdx.z ? dVs : dKs;
  float* dst = blockIdx.z ? dV : dK;
  const int CPR = D / 4;
  const size_t h = blockIdx.y, c = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= (size_t)rows * CPR) return;
  const int p = (int)(c / CPR), cc = (int)(c % CPR);
  float4* o = reinterpret_cast<float4*>(dst + (h * N + perm[h * N + p]) * D) + cc;
  const float4 a = reinterpret_cast<const float4*>(src + (h * N + p) * D)[cc];
  float4 v = *o;
  v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
  *o = v;
}

template <typename T, int D>
int run_bwd_chunk(const MuseDims& d, const T* Q, const T* dO, const float* qc, const int32_t* aq, const float* LSE,
                  FFWorkspace& w, int h0, int hn, hipStream_t sq_, hipStream_t sk_, hipStream_t sdiag, hipEvent_t diag, bool apart) {
  // the far-field part of dQ goes to stream sq_, the cell gradients and what they give to keys and values to
  // stream sk_: the two share inputs only.  Either adds its last kernel's results to what the block-diagonal kernels left, which run on
  // stream sdiag and have ended at the event diag (apart: the keys' and values' stay bucketed, for k_scatter_rows).
  auto behind_diagonal = [&](hipStream_t s) { return s == sdiag ? hipSuccess : hipStreamWaitEvent(s, diag, 0); };
  const int NBm = d.nb - 1;
  const int W = (d.Ck + 31) / 32;
  dim3 gt((d.Bs / 32 + d.Cq + 1 + 7) / 8 * 8, NBm, hn);
  hipStream_t st = sq_;
  if (d.r == 0) MUSE_HIP_CHECK(behind_diagonal(st));
  { MuseProf prof_("k_ff_bwd_dq", st); hipLaunchKernelGGL((k_ff_bwd_dq<T, D>), gt, dim3(64), 0, st, Q, dO, qc, w.A_mu, w.A_k, (const T*)w.A_v, (const bf16_t*)w.A_kb,
                     w.perm_q, w.off_q, w.tile_off, LSE, w.delta, w.selmask, d.r > 0 ? w.dQff : w.dQacc, d.r == 0, h0, d.N, d.nb, d.Cq, d.Ck, d.scale); }
  if (d.r > 0) {
    MUSE_HIP_CHECK(behind_diagonal(st));
    const dim3 g2 = far_grid(d, hn);
    auto go = [&](auto* kernel) {
      MuseProf prof_("k_comp2_bwd_dq", st);
      hipLaunchKernelGGL(kernel, g2, dim3(256), 0, st, Q, dO, qc, (const T*)w.Ks, (const T*)w.Vs, w.L, w.off_k, w.s_mu, w.s_k, (const T*)w.s_v,
                         w.perm_q, aq, LSE, w.delta, w.slotinfo, w.ret_part, w.dQff, w.dQacc, h0, d.N, d.nb, d.Bs, d.Cq, d.Ck, d.r, d.k2e, d.Hq, d.Hkv, d.scale);
    };
    if (d.nb <= 9) go(k_comp2_bwd_dq<T, D, 1>);
    else go(k_comp2_bwd_dq<T, D, 2>);
  }
  st = sk_;
  if constexpr (sizeof(T) == 2) {
    const int rc2 = muse_launch_ff_bwd_cells_mx(d, Q, dO, qc, LSE, w, h0, hn, st);
    if (rc2) return rc2;
  } else {
    { MuseProf prof_("k_ff_bwd_cells", st); hipLaunchKernelGGL((k_ff_bwd_cells<T, D>), dim3(W, NBm * d.Cq, hn), dim3(64), 0, st, Q, dO, qc, w.A_mu, w.A_k, (const float*)w.A_v,
                       w.perm_q, w.off_q, LSE, w.delta, w.selmask, w.g_A_c, w.g_A_k, w.g_A_v, h0, d.N, d.nb, d.Cq, d.Ck,
                       d.scale); }
    { MuseProf prof_("k_cell_grads", st); hipLaunchKernelGGL((k_cell_grads<D>), dim3(W, d.Cq, hn), dim3(256), 0, st, w.s_mu, w.A_mu, w.g_A_c,
                       w.g_A_k, w.g_A_v, w.g_s_c, (float*)w.g_s_k, (float*)w.g_s_v, d.nb, d.Cq, d.Ck); }
  }
  if (d.r > 0) {
    const int rc2 = muse_launch_chain_grads<T>(d, Q, dO, qc, LSE, w, h0, hn, st);
    if (rc2) return rc2;
  }
  const int G_ = d.Hq / d.Hkv;
  if (!apart) MUSE_HIP_CHECK(behind_diagonal(st));
  if (sizeof(T) == 2) {
    int rc2 = muse_launch_cells_to_keys_mx(d, w.Ks, w.Vs, qc, w.qcb, w.L, w.s_mu, w.g_s_c, w.g_s_k, w.g_s_v, w.off_k, w.perm_k, w.dKs, w.dVs, apart ? nullptr : w.dKacc, apart ? nullptr : w.dVacc, h0,
                                           hn, st);
    if (rc2) return rc2;
  } else
  { MuseProf prof_("k_cells_to_keys", st); hipLaunchKernelGGL((k_cells_to_keys<T, D>), dim3(d.Ck, NBm, hn / G_), dim3(64), 0, st, (const T*)w.Ks, (const T*)w.Vs,
                     qc, w.L, w.s_mu, w.g_s_c, (const float*)w.g_s_k, (const float*)w.g_s_v, w.off_k, w.dKs, w.dVs, h0, d.N, d.nb, d.Cq, d.Ck, d.Hq,
                     d.Hkv, d.scale, d.frozen_weights ? 1 : 0); }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

// Whether k_cells_to_keys_mx adds to the block diagonal's gradients itself: it waits for them then, and each of its waves reads and writes two
// more rows a key.  That saves a pass over dK and dV, and pays where its waves fill the device and the rows are many (to 5 % of the backward
// where there is no retrieval, 1 % else); a few long waves lose what runs beside the block diagonal, up to 40 %.  Backward, us, added here / by
// k_scatter_rows behind both streams (1169 sizes: here 2 % slower on average, and slower than scattering every tensor by itself in 143):
//   16 heads of 6.6k, r = 0, 17 x 227          379 / 401        16 of 23k, r = 2, 39 x 81      1546 / 1570     16 of 24k, r = 8, 11 x 169  2261 / 2290
//   8 of 19k, r = 16, 72 x 330                1831 / 1859       32 (16) of 13k, r = 8, 12 x 239 2521 / 2531
//   fewer waves: 2 heads of 63k, r = 0, 58 x 15  871 / 695      64 (16) of 7k, r = 0, 244 x 8  2199 / 1943     8 of 26k, r = 1, 32 x 16      943 / 927
//   fp32: 8 of 30k, D = 128, r = 0, 10 x 788   15790 / 15421    2 of 38k, r = 1, 16 x 238      2500 / 2481     8 of 19k, 222 x 66, r = 1     4797 / 4820
bool keys_add_here(const MuseDims& d) {
  const size_t keys = (size_t)d.B * d.Hkv * (d.N - d.Bs);
  return d.dtype == MUSE_DTYPE_BF16 && (size_t)d.B * d.Hkv * (d.nb - 1) * d.Ck >= 4096 && keys * 2 * d.D * 4 >= 48 << 20;
}

template <typename T>
int run_bwd_typed(const MuseDims& d, const T* Q, const T* K, const T* V, const T* O, const float* LSE, const T* dO,
                  const float* qc, const int32_t* aq, const int32_t* ak, const int32_t* selc, const int32_t* selb,
                  void* dQ, void* dK, void* dV, FFWorkspace& w, hipStream_t st) {
  const int HQ = d.B * d.Hq, HK = d.B * d.Hkv, N = d.N, D = d.D;
  const size_t nq = (size_t)HQ * N, nk = (size_t)HK * N;
  int rc;
  const bool reuse = d.keep_state;  // bucketing, bucketed copies and summaries are still in the workspace
  if (!reuse && (rc = muse_ff_prepare<T>(d, K, V, aq, ak, w, st))) return rc;
  if ((rc = muse_launch_delta(d, O, dO, w.delta, st))) return rc;
  // the block-diagonal backward (matrix-core bound) runs beside the far field (memory bound) on a second
  // stream; it writes the accumulators, to which the far field's last kernels add, or k_scatter_rows behind both
  MuseAux& ax = muse_aux_stream();
  const bool two = ax.state == 1 && !muse_profiling();
  hipStream_t sb = two ? ax.s : st;
  // on every way out after the fork, the caller's stream waits for what the second stream was given
  struct AuxJoin {
    MuseAux& ax; hipStream_t st, sb; bool armed;
    ~AuxJoin() {
      if (armed && hipEventRecord(ax.join, sb) == hipSuccess) (void)hipStreamWaitEvent(st, ax.join, 0);
    }
  } guard{ax, st, sb, false};
  if (two) {
    MUSE_HIP_CHECK(hipEventRecord(ax.fork, st));
    MUSE_HIP_CHECK(hipStreamWaitEvent(sb, ax.fork, 0));
    guard.armed = true;
  }
  if ((rc = muse_launch_attn_bwd(d, d.Bs, Q, K, V, dO, LSE, w.delta, w.dQacc, w.dKacc, w.dVacc, sb))) return rc;
  // With all heads in one chunk the far-field part of dQ follows on the second stream (it needs the selection
  // info and the inverse index, which the first stream builds: event `mid`), beside the cell gradients.
  const bool split = two && w.hc >= HQ, apart = !keys_add_here(d);
  if (two) MUSE_HIP_CHECK(hipEventRecord(ax.join, sb));  // the block-diagonal gradients are there
  {
    FillRanges f;
    f.add(w.dKs, nk * D, 0);
    f.add(w.dVs, nk * D, 0);
    if (d.nb > 1 && d.r == 0) f.add(w.selmask, nq * ((d.Ck + 31) / 32), 0);
    if ((rc = muse_launch_fills(f, st))) return rc;
  }
  if (d.nb > 1) {
    const int W = (d.Ck + 31) / 32;
    if (d.r > 0) {
      { MuseProf prof_("k_selinfo", st); 
        auto go = [&](auto* kernel) { hipLaunchKernelGGL(kernel, dim3((N + 255) / 256, HQ), dim3(256), 0, st, selc, selb, w.perm_q, w.selmask, w.slotinfo, N, d.r, d.k2e, W); };
        if (d.r <= 8) go(k_selinfo<8>);
        else if (d.r <= 16) go(k_selinfo<16>);
        else go(k_selinfo<32>); }
    }
    MUSE_LAUNCH_CHECK();
    if (d.r > 0) {
      // retrieval (component 3): inverse index (kept from the forward when the state is reused), then per pair
      // (the forward of fp32 inputs does without it)
      if (!reuse || sizeof(T) == 4)
        if ((rc = muse_ff_build_inverse_index(d, selc, selb, w, st))) return rc;
      if constexpr (sizeof(T) == 2) {
        if ((rc = muse_launch_c3_pairs(d, Q, dO, LSE, w, st))) return rc;
        if (split) {
          MUSE_HIP_CHECK(hipEventRecord(ax.mid, st));
          MUSE_HIP_CHECK(hipStreamWaitEvent(sb, ax.mid, 0));
        }
        if ((rc = muse_launch_ret_bwd_dq_pairs(d, Q, dO, w.Ks, w.Vs, LSE, w.delta, w.off_k, w.run_off, w.run_map, w.run_cap, w.hits,
                                               w.hit_cap, w.ret_part, split ? sb : st)))
          return rc;
      } else {
        if ((rc = muse_launch_c3_pairs_f32(d, Q, dO, LSE, w, st))) return rc;
      }
    }
    for (int h0 = 0; h0 < HQ; h0 += w.hc) {
      int hn = HQ - h0 < w.hc ? HQ - h0 : w.hc;
      if (!reuse && (rc = muse_ff_summaries<T>(d, qc, w, h0, hn, st))) return rc;
      if (!reuse && (rc = muse_ff_block_summaries<T>(d, selc, w, h0, hn, false, st))) return rc;
      if (split) {  // everything the dQ side reads is now queued on the first stream
        MUSE_HIP_CHECK(hipEventRecord(ax.mid, st));
        MUSE_HIP_CHECK(hipStreamWaitEvent(sb, ax.mid, 0));
      }
      if (D == 64) rc = run_bwd_chunk<T, 64>(d, Q, dO, qc, aq, LSE, w, h0, hn, split ? sb : st, st, sb, ax.join, apart);
      else rc = run_bwd_chunk<T, 128>(d, Q, dO, qc, aq, LSE, w, h0, hn, split ? sb : st, st, sb, ax.join, apart);
      if (rc) return rc;
    }
  }
  if (split) MUSE_HIP_CHECK(hipEventRecord(ax.join, sb));
  if (two) MUSE_HIP_CHECK(hipStreamWaitEvent(st, ax.join, 0));
  guard.armed = false;
  if (apart && d.nb > 1) {
    MuseProf prof_("k_scatter_rows", st);
    const int rows = N - d.Bs;
    hipLaunchKernelGGL(k_scatter_rows, dim3((unsigned)(((size_t)rows * (D / 4) + 255) / 256), HK, 2), dim3(256), 0, st, w.dKs, w.dVs, w.perm_k, w.dKacc,
                       w.dVacc, N, rows, D);
    MUSE_LAUNCH_CHECK();
  }
  if (d.grad_dtype != MUSE_DTYPE_FP32) {
    CastRanges c;
    c.add(w.dQacc, dQ, nq * D);
    c.add(w.dKacc, dK, nk * D);
    c.add(w.dVacc, dV, nk * D);
    if ((rc = muse_launch_casts(c, d.grad_dtype, 1.f, st))) return rc;
  }
  return MUSE_OK;
}

}  // namespace

int muse_run_bwd(const MuseDims& d, const void* Q, const void* K, const void* V, const void* O, const float* LSE,
                 const void* dO, const float* qc, const int32_t* aq, const int32_t* ak, const int32_t* selc,
                 const int32_t* selb, void* dQ, void* dK, void* dV, void* ws, size_t ws_bytes, hipStream_t st) {
  FFWorkspace w;
  if (!muse_ff_carve(d, true, ws, ws_bytes, &w, dQ, dK, dV)) return MUSE_ERR_WORKSPACE_TOO_SMALL;
  if (d.keep_state && w.hc < d.B * d.Hq) return MUSE_ERR_WORKSPACE_TOO_SMALL;
  if (d.dtype == MUSE_DTYPE_FP32)
    return run_bwd_typed<float>(d, (const float*)Q, (const float*)K, (const float*)V, (const float*)O, LSE,
                                (const float*)dO, qc, aq, ak, selc, selb, dQ, dK, dV, w, st);
  return run_bwd_typed<bf16_t>(d, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, LSE,
                               (const bf16_t*)dO, qc, aq, ak, selc, selb, dQ, dK, dV, w, st);
}
