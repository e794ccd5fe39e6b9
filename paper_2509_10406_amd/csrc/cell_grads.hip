// Gradients of the cells (component 1) for bf16 inputs: the queries of a (block, query cluster i) group against the
// accumulated summaries they saw are a dense attention-backward block with the summaries in the role of keys and values:
//   g_A_k = sum dl q~,  g_A_v = sum p dO,  g_A_c = sum [dl (1 - q~.kbar) - p dO.vbar]
// and an accumulated cell is a sum over the per-block cells before it, so what a per-block cell receives is the reverse
// accumulation over the key blocks a = nb-2 .. 0 (all factors <= 1):
//   R[a] = g_A[a] + exp(Amu[a] - Amu[a+1]) R[a+1],   G[a] = exp(mu[a] - Amu[a]) R[a]   (written out)
// Operands are rounded to bf16 for the matrix cores (gradients only; no selection depends on them); R stays in fp32.
//
// A wave owns one unit of 16 key clusters of one query cluster (v_mfma_f32_16x16x32_bf16, the clusters being the columns)
// and walks the key blocks downwards: the accumulators of the matrix instructions ARE R, decayed by a factor per lane
// between two blocks.  The waves of a workgroup take neighbouring units and share the staged queries of the group (kRows
// at a time, row-major: the rows serve S and dP as they lie and G_k, G_v through transposed reads).  Two stages and the
// next block's summaries in flight, so a block costs one barrier.
//
// Bound at D = 64 by vector instructions (0.67 of the busy cycles at 16 heads of 64k tokens, 256 x 1024 and 128 x 128 clusters: 32
// queries per group on average, so a stage is often half empty, and both its halves of 16 rows are always worked through) beside
// the summaries in and the gradients out, 16.0 GB there: 3.1 to 3.3 ms, the copy rate.  At D = 128 (32 heads of 32k, 128 x 512) by
// that traffic, 5.4 TB/s, with the vector pipe 0.42 busy.  With the reverse accumulation as a launch of its own the gradients of the accumulated cells
// took a round trip through HBM in 16 bits: 3.25 + 3.37 ms there, 2.88 + 3.36 (now 2.89) at 32 heads of 32k, D = 128, 128 x 512,
// 0.44 + 0.17 (now 0.30) at 16 heads of 64k with 128 x 128.
#include "ff_common.h"
#include "lds_tile.h"

namespace {

// Three waves per SIMD at D = 64, two at D = 128 (registers).  Units per workgroup: ms at 16 heads of 64k tokens, D = 64,
// 256 x 1024 clusters with 2 / 4 / 8 waves 3.87 / 3.13 / 4.48 (a third workgroup of 8 does not fit); at 32 heads of 32k, D = 128,
// 128 x 512 clusters 5.46 / 3.46 / 2.89.  Stages of 64 queries in place of 32: 4.32 and 3.62.
//
// APART: few units leave the chip to a chain of nb - 1 blocks, whose stages are round trips of 1 to 2 us.  The waves of a workgroup
// then share one unit and take a key block each, with their own staged queries; what they have summed up goes from wave to wave
// through LDS, later blocks first, R = own + f R as above.  The lines between the two are in cells_apart.
template <int D, bool APART>
struct CellCfg {
  static constexpr int kWaves = D == 64 && !APART ? 4 : 8;    // units of a workgroup; APART: key blocks at a time
  static constexpr int kRows = 32;                            // queries staged at a time
  static constexpr int kOcc = D == 64 && !APART ? 3 : 2;      // waves per SIMD
};

template <int D, bool APART>
__global__ void __launch_bounds__((64 * CellCfg<D, APART>::kWaves)) __attribute__((amdgpu_waves_per_eu(CellCfg<D, APART>::kOcc, CellCfg<D, APART>::kOcc))) k_ff_bwd_cells_mx(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ dO, const float* __restrict__ qc,
    const float* __restrict__ s_mu, const float* __restrict__ A_mu, const bf16_t* __restrict__ A_kb,
    const bf16_t* __restrict__ A_v, const int32_t* __restrict__ perm_q, const int32_t* __restrict__ off_q,
    const float* __restrict__ LSE, const float* __restrict__ delta, const uint32_t* __restrict__ selmask,
    float* __restrict__ G_c, bf16_t* __restrict__ G_k, bf16_t* __restrict__ G_v, int h0, int N, int nb, int Cq, int Ck,
    float scale) {
  using Cfg = CellCfg<D, APART>;
  constexpr int KX = D / 32, MT = D / 16, CPR = D / 8, NW = Cfg::kWaves, RP = Cfg::kRows, NT = APART ? 64 : 64 * NW;
  constexpr int NU = RP * CPR / NT;   // 16-byte chunks of a tensor per thread and stage
  constexpr int NBUF = APART ? NW : 2, STEP = APART ? NW : 1;
  __shared__ __attribute__((aligned(16))) bf16_t qs[NBUF][RP * D];
  __shared__ __attribute__((aligned(16))) bf16_t gs[NBUF][RP * D];
  __shared__ __attribute__((aligned(16))) float ls[NBUF][RP];
  __shared__ __attribute__((aligned(16))) float ds[NBUF][RP];
  __shared__ __attribute__((aligned(16))) uint32_t mws[NW][RP];
  __shared__ __attribute__((aligned(16))) bf16_t tws[APART ? 1 : NW][16][D + 8];
  __shared__ __attribute__((aligned(16))) f32x4_t carry[APART ? 2 * MT : 1][64];  // APART: R of the block handed on, as the lanes hold it
  __shared__ float2 carry_c[64];                                                 // and its scalar part with Amu
  __shared__ __attribute__((aligned(16))) float cs[D];
  __shared__ int2 grp[16];  // [a]: positions of the group that sees the accumulation up to key block a
  const int hl = blockIdx.z, hq = h0 + hl;
  const int NBm = nb - 1, W = (Ck + 31) / 32, nunit = (Ck + 15) / 16, ng = APART ? nunit : (nunit + NW - 1) / NW;
  // the workgroups of one query cluster run on one XCD (x % 8), one after the other: they stage the same queries (APART: on all,
  // there are few)
  const int xcd = blockIdx.x % 8, idx = APART ? blockIdx.x : blockIdx.x / 8;
  const int i = APART ? idx / ng : idx / ng * 8 + xcd;
  if (i >= Cq) return;
  const int wave = APART ? __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : threadIdx.x / 64, lane = threadIdx.x % 64, c16 = lane % 16, g = lane / 16;
  const int unit = APART ? idx % ng : idx % ng * NW + wave;
  const bool live = unit < nunit;  // the last workgroup's waves may have nothing but the staging to do
  const int jc = unit * 16 + c16, jcl = min(jc, Ck - 1), bit = 16 * (unit & 1) + c16;
  const bool jvalid = jc < Ck;
  const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1);
  const int32_t* pq = perm_q + (size_t)hq * N;
  const bf16_t *Qh = Q + (size_t)hq * N * D, *Gh = dO + (size_t)hq * N * D;
  const float *Lh = LSE + (size_t)hq * N, *Dh = delta + (size_t)hq * N;
  const int stid = APART ? lane : (int)threadIdx.x;  // the thread's number among those that stage a group's queries
  bf16_t(*tw)[D + 8] = APART ? reinterpret_cast<bf16_t(*)[D + 8]>(qs[wave]) : tws[wave];  // the rows on their way out
  const uint32_t* sm = selmask + ((size_t)hq * W + min(unit / 2, W - 1)) * N;
  if (threadIdx.x < NBm) grp[threadIdx.x] = make_int2(oq[(threadIdx.x + 1) * Cq + i], oq[(threadIdx.x + 1) * Cq + i + 1]);
  if (threadIdx.x < D) cs[threadIdx.x] = qc[((size_t)hq * Cq + i) * D + threadIdx.x];
  __syncthreads();

  struct CT {  // the unit's accumulated summaries as this lane's operands (cluster c16, dims 32 x + 8 g ..)
    bf16x8_t kf[KX], vf[KX];
    float amu, mu;  // raw: any arithmetic on a prefetched value would wait for the whole prefetch at once
  };
  auto cell_at = [&](int a) { return (((size_t)hl * NBm + a) * Cq + i) * Ck; };
  auto load_ct = [&](int a, CT& c) {
    const size_t cell = cell_at(a);
    const bf16_t *kb = A_kb + cell * D, *vb = A_v + cell * D;  // uniform; the lane's offset takes 32 bits
    const uint32_t o = (uint32_t)(jcl * D + 8 * g);
#pragma unroll
    for (int x = 0; x < KX; ++x) {
      c.kf[x] = *reinterpret_cast<const bf16x8_t*>(kb + (o + 32 * x));
      c.vf[x] = *reinterpret_cast<const bf16x8_t*>(vb + (o + 32 * x));
    }
    c.amu = (A_mu + cell)[(uint32_t)jcl];
    c.mu = (s_mu + cell)[(uint32_t)jcl];
  };
  // The stages in order: (a, q0), the queries q0 .. of the group of key block a; an empty group is one stage of no rows.
  struct Cur { int a, q0, hi; };
  auto advance = [&](Cur c) {  // past the end: the last stage again
    c.q0 += RP;
    if (c.q0 >= c.hi && c.a >= STEP) {
      c.a -= STEP;
      const int2 gr = grp[c.a];
      c.q0 = __builtin_amdgcn_readfirstlane(gr.x);
      c.hi = __builtin_amdgcn_readfirstlane(gr.y);
    }
    return c;
  };
  // a row past the group's end repeats its first one (weight 0); an empty group's are never used
  auto pos_of = [&](const Cur& c, int row) { return min(c.q0 + row < c.hi ? c.q0 + row : c.q0, N - 1); };
  // sequence positions of this thread's rows, one stage ahead of the rows (APART: of row lane, handed out by shuffles)
  constexpr int NP = APART ? 1 : NU;
  int pos[NP];
  typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
  u4_t rq[NU], rg[NU];  // its chunks of a stage on their way
  float rl[NP], rd[NP];
  uint32_t rm;
  auto load_pos = [&](const Cur& c) {
#pragma unroll
    for (int u = 0; u < NP; ++u) pos[u] = pq[pos_of(c, APART ? lane % RP : (stid + NT * u) / CPR)];
  };
  auto load_rows = [&](const Cur& c) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int p = APART ? __shfl(pos[0], (stid + NT * u) / CPR, 64) : pos[APART ? 0 : u];
      const uint32_t o = (uint32_t)(p * D + (stid + NT * u) % CPR * 8);
      rq[u] = *reinterpret_cast<const u4_t*>(Qh + o);
      rg[u] = *reinterpret_cast<const u4_t*>(Gh + o);
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      rl[u] = Lh[(uint32_t)pos[u]];
      rd[u] = Dh[(uint32_t)pos[u]];
    }
    rm = sm[pos_of(c, lane % RP)];
  };
  auto commit = [&](const Cur& c, int buf) {
    int tid = stid;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = tid + NT * u, row = t / CPR, cc = t % CPR;
      const float4 c0 = *reinterpret_cast<const float4*>(cs + cc * 8), c1 = *reinterpret_cast<const float4*>(cs + cc * 8 + 4);
      auto two = [&](uint32_t w, float x, float y) {
        return pack_bf16x2(scale * (__uint_as_float(w << 16) - x), scale * (__uint_as_float(w & 0xffff0000u) - y));
      };
      *reinterpret_cast<uint4*>(qs[buf] + tile_at<D>(row, cc)) =
          make_uint4(two(rq[u].x, c0.x, c0.y), two(rq[u].y, c0.z, c0.w), two(rq[u].z, c1.x, c1.y), two(rq[u].w, c1.z, c1.w));
      *reinterpret_cast<u4_t*>(gs[buf] + tile_at<D>(row, cc)) = rg[u];
      if (!APART && cc == 0) {
        ls[buf][row] = c.q0 + row < c.hi ? rl[APART ? 0 : u] * 1.4426950408889634f : __builtin_huge_valf();  // +inf -> p = 0 for padding rows
        ds[buf][row] = rd[APART ? 0 : u];
      }
    }
    if (APART && lane < RP) {
      ls[buf][lane] = c.q0 + lane < c.hi ? rl[0] * 1.4426950408889634f : __builtin_huge_valf();
      ds[buf][lane] = rd[0];
    }
    if (lane < RP) mws[wave][lane] = rm;
  };

  f32x4_t gk[MT], gv[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < 4; ++t) { gk[m][t] = 0.f; gv[m][t] = 0.f; }
  float rc = 0.f, an = 0.f;
  CT cur, nxt;
  Cur here, ahead;  // the stage whose rows are committed next, and the one behind it
  {
    const int a = max(NBm - 1 - (APART ? wave : 0), 0);
    const int2 gr = grp[a];
    here = {a, __builtin_amdgcn_readfirstlane(gr.x), __builtin_amdgcn_readfirstlane(gr.y)};
  }
  load_pos(here);
  if constexpr (!APART) load_ct(here.a, nxt);
  load_rows(here);
  ahead = advance(here);
  load_pos(ahead);
  int buf = APART ? wave : 0;
  for (int top = NBm - 1; top >= 0; top -= STEP) {
    const int a = APART ? top - wave : top;
    const bool mine = !APART || a >= 0;
    float csum = 0.f, amu2 = 0.f;
    if (APART && mine) load_ct(a, cur);
    for (bool first = true; mine; first = false) {
      commit(here, buf);
      if constexpr (APART) wave_lds_fence();
      else __syncthreads();
      const int nrow = here.hi - here.q0, ntl = min((nrow + 31) / 32, RP / 32);
      const bool last = nrow <= RP;
      here = ahead;
      load_rows(here);
      ahead = advance(here);
      load_pos(ahead);
      if (first) {
        if constexpr (!APART) {
          cur = nxt;
          load_ct(max(a - 1, 0), nxt);
        }
        const float f = (!APART && a < NBm - 1 && cur.amu > MUSE_NEG_INF) ? __expf(cur.amu - an) : 0.f;
        an = cur.amu;
        amu2 = jvalid ? cur.amu * 1.4426950408889634f : MUSE_NEG_INF;
        rc = APART ? 0.f : rc * f;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            gk[m][t] = APART ? 0.f : gk[m][t] * f;
            gv[m][t] = APART ? 0.f : gv[m][t] * f;
          }
      }
      // LDS offsets are made from the lane number here, not kept in registers over the whole walk
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const int c16 = ln % 16, g = ln / 16;
      for (int qt = 0; live && qt < ntl; ++qt) {
        bf16x8_t pf, df;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int r0 = 32 * qt + 16 * u;
          f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int x = 0; x < KX; ++x) {
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_row<D>(qs[buf], r0 + c16, 4 * x + g), cur.kf[x], s, 0, 0, 0);
            dp = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_row<D>(gs[buf], r0 + c16, 4 * x + g), cur.vf[x], dp, 0, 0, 0);
          }
          const float4 l4 = *reinterpret_cast<const float4*>(&ls[buf][r0 + 4 * g]), d4 = *reinterpret_cast<const float4*>(&ds[buf][r0 + 4 * g]);
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
          const bf16x8_t ag = tr_join(tile_tr4<D>(gs[buf], rr, 16 * m + cc), tile_tr4<D>(gs[buf], rr + 16, 16 * m + cc));
          gv[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag, pf, gv[m], 0, 0, 0);
          const bf16x8_t aq = tr_join(tile_tr4<D>(qs[buf], rr, 16 * m + cc), tile_tr4<D>(qs[buf], rr + 16, 16 * m + cc));
          gk[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, df, gk[m], 0, 0, 0);
        }
      }
      if constexpr (!APART) buf ^= 1;
      if (last) break;
      wave_lds_fence();  // the next stage rewrites this wave's mask words (APART: and its rows)
    }
    csum += __shfl_xor(csum, 16, 64);
    csum += __shfl_xor(csum, 32, 64);
    rc += csum;
    if constexpr (APART) {
      for (int w = 0; w < min(NW, top + 1); ++w) {
        if (w == wave) {
          if (a < NBm - 1) {
            const float2 in = carry_c[lane];
            const float f = cur.amu > MUSE_NEG_INF ? __expf(cur.amu - in.y) : 0.f;
            rc = fmaf(f, in.x, rc);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
              const f32x4_t k4 = carry[m][lane], v4 = carry[MT + m][lane];
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                gk[m][t] = fmaf(f, k4[t], gk[m][t]);
                gv[m][t] = fmaf(f, v4[t], gv[m][t]);
              }
            }
          }
          carry_c[lane] = make_float2(rc, cur.amu);
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            carry[m][lane] = gk[m];
            carry[MT + m][lane] = gv[m];
          }
        }
        __syncthreads();
      }
    }
    if (!live || !mine) continue;
    const float wgt = cur.mu > MUSE_NEG_INF ? __expf(cur.mu - cur.amu) : 0.f;
    const size_t cell = cell_at(a);
    // rows go out through a per-wave LDS tile: a store instruction then writes 64 / (D/8) whole rows of consecutive
    // clusters (contiguous memory)
#pragma unroll
    for (int arr = 0; arr < 2; ++arr) {
      wave_lds_fence();
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const f32x4_t& r = arr == 0 ? gk[m] : gv[m];
        *reinterpret_cast<uint2*>(&tw[c16][16 * m + 4 * g]) = make_uint2(pack_bf16x2(wgt * r[0], wgt * r[1]), pack_bf16x2(wgt * r[2], wgt * r[3]));
      }
      wave_lds_fence();
      bf16_t* dst = arr == 0 ? G_k : G_v;
#pragma unroll
      for (int it = 0; it < 16 * CPR / 64; ++it) {
        const int row = it * (64 / CPR) + lane / CPR, cc = lane % CPR;
        if (unit * 16 + row < Ck) {
          const u4_t v = *reinterpret_cast<const u4_t*>(&tw[row][cc * 8]);
          __builtin_nontemporal_store(v, reinterpret_cast<u4_t*>(dst + (cell + unit * 16 + row) * D + cc * 8));  // written once, read by later kernels
        }
      }
    }
    if (jvalid && g == 0) G_c[cell + jc] = wgt * rc;
  }
}

// Key blocks side by side (APART) for few units, counted once for every round of eight key blocks, and enough key blocks to share out.
// By the heads of the call, not of a chunk: the bits do not depend on the workspace.  us, one after the other / side by side, 8
// blocks unless said:
//   units   D = 64: 227 / 60 at one head of 16k with 4 x 8 clusters (4 units), 278 / 70 at 4 of 8k with 1 x 512 (128), 87 / 43 at one of
//           32k with 64 x 128 (512), 99 / 66 at 16 of 16k with 32 x 32 (1024), 84 / 103 at 2 of 64k with 128 x 128 (2048), 134 / 210 at
//           16 of 32k with 64 x 64 (4096); D = 128: 195 / 86, 411 / 125, 165 / 60, 166 / 132, 153 / 182 and 245 / 360
//   blocks  D = 64: 44 / 70 with 2, 39 / 26 with 3, 82 / 68 with 4; D = 128: 48 / 56 with 3, 129 / 135 with 4; with 12
//           (two rounds) at 1024 units 74 / 72 and 103 / 133, with 16 at 512 97 / 51 and 139 / 101
static bool cells_apart(const MuseDims& d, int nunit) {
  const int rounds = (d.nb - 1 + 7) / 8;
  return d.nb - 1 >= (d.D == 64 ? 2 : 4) && (long long)d.B * d.Hq * d.Cq * nunit * rounds <= 1024;
}

}  // namespace

int muse_launch_ff_bwd_cells_mx(const MuseDims& d, const void* Q, const void* dO, const float* qc, const float* LSE,
                                FFWorkspace& w, int h0, int hn, hipStream_t st) {
  const int nunit = (d.Ck + 15) / 16;
  const bool apart = cells_apart(d, nunit);
  auto go = [&](auto* kernel, int waves) {
    MuseProf prof_("k_ff_bwd_cells_mx", st);
    const int ng = apart ? nunit : (nunit + waves - 1) / waves;
    hipLaunchKernelGGL(kernel, dim3((apart ? d.Cq : (d.Cq + 7) / 8 * 8) * ng, 1, hn), dim3(64 * waves), 0, st, (const bf16_t*)Q, (const bf16_t*)dO,
                       qc, w.s_mu, w.A_mu, (const bf16_t*)w.A_kb, (const bf16_t*)w.A_v, w.perm_q, w.off_q, LSE, w.delta,
                       w.selmask, w.g_s_c, (bf16_t*)w.g_s_k, (bf16_t*)w.g_s_v, h0, d.N, d.nb, d.Cq, d.Ck, d.scale);
  };
  if (d.D == 64) apart ? go(k_ff_bwd_cells_mx<64, true>, CellCfg<64, true>::kWaves) : go(k_ff_bwd_cells_mx<64, false>, CellCfg<64, false>::kWaves);
  else apart ? go(k_ff_bwd_cells_mx<128, true>, CellCfg<128, true>::kWaves) : go(k_ff_bwd_cells_mx<128, false>, CellCfg<128, false>::kWaves);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
