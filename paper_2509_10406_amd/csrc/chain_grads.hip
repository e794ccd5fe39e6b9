// Component 2 of the per-block cell gradients (backward of the monopole attention over the non-retrieved blocks of the
// retrieved clusters): every query of cluster i in a later block that retrieved cluster j but not block a adds
//   g_k += dl q~,  g_v += p dO,  g_c += dl (1 - q~.kbar) - p dO.vbar
// to the row of cell (a, i, j) that component 1 wrote (k_ff_bwd_cells_mx; fp32 inputs: k_cell_grads).
//
// For a chain (i, j) that is an attention-backward block of the chain's queries e against its key blocks a, and it
// runs on the matrix cores: S[e, a] and dP[e, a] from the gathered rows as they are loaded, then
// G^T[d, a] += Q^T[d, e] dl[e, a] with the rows read back transposed from LDS.  Nothing is rounded on the way: for
// bf16 inputs the queries' and gradients' bf16 rows are operands as they are, every fp32 factor (k-bar, p, dl) is
// split into three bf16 terms (24 significant bits, exact products, fp32 sums), and the query centroid's share of q~
// leaves the products as scalars per cell; fp32 inputs use fp32 MFMA.
//
// One workgroup of 4 waves per (head, query cluster i, word of 32 key clusters, every S-th bit of it).  It lists the
// queries of all its retrieved chains at once, a chunk of the cluster's queries at a time: a ballot per chain over the
// selection-mask words gives every query its place, so the lists are in bucketed order without an atomic, every sum
// has a fixed order and a cell one owner.  Then a wave takes two chains at a time (up to 8 key blocks: the 16 columns
// of the matrix instructions; one chain beyond that), whose summaries and first queries' rows are one round trip to
// memory.  With fewer such groups than waves, the waves share a group's tiles and add up through LDS.
//
// A query with an infinity or NaN in its rows (its LSE or delta is not finite then) is kept out of the lists: in a tile it
// would reach the cells that it does not use, those of later blocks among them, as 0 * inf.  k_chain_odd adds its share.
//
// Bound by the scattered rows of the chains' cells (s_k, s_v read, G_k, G_v read and written, 640 to 1280 bytes per cell)
// and their latency where chains have few queries, by the gathered query rows where they have many.  A workgroup per
// (head, query cluster) on the vector units, as this was before, left small problems to a few workgroups: 1.64 -> 0.09 ms
// at 12 heads of 6k tokens with 23 x 71 clusters, 3.86 -> 0.76 ms at 16 heads of 64k tokens with 128 x 128 clusters,
// 2.8 -> 2.3 ms there with 256 x 1024, 8.2 -> 6.1 ms at D = 128 (32 heads of 32k, 128 x 512, r = 16).
#include "ff_common.h"
#include "fp32_sum.h"
#include "lds_tile.h"

namespace {

__device__ __forceinline__ bool both_finite(float a, float b) { return fabsf(a) < __builtin_huge_valf() && fabsf(b) < __builtin_huge_valf(); }

__device__ __forceinline__ void split3(float x, __bf16& hi, __bf16& mid, __bf16& lo) {
  hi = (__bf16)x;
  const float r = x - (float)hi;
  mid = (__bf16)r;
  lo = (__bf16)(r - (float)mid);
}

constexpr int kListCap = 4096;  // listed (query, chain) entries of a chunk
constexpr int kChunk = 512;     // queries of a chunk

template <typename T, int D, int P>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? (D == 64 ? 3 : 2) : (D == 64 ? 2 : 1), D == 64 ? 3 : 2))) k_chain_grads(
    const T* __restrict__ Q, const T* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ s_mu,
    const float* __restrict__ s_k, const T* __restrict__ s_v, const int32_t* __restrict__ perm_q,
    const int32_t* __restrict__ off_q, const float* __restrict__ LSE, const float* __restrict__ delta,
    const uint32_t* __restrict__ selmask, const int32_t* __restrict__ slotinfo, const uint32_t* __restrict__ chainmask,
    float* __restrict__ G_c, T* __restrict__ G_k, T* __restrict__ G_v, int h0, int N, int nb, int Cq, int Ck, int r,
    int S, uint32_t pattern, float scale) {
  constexpr bool kH = sizeof(T) == 2;
  constexpr int ET = 16, PAD = kH ? 8 : 4;  // queries per tile; padding of its LDS rows
  constexpr int MT = D / 16, KS = D / 32;
  constexpr int NA = 16 / P;                // columns (key blocks) of a chain
  using F4 = Frag<T, 4>;
  __shared__ __attribute__((aligned(16))) T rows[4][2][ET][D + PAD];
  __shared__ __attribute__((aligned(16))) float2 tsc[4][ET];    // (LSE, delta) of a tile's queries
  __shared__ __attribute__((aligned(16))) uint32_t tum[4][ET];  // the columns they add to
  __shared__ uint32_t list[kListCap];                           // staged query << 16 | key blocks it adds to
  __shared__ uint32_t nS[kChunk];                               // position | block << 22
  __shared__ float2 ldS[kChunk];                                // (LSE, delta)
  __shared__ unsigned long long balS[32 * 8];                   // [chain][64-query group]: the lanes of its queries
  __shared__ int startS[32 * 8 + 1];                            // first list entry of (chain, group)
  __shared__ int bitS[32];                                      // bit of the k-th retrieved chain of the word
  __shared__ int cum[18], seg[17];  // cum[b] = queries of the cluster in blocks 1 .. b-1; first bucketed position in b
  __shared__ float red[4][2][64];
  static_assert(sizeof(rows[0]) >= MT * 4 * 64 * 4, "one of a wave's two accumulators fits its row tiles");

  // all workgroups of a query cluster on one XCD (x % 8; the grid's x extent is a multiple of 8): its L2 keeps the rows
  const int W = (Ck + 31) / 32, per = W * S;
  const int i = blockIdx.x % 8 + 8 * (blockIdx.x / 8 / per), jt = blockIdx.x / 8 % per / S, sub = blockIdx.x / 8 % per % S;
  if (i >= Cq) return;
  const int hl = blockIdx.y, hq = h0 + hl, NBm = nb - 1;
  const uint32_t word = chainmask[((size_t)hl * Cq + i) * W + jt] & (pattern << sub);
  if (!word) return;
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, c16 = lane % 16, g = lane / 16;
  const int nact = __popc(word), ng = (nact + P - 1) / P;
  const int wpc = ng == 1 ? 4 : ng == 2 ? 2 : 1, part_w = wave % wpc;  // waves per group of chains
  const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1);
  if (tid == 0) {
    int run = 0;
    cum[0] = 0;
    cum[1] = 0;
    for (int b = 1; b < nb; ++b) {
      const int lo = oq[b * Cq + i];
      seg[b] = lo;
      run += oq[b * Cq + i + 1] - lo;
      cum[b + 1] = run;
    }
  }
  if (tid < 32 && ((word >> tid) & 1u)) bitS[__popc(word & ((1u << tid) - 1u))] = tid;
  __syncthreads();
  const int Tq = cum[nb];
  const float* qci = qc + ((size_t)hq * Cq + i) * D;
  T (*qrow)[D + PAD] = rows[wave][0];
  T (*grow)[D + PAD] = rows[wave][1];
  const int per_chunk = kListCap / (r < 32 ? r : 32) < kChunk ? kListCap / (r < 32 ? r : 32) : kChunk;
  const unsigned long long below = (1ull << lane) - 1ull;

  for (int c0 = 0; c0 < Tq; c0 += per_chunk) {
    const int nq = Tq - c0 < per_chunk ? Tq - c0 : per_chunk;
    __syncthreads();  // the previous chunk is consumed
    // ---- the chunk's lists ----
    uint32_t w2[2] = {0u, 0u};
    int p2[2], b2[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const int t = tid + 256 * z, idx = c0 + t;
      p2[z] = 0; b2[z] = 1;
      if (t < nq) {
        int b = 1;
        while (idx >= cum[b + 1]) ++b;
        b2[z] = b;
        p2[z] = seg[b] + idx - cum[b];
        w2[z] = selmask[((size_t)hq * W + jt) * N + p2[z]] & word;
      }
    }
    int n2[2];
    float2 ld2[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) n2[z] = w2[z] ? perm_q[(size_t)hq * N + p2[z]] : 0;
#pragma unroll
    for (int z = 0; z < 2; ++z) ld2[z] = make_float2(LSE[(size_t)hq * N + n2[z]], delta[(size_t)hq * N + n2[z]]);
#pragma unroll
    for (int z = 0; z < 2; ++z) w2[z] = both_finite(ld2[z].x, ld2[z].y) ? w2[z] : 0u;
    {
      int k = 0;
      for (uint32_t rest = word; rest; rest &= rest - 1, ++k) {
        const int bit = __ffs((int)rest) - 1;
        const unsigned long long b0 = __ballot((w2[0] >> bit) & 1u), b1 = __ballot((w2[1] >> bit) & 1u);
        if (lane == 0) { balS[8 * k + wave] = b0; balS[8 * k + 4 + wave] = b1; }
      }
    }
#pragma unroll
    for (int z = 0; z < 2; ++z)
      if (w2[z]) {
        nS[tid + 256 * z] = (uint32_t)n2[z] | ((uint32_t)b2[z] << 22);
        ldS[tid + 256 * z] = ld2[z];
      }
    __syncthreads();
    if (wave == 0) {
      int cnt[4], mine = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        cnt[u] = 4 * lane + u < 8 * nact ? __popcll(balS[4 * lane + u]) : 0;
        mine += cnt[u];
      }
      int incl = mine;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      int run = incl - mine;
#pragma unroll
      for (int u = 0; u < 4; ++u) { startS[4 * lane + u] = run; run += cnt[u]; }
      if (lane == 63) startS[256] = run;
    }
    __syncthreads();
#pragma unroll
    for (int z = 0; z < 2; ++z)
      if (w2[z]) {
        const int32_t* si = slotinfo + ((size_t)hq * N + p2[z]) * r;
        for (int s0 = 0; s0 < r; s0 += 8) {
          int x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = s0 + u < r ? si[s0 + u] : -1;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int bit = x[u] & 31;
            if (x[u] >= 0 && ((x[u] & 0xffff) >> 5) == jt && ((word >> bit) & 1u)) {
              const int at = 8 * __popc(word & ((1u << bit) - 1u)) + wave + 4 * z;
              list[startS[at] + __popcll(balS[at] & below)] =
                  ((uint32_t)(tid + 256 * z) << 16) | (((1u << b2[z]) - 1u) & ~((uint32_t)x[u] >> 16) & 0xffffu);
            }
          }
        }
      }
    __syncthreads();

    // ---- the chains, P at a time ----
    for (int k0 = P * (wave / wpc); k0 < nact; k0 += P * 4 / wpc) {
      const int ch = c16 / NA, a = c16 % NA;  // this lane's column: chain k0 + ch, key block a
      const bool live = k0 + ch < nact && a < NBm;
      const int j = jt * 32 + bitS[k0 + ch < nact ? k0 + ch : k0];
      const int elo = startS[8 * k0], emid = startS[8 * (k0 + 1)], ehi = k0 + P <= nact ? startS[8 * (k0 + P)] : emid;
      const size_t cell = (((size_t)hl * NBm + (a < NBm ? a : NBm - 1)) * Cq + i) * Ck + j;
      f32x4_t gk[MT], gv[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) { gk[m][t] = 0.f; gv[m][t] = 0.f; }
      float gc = 0.f, dsum = 0.f;
      if (elo + part_w * ET < ehi) {
        // the summaries of the column's cell: dims 32 x + 8 g .. (bf16 operands) or 16 u + 4 g .. (fp32)
        float4 kraw[MT], vrawf[kH ? 1 : MT];
        uint4 vraw[kH ? KS : 1];
        const float mu = s_mu[cell];
        if constexpr (kH) {
#pragma unroll
          for (int x = 0; x < KS; ++x) {
            kraw[2 * x] = *reinterpret_cast<const float4*>(s_k + cell * D + 32 * x + 8 * g);
            kraw[2 * x + 1] = *reinterpret_cast<const float4*>(s_k + cell * D + 32 * x + 8 * g + 4);
            vraw[x] = *reinterpret_cast<const uint4*>(s_v + cell * D + 32 * x + 8 * g);
          }
        } else {
#pragma unroll
          for (int u = 0; u < MT; ++u) {
            kraw[u] = *reinterpret_cast<const float4*>(s_k + cell * D + 16 * u + 4 * g);
            vrawf[u] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(s_v) + cell * D + 16 * u + 4 * g);
          }
        }
        // rows of a tile's queries: query c16, the same dims as the summaries
        uint4 qr[kH ? KS : MT], gr[kH ? KS : MT];
        uint32_t um_next = 0;
        float2 sc_next;
        auto load_tile = [&](int e0) {
          const int e = e0 + c16;
          const uint32_t ent = list[e < ehi ? e : ehi - 1], t = ent >> 16;
          const size_t qn = ((size_t)hq * N + (nS[t] & 0x3fffffu)) * D;
#pragma unroll
          for (int x = 0; x < (kH ? KS : MT); ++x) {
            qr[x] = *reinterpret_cast<const uint4*>(Q + qn + (kH ? 32 * x + 8 * g : 16 * x + 4 * g));
            gr[x] = *reinterpret_cast<const uint4*>(dO + qn + (kH ? 32 * x + 8 * g : 16 * x + 4 * g));
          }
          um_next = e < ehi ? (P == 2 && e >= emid ? (ent & 0xffu) << 8 : ent & 0xffffu) : 0u;
          sc_next = ldS[t];
        };
        load_tile(elo + part_w * ET);

        bf16x8_t kb[kH ? 3 : 1][kH ? KS : 1];
        float ck = 0.f;  // bf16 inputs: the centroid's share scale * qc_i . k-bar of the scores
        if constexpr (kH) {
#pragma unroll
          for (int x = 0; x < KS; ++x) {
            const float v[8] = {kraw[2 * x].x, kraw[2 * x].y, kraw[2 * x].z, kraw[2 * x].w,
                                kraw[2 * x + 1].x, kraw[2 * x + 1].y, kraw[2 * x + 1].z, kraw[2 * x + 1].w};
            const float4 a4 = *reinterpret_cast<const float4*>(qci + 32 * x + 8 * g), b4 = *reinterpret_cast<const float4*>(qci + 32 * x + 8 * g + 4);
            const float q8[8] = {a4.x, a4.y, a4.z, a4.w, b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              __bf16 hi, mid, lo;
              split3(v[e], hi, mid, lo);
              kb[0][x][e] = hi; kb[1][x][e] = mid; kb[2][x][e] = lo;
              ck = fmaf(q8[e], v[e], ck);
            }
          }
          ck += __shfl_xor(ck, 16, 64);
          ck += __shfl_xor(ck, 32, 64);
          ck *= scale;
        }

        for (int e0 = elo + part_w * ET; e0 < ehi; e0 += ET * wpc) {
          f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
          wave_lds_fence();  // the previous tile's LDS rows are read
          if constexpr (kH) {
#pragma unroll
            for (int x = 0; x < KS; ++x) {
              const bf16x8_t qv = __builtin_bit_cast(bf16x8_t, qr[x]), gvv = __builtin_bit_cast(bf16x8_t, gr[x]);
#pragma unroll
              for (int z = 0; z < 3; ++z) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qv, kb[z][x], s, 0, 0, 0);
              dp = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gvv, __builtin_bit_cast(bf16x8_t, vraw[x]), dp, 0, 0, 0);
              *reinterpret_cast<uint4*>(&qrow[c16][32 * x + 8 * g]) = qr[x];
              *reinterpret_cast<uint4*>(&grow[c16][32 * x + 8 * g]) = gr[x];
            }
          } else {
            FoldSum ss, dps;
#pragma unroll
            for (int x = 0; x < MT; ++x) {
              const float4 c4 = *reinterpret_cast<const float4*>(qci + 16 * x + 4 * g);
              float4 qv = __builtin_bit_cast(float4, qr[x]);
              const float4 gvv = __builtin_bit_cast(float4, gr[x]);
              qv = make_float4(scale * (qv.x - c4.x), scale * (qv.y - c4.y), scale * (qv.z - c4.z), scale * (qv.w - c4.w));
              const float q4[4] = {qv.x, qv.y, qv.z, qv.w}, k4[4] = {kraw[x].x, kraw[x].y, kraw[x].z, kraw[x].w};
              const float g4[4] = {gvv.x, gvv.y, gvv.z, gvv.w}, v4[4] = {vrawf[x].x, vrawf[x].y, vrawf[x].z, vrawf[x].w};
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                ss.add(t, q4[t], k4[t]);
                dps.add(t, g4[t], v4[t]);
              }
              ss.fold(x);
              dps.fold(x);
              *reinterpret_cast<float4*>(&qrow[c16][16 * x + 4 * g]) = qv;
              *reinterpret_cast<float4*>(&grow[c16][16 * x + 4 * g]) = gvv;
            }
            s = ss.total;
            dp = dps.total;
          }
          if (lane < ET) { tsc[wave][lane] = sc_next; tum[wave][lane] = um_next; }
          wave_lds_fence();
          if (e0 + ET * wpc < ehi) load_tile(e0 + ET * wpc);
          // rows 4 g + t of the tile: queries; this lane's column: a cell
          const uint4 um4 = *reinterpret_cast<const uint4*>(&tum[wave][4 * g]);
          const float4 a4 = *reinterpret_cast<const float4*>(&tsc[wave][4 * g]), b4 = *reinterpret_cast<const float4*>(&tsc[wave][4 * g + 2]);
          const uint32_t use[4] = {um4.x, um4.y, um4.z, um4.w};
          const float ls[4] = {a4.x, a4.z, b4.x, b4.z}, de[4] = {a4.y, a4.w, b4.y, b4.w};
          float pr[4], dl[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float sv = kH ? fmaf(scale, s[t], -ck) : s[t];
            pr[t] = ((use[t] >> c16) & 1u) ? __expf(sv + mu - ls[t]) : 0.f;  // an empty cell has mu = -inf: p = 0
            dl[t] = pr[t] * (dp[t] - de[t]);
            gc += dl[t] * (1.f - sv) - pr[t] * dp[t];
            dsum += dl[t];
          }
          if constexpr (kH) {
            s16x4_t pf[3], df[3];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              __bf16 hi, mid, lo;
              split3(pr[t], hi, mid, lo);
              pf[0][t] = __builtin_bit_cast(short, hi); pf[1][t] = __builtin_bit_cast(short, mid); pf[2][t] = __builtin_bit_cast(short, lo);
              split3(dl[t], hi, mid, lo);
              df[0][t] = __builtin_bit_cast(short, hi); df[1][t] = __builtin_bit_cast(short, mid); df[2][t] = __builtin_bit_cast(short, lo);
            }
#pragma unroll
            for (int m = 0; m < MT; ++m) {
              const s16x4_t qa = lds_tr4(reinterpret_cast<const bf16_t*>(&qrow[4 * g + c16 / 4][16 * m + 4 * (c16 % 4)]));
              const s16x4_t ga = lds_tr4(reinterpret_cast<const bf16_t*>(&grow[4 * g + c16 / 4][16 * m + 4 * (c16 % 4)]));
#pragma unroll
              for (int z = 0; z < 3; ++z) {
                gk[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qa, df[z], gk[m], 0, 0, 0);
                gv[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ga, pf[z], gv[m], 0, 0, 0);
              }
            }
          } else {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                gk[m] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)qrow[4 * g + t][16 * m + c16], dl[t], gk[m], 0, 0, 0);
                gv[m] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)grow[4 * g + t][16 * m + c16], pr[t], gv[m], 0, 0, 0);
              }
          }
        }
        gc += __shfl_xor(gc, 16, 64);
        gc += __shfl_xor(gc, 32, 64);
        dsum += __shfl_xor(dsum, 16, 64);
        dsum += __shfl_xor(dsum, 32, 64);
      }
      if (wpc > 1) {  // every wave of the workgroup has one group: its waves' sums are added in wave order
        float* mine = reinterpret_cast<float*>(&rows[wave][0][0][0]) + lane;
        red[wave][0][lane] = gc;
        red[wave][1][lane] = dsum;
        auto gather = [&](f32x4_t(&acc)[MT]) {
          __syncthreads();
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < 4; ++t) mine[64 * (4 * m + t)] = acc[m][t];
          __syncthreads();
          if (part_w == 0)
            for (int o = 1; o < wpc; ++o) {
              const float* oth = reinterpret_cast<const float*>(&rows[wave + o][0][0][0]) + lane;
#pragma unroll
              for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[m][t] += oth[64 * (4 * m + t)];
            }
        };
        gather(gk);
        gather(gv);
        if (part_w == 0)
          for (int o = 1; o < wpc; ++o) { gc += red[wave + o][0][lane]; dsum += red[wave + o][1][lane]; }
      }
      // added to the rows of component 1; a chain's list ascends in the block, so its last query's block bounds the
      // key blocks that received anything
      const int clo = ch == 0 ? elo : emid, chi = ch == 0 ? emid : ehi;
      const int amax = chi > clo ? (int)(nS[list[chi - 1] >> 16] >> 22) : 0;
      if (part_w == 0 && live && a < amax) {
        typename F4::raw ogk[MT], ogv[MT];
        const float ogc = G_c[cell];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          ogk[m] = F4::ld(G_k, cell * D + 16 * m + 4 * g);
          ogv[m] = F4::ld(G_v, cell * D + 16 * m + 4 * g);
        }
        if (g == 0) G_c[cell] = ogc + gc;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          float ok4[4], ov4[4];
          const float4 c4 = *reinterpret_cast<const float4*>(qci + 16 * m + 4 * g);
          const float q4[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            ok4[t] = F4::get(ogk[m], t) + (kH ? scale * fmaf(-dsum, q4[t], gk[m][t]) : gk[m][t]);
            ov4[t] = F4::get(ogv[m], t) + gv[m][t];
          }
          st4(G_k, cell * D + 16 * m + 4 * g, ok4);
          st4(G_v, cell * D + 16 * m + 4 * g, ov4);
        }
      }
    }
  }
}

// The queries that k_chain_grads keeps out, one by one: a workgroup per (head, query cluster) looks through the cluster's LSE
// and delta, and its waves share the chains of a query that is not finite (a chain has one wave: a cell one owner).  A kernel
// of its own, because the registers for it cost k_chain_grads 11 % (16 heads of 64k tokens, 256 x 1024 clusters); where every
// query is finite it takes 50 us there and 8 us at 12 heads of 6k with 23 x 71 clusters.
constexpr int kOddWaves = 16;
template <typename T, int D>
__global__ void __launch_bounds__(64 * kOddWaves) k_chain_odd(
    const T* __restrict__ Q, const T* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ s_mu,
    const float* __restrict__ s_k, const T* __restrict__ s_v, const int32_t* __restrict__ perm_q, const int32_t* __restrict__ off_q,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ slotinfo, float* __restrict__ G_c,
    T* __restrict__ G_k, T* __restrict__ G_v, int h0, int N, int nb, int Cq, int Ck, int r, float scale) {
  constexpr int Z = 4;  // queries per thread and round
  __shared__ unsigned long long odd[Z][kOddWaves];
  __shared__ int cum[65], seg[64];  // as in k_chain_grads
  const int i = blockIdx.x, hl = blockIdx.y, hq = h0 + hl, NBm = nb - 1;
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  const float* qci = qc + ((size_t)hq * Cq + i) * D;
  if (wave == 0) {
    const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1) + i;
    const bool far = lane >= 1 && lane < nb;
    const int lo = far ? oq[lane * Cq] : 0;
    int incl = far ? oq[lane * Cq + 1] - lo : 0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    cum[lane + 1] = incl;
    seg[lane] = lo;
  }
  __syncthreads();
  const int Tq = cum[nb];
  auto block_of = [&](int idx) {
    int b = 1;
    while (idx >= cum[b + 1]) ++b;
    return b;
  };
  for (int c0 = 0; c0 < Tq; c0 += 64 * kOddWaves * Z) {
    bool bad[Z];
#pragma unroll
    for (int z = 0; z < Z; ++z) {
      const int idx = c0 + 64 * kOddWaves * z + threadIdx.x;
      bad[z] = false;
      if (idx < Tq) {
        const int b = block_of(idx);
        const size_t qn = (size_t)hq * N + perm_q[(size_t)hq * N + seg[b] + idx - cum[b]];
        bad[z] = !both_finite(LSE[qn], delta[qn]);
      }
    }
    if (!__syncthreads_or(bad[0] || bad[1] || bad[2] || bad[3])) continue;
#pragma unroll
    for (int z = 0; z < Z; ++z) {
      const unsigned long long m = __ballot(bad[z]);
      if (lane == 0) odd[z][wave] = m;
    }
    __syncthreads();
    for (int w = 0; w < kOddWaves * Z; ++w)
      for (unsigned long long rest = odd[w / kOddWaves][w % kOddWaves]; rest; rest &= rest - 1) {
        const int idx = c0 + 64 * w + __ffsll((long long)rest) - 1, b = block_of(idx);
        const size_t pos = (size_t)hq * N + seg[b] + idx - cum[b], qn = (size_t)hq * N + perm_q[pos];
        for (int t = 0; t < r; ++t) {
          const int x = slotinfo[pos * r + t], j = x & 0xffff;
          if (x < 0 || j % kOddWaves != wave) continue;
          for (int a = 0; a < b; ++a) {
            if (((uint32_t)x >> (16 + a)) & 1u) continue;
            const size_t cell = (((size_t)hl * NBm + a) * Cq + i) * Ck + j;
            float q[D / 64], g[D / 64], sv = 0.f, dp = 0.f;
#pragma unroll
            for (int y = 0; y < D / 64; ++y) {
              const int d = lane + 64 * y;
              q[y] = scale * (Elem<T>::ld(Q, qn * D + d) - qci[d]);
              g[y] = Elem<T>::ld(dO, qn * D + d);
              sv = fmaf(q[y], s_k[cell * D + d], sv);
              dp = fmaf(g[y], Elem<T>::ld(s_v, cell * D + d), dp);
            }
            sv = wave_sum(sv);
            dp = wave_sum(dp);
            const float p = __expf(sv + s_mu[cell] - LSE[qn]), dl = p * (dp - delta[qn]);
#pragma unroll
            for (int y = 0; y < D / 64; ++y) {
              const size_t at = cell * D + lane + 64 * y;
              Elem<T>::st(G_k, at, Elem<T>::ld(G_k, at) + dl * q[y]);
              Elem<T>::st(G_v, at, Elem<T>::ld(G_v, at) + p * g[y]);
            }
            if (lane == 0) G_c[cell] += dl * (1.f - sv) - p * dp;
          }
        }
      }
    __syncthreads();
  }
}

template <typename T, int D>
void launch(const MuseDims& d, const T* Q, const T* dO, const float* qc, const float* LSE, FFWorkspace& w, int h0, int hn,
            hipStream_t st) {
  // S: the chains of a 32-cluster word are spread over S workgroups until the grid can fill the device (a workgroup
  // stages its cluster's queries, so more than that only repeats the staging).  S decides which chains share a wave and how
  // many waves share a chain, and with that the order of the sums: it is taken from all heads of the call, not from the
  // heads of this chunk, so that the bits do not depend on the size of the workspace.
  const int W = (d.Ck + 31) / 32, cq8 = (d.Cq + 7) / 8 * 8;
  int S = 1;
  while (S < 16 && (long long)W * S * d.Cq * d.B * d.Hq < 2048) S *= 2;
  const uint32_t pattern = S == 1 ? 0xffffffffu : S == 2 ? 0x55555555u : S == 4 ? 0x11111111u : S == 8 ? 0x01010101u : 0x00010001u;
  auto go = [&](auto* kernel) { MuseProf prof_("k_chain_grads", st); hipLaunchKernelGGL(kernel, dim3((unsigned)(cq8 * W * S), hn), dim3(256), 0, st, Q, dO, qc, w.s_mu, w.s_k,
                     (const T*)w.s_v, w.perm_q, w.off_q, LSE, w.delta, w.selmask, w.slotinfo, w.chainmask, w.g_s_c,
                     (T*)w.g_s_k, (T*)w.g_s_v, h0, d.N, d.nb, d.Cq, d.Ck, d.r, S, pattern, d.scale); };
  if (d.nb <= 9) go(k_chain_grads<T, D, 2>);
  else go(k_chain_grads<T, D, 1>);
  MuseProf prof_("k_chain_odd", st);
  hipLaunchKernelGGL((k_chain_odd<T, D>), dim3(d.Cq, hn), dim3(64 * kOddWaves), 0, st, Q, dO, qc, w.s_mu, w.s_k, (const T*)w.s_v, w.perm_q,
                     w.off_q, LSE, w.delta, w.slotinfo, w.g_s_c, (T*)w.g_s_k, (T*)w.g_s_v, h0, d.N, d.nb, d.Cq, d.Ck, d.r, d.scale);
}

}  // namespace

template <typename T>
int muse_launch_chain_grads(const MuseDims& d, const T* Q, const T* dO, const float* qc, const float* LSE, FFWorkspace& w,
                            int h0, int hn, hipStream_t st) {
  if (d.D == 64) launch<T, 64>(d, Q, dO, qc, LSE, w, h0, hn, st);
  else launch<T, 128>(d, Q, dO, qc, LSE, w, h0, hn, st);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
template int muse_launch_chain_grads<float>(const MuseDims&, const float*, const float*, const float*, const float*, FFWorkspace&, int, int, hipStream_t);
template int muse_launch_chain_grads<bf16_t>(const MuseDims&, const bf16_t*, const bf16_t*, const float*, const float*, FFWorkspace&, int, int, hipStream_t);
