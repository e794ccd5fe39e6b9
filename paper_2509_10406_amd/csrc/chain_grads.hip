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
// bf16 inputs: k_chain_lists sorts the (query, slot) entries of a query cluster by key cluster, once for all its chains, and
// k_chain_grads takes them P chains at a time (up to 8 key blocks: the 16 columns of the matrix instructions are two chains;
// one chain beyond that).  fp32 inputs (k_chain_grads_f32; the lists' places in the workspace hold something else there): one workgroup
// of 4 waves per (head, query cluster i, word of 32 key clusters, every S-th bit of it) lists the queries of all its retrieved chains at
// once, a chunk of the cluster's queries at a time: a ballot per chain over the selection-mask words gives every query its
// place.  Either way the lists' order comes from ballots, not from atomics, every sum has a fixed order and a cell one owner; and with
// fewer groups of chains than waves, the waves share a group's tiles and add up through LDS.
//
// A query with an infinity or NaN in its rows (its LSE or delta is not finite then) is kept out of the lists: in a tile it
// would reach the cells that it does not use, those of later blocks among them, as 0 * inf.  k_chain_odd adds its share.
//
// Bound by the scattered rows of the chains' cells (s_k, s_v read, G_k, G_v read and written, 640 to 1280 bytes per cell)
// where chains have few queries, by the gathered query rows where they have many.  us of all launches, bf16 inputs, with the lists made by
// every word's workgroup (whose preparation, a dozen round trips for three to four chains, took most of the time) and rows in
// pieces of 32 and 64 bytes / now (lists + gradients): 2590 / 126 + 894 at 16 heads of 64k with 256 x 1024 clusters, 790 / 80 + 485 there
// with 128 x 128, 8180 / 177 + 4459 at 32 heads of 64k with rotary rows (five times as many chains; 2630 without the read, addition and
// write of G, with the writes in pieces), 6160 / 166 + 3340 at 32 of 32k with D = 128, 144 / 25 + 77 at 8 of 16k with 64 x 256,
// 108 / 23 + 84 at 12 of 6k with 23 x 71.  With four waves per SIMD at D = 64 and three at D = 128 the registers spill: twice the time.
#include <algorithm>
#include <type_traits>

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

template <int D, int P>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1, D == 64 ? 3 : 2))) k_chain_grads_f32(
    const float* __restrict__ Q, const float* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ s_mu,
    const float* __restrict__ s_k, const float* __restrict__ s_v, const int32_t* __restrict__ perm_q,
    const int32_t* __restrict__ off_q, const float* __restrict__ LSE, const float* __restrict__ delta,
    const uint32_t* __restrict__ selmask, const int32_t* __restrict__ slotinfo, const uint32_t* __restrict__ chainmask,
    float* __restrict__ G_c, float* __restrict__ G_k, float* __restrict__ G_v, int h0, int N, int nb, int Cq, int Ck, int r,
    int S, uint32_t pattern, float scale) {
  constexpr int ET = 16, PAD = 4;  // queries per tile; padding of its LDS rows
  constexpr int MT = D / 16;
  constexpr int NA = 16 / P;                // columns (key blocks) of a chain
  using F4 = Frag<float, 4>;
  __shared__ __attribute__((aligned(16))) float rows[4][2][ET][D + PAD];
  __shared__ __attribute__((aligned(16))) float2 tsc[4][ET];    // (LSE, delta) of a tile's queries
  __shared__ __attribute__((aligned(16))) uint32_t tum[4][ET];  // the columns they add to
  __shared__ uint32_t list[kListCap];                           // staged query << 16 | key blocks it adds to
  __shared__ uint32_t nS[kChunk];                               // position | block << 22
  __shared__ float2 ldS[kChunk];                                // (LSE, delta)
  __shared__ unsigned long long balS[32 * 8];                   // [chain][64-query group]: the lanes of its queries
  __shared__ int startS[32 * 8 + 1];                            // first list entry of (chain, group)
  __shared__ int bitS[32];                                      // bit of the k-th retrieved chain of the word
  __shared__ int cum[18], seg[17];  // cum[b] = queries of the cluster in blocks 1 .. b-1; first bucketed position in b
  __shared__ float red[4][64];
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
  float (*qrow)[D + PAD] = rows[wave][0];
  float (*grow)[D + PAD] = rows[wave][1];
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
      float gc = 0.f;
      if (elo + part_w * ET < ehi) {
        // the summaries of the column's cell: dims 16 u + 4 g ..
        float4 kraw[MT], vraw[MT];
        const float mu = s_mu[cell];
#pragma unroll
        for (int u = 0; u < MT; ++u) {
          kraw[u] = *reinterpret_cast<const float4*>(s_k + cell * D + 16 * u + 4 * g);
          vraw[u] = *reinterpret_cast<const float4*>(s_v + cell * D + 16 * u + 4 * g);
        }
        // rows of a tile's queries: query c16, the same dims as the summaries
        uint4 qr[MT], gr[MT];
        uint32_t um_next = 0;
        float2 sc_next;
        auto load_tile = [&](int e0) {
          const int e = e0 + c16;
          const uint32_t ent = list[e < ehi ? e : ehi - 1], t = ent >> 16;
          const size_t qn = ((size_t)hq * N + (nS[t] & 0x3fffffu)) * D;
#pragma unroll
          for (int x = 0; x < MT; ++x) {
            qr[x] = *reinterpret_cast<const uint4*>(Q + qn + 16 * x + 4 * g);
            gr[x] = *reinterpret_cast<const uint4*>(dO + qn + 16 * x + 4 * g);
          }
          um_next = e < ehi ? (P == 2 && e >= emid ? (ent & 0xffu) << 8 : ent & 0xffffu) : 0u;
          sc_next = ldS[t];
        };
        load_tile(elo + part_w * ET);

        for (int e0 = elo + part_w * ET; e0 < ehi; e0 += ET * wpc) {
          f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
          wave_lds_fence();  // the previous tile's LDS rows are read
            FoldSum ss, dps;
#pragma unroll
            for (int x = 0; x < MT; ++x) {
              const float4 c4 = *reinterpret_cast<const float4*>(qci + 16 * x + 4 * g);
              float4 qv = __builtin_bit_cast(float4, qr[x]);
              const float4 gvv = __builtin_bit_cast(float4, gr[x]);
              qv = make_float4(scale * (qv.x - c4.x), scale * (qv.y - c4.y), scale * (qv.z - c4.z), scale * (qv.w - c4.w));
              const float q4[4] = {qv.x, qv.y, qv.z, qv.w}, k4[4] = {kraw[x].x, kraw[x].y, kraw[x].z, kraw[x].w};
              const float g4[4] = {gvv.x, gvv.y, gvv.z, gvv.w}, v4[4] = {vraw[x].x, vraw[x].y, vraw[x].z, vraw[x].w};
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
            const float sv = s[t];
            pr[t] = ((use[t] >> c16) & 1u) ? __expf(sv + mu - ls[t]) : 0.f;  // an empty cell has mu = -inf: p = 0
            dl[t] = pr[t] * (dp[t] - de[t]);
            gc += dl[t] * (1.f - sv) - pr[t] * dp[t];
          }
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                gk[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(qrow[4 * g + t][16 * m + c16], dl[t], gk[m], 0, 0, 0);
                gv[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(grow[4 * g + t][16 * m + c16], pr[t], gv[m], 0, 0, 0);
              }
        }
        gc += __shfl_xor(gc, 16, 64);
        gc += __shfl_xor(gc, 32, 64);
      }
      if (wpc > 1) {  // every wave of the workgroup has one group: its waves' sums are added in wave order
        float* mine = reinterpret_cast<float*>(&rows[wave][0][0][0]) + lane;
        red[wave][lane] = gc;
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
          for (int o = 1; o < wpc; ++o) gc += red[wave + o][lane];
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
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            ok4[t] = F4::get(ogk[m], t) + gk[m][t];
            ov4[t] = F4::get(ogv[m], t) + gv[m][t];
          }
          st4(G_k, cell * D + 16 * m + 4 * g, ok4);
          st4(G_v, cell * D + 16 * m + 4 * g, ov4);
        }
      }
    }
  }
}

// ---- bf16 inputs ----
// The listed queries of every chain, by (head, query cluster i): a workgroup sorts its cluster's (query, slot) entries by key
// cluster.  A wave takes a range of the queries, 64 at a time and slot by slot; the lanes of one chain are found by ballots over
// the bits of its number and ranked by lane (no atomic decides an order), its waves' shares lie one behind the other.
//   chains [head][..]: (j | the last block of its queries << 16, first entry) of the cluster's chains, ascending j, and (0, entries);
//                      cluster i's begin at head_of[head][i].y + i
//   lists  [head][..]: (position, key blocks the query adds to), from head_of[head][i].y
//   head_of [head][i]: (chains, and bit 16 where a query is not finite; first entry)
// 16 bytes of every lane from its p to LDS at at + 16 lane (rows_to_lds with a 64-bit address)
__device__ __forceinline__ void far_rows_to_lds(uint32_t at, const void* p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(p) : "memory");
}
// what is read from LDS is in registers, and its place may be written
__device__ __forceinline__ void lds_read() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

constexpr int kListWaves = 16;  // most waves of a workgroup
// BITS >= the bits of a cluster's number; V4: r is a multiple of 4
template <bool V4, int BITS>
__global__ void __launch_bounds__(64 * kListWaves) k_chain_lists(
    const int32_t* __restrict__ perm_q, const int32_t* __restrict__ off_q, const float* __restrict__ LSE,
    const float* __restrict__ delta, const int32_t* __restrict__ slotinfo, uint2* __restrict__ chains, uint2* __restrict__ lists,
    int2* __restrict__ head_of, int h0, int N, int Bs, int nb, int Cq, int Ck, int r) {
  const int NW = blockDim.x / 64;
  extern __shared__ int cnt[];  // [wave][Ck] entries, then the next place; [Ck] the last block
  int* lastb = cnt + NW * Ck;
  __shared__ int cum[65], seg[64], first;  // cum[b] = queries of the cluster in blocks 1 .. b-1; first bucketed position in b
  __shared__ int2 part[kListWaves];
  const int i = blockIdx.x, hq = h0 + blockIdx.y, tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  for (int t = tid; t < (NW + 1) * Ck; t += 64 * NW) cnt[t] = 0;
  if (wave == 0) {
    const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1) + i;
    const bool far = lane >= 1 && lane < nb;
    const int lo = far ? oq[lane * Cq] : 0;
    int incl = far ? oq[lane * Cq + 1] - lo : 0, before = far ? lo - lane * Bs : 0;  // (at most 16 blocks)
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
      before += __shfl_xor(before, o, 64);
    }
    cum[lane + 1] = incl;
    seg[lane] = lo;
    if (lane == 0) first = before * r;
  }
  __syncthreads();
  const int Tq = __builtin_amdgcn_readfirstlane(cum[nb]), per = (Tq + 64 * NW - 1) / (64 * NW) * 64;
  const int qlo = wave * per, qhi = min(qlo + per, Tq);
  const size_t hn = (size_t)hq * N;
  bool odd = false;
  const unsigned long long below = (1ull << lane) - 1ull;
  // f(cluster or -1, lanes of the same cluster, position, key blocks the query adds to, block) for every slot of the wave's
  // queries, 64 of them at a time
  int x[8], n = 0, b = 0;
  bool finite = true;
  const bool held = per == 64 && r <= 8;  // the second time these are here
  auto walk = [&](bool again, auto f) {
    for (int q0 = qlo; q0 < qhi; q0 += 64) {
      const int idx = min(q0 + lane, qhi - 1);
      if (!again || !held) {
        b = 1;
#pragma unroll
        for (int z = 2; z < 16; ++z) b += idx >= cum[z];  // (cum of a block there is not: all queries)
      }
      const size_t p = hn + seg[b] + idx - cum[b];
      const int32_t* si = slotinfo + p * r;
      auto load = [&](int s0) {
        if constexpr (V4) {
#pragma unroll
          for (int u = 0; u < 8; u += 4) {
            const int4 v = s0 + u < r ? *reinterpret_cast<const int4*>(si + s0 + u) : make_int4(-1, -1, -1, -1);
            x[u] = v.x; x[u + 1] = v.y; x[u + 2] = v.z; x[u + 3] = v.w;
          }
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = s0 + u < r ? si[s0 + u] : -1;
        }
      };
      if (!again || !held) {
        n = perm_q[p];
        load(0);
        finite = both_finite(LSE[hn + n], delta[hn + n]);
        odd |= !finite;
      }
      const bool ok = finite && q0 + lane < qhi;
      for (int s0 = 0; s0 < r; s0 += 8) {
        int y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = x[u];
        if (s0 + 8 < r) load(s0 + 8);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + u < r) {
            const int j = ok && y[u] >= 0 ? y[u] & 0xffff : -1;
            unsigned long long m = __ballot(j >= 0);
#pragma unroll
            for (int z = 0; z < BITS; ++z) {
              const bool one = (j >> z) & 1;
              const unsigned long long ones = __ballot(one);
              m &= one ? ones : ~ones;
            }
            f(j, m, n, ((1u << b) - 1u) & ~((uint32_t)y[u] >> 16), b);
          }
      }
    }
  };
  walk(false, [&](int j, unsigned long long m, int, uint32_t, int) {
    if (j >= 0 && !(m & below)) cnt[wave * Ck + j] += __popcll(m);
    wave_lds_fence();
  });
  odd = __syncthreads_or(odd);
  // chains and entries in front of this thread's clusters
  const int step = (Ck + 64 * NW - 1) / (64 * NW), jlo = min(tid * step, Ck), jhi = min(jlo + step, Ck);
  int2 mine = make_int2(0, 0);
  for (int j = jlo; j < jhi; ++j) {
    int n = 0;
#pragma unroll 4
    for (int w = 0; w < NW; ++w) n += cnt[w * Ck + j];
    mine.x += n > 0;
    mine.y += n;
  }
  int2 incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(incl.x, o, 64), y = __shfl_up(incl.y, o, 64);
    if (lane >= o) { incl.x += x; incl.y += y; }
  }
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  int2 run = make_int2(incl.x - mine.x, incl.y - mine.y);
  for (int w = 0; w < wave; ++w) { run.x += part[w].x; run.y += part[w].y; }
  const int2 begin = run;
  for (int j = jlo; j < jhi; ++j)
#pragma unroll 4
    for (int w = 0; w < NW; ++w) {
      const int n = cnt[w * Ck + j];
      cnt[w * Ck + j] = run.y;
      run.y += n;
    }
  __syncthreads();
  uint2* out = lists + hn * r + first;
  walk(true, [&](int j, unsigned long long m, int n, uint32_t mask, int b) {
    if (j >= 0) {
      const int at = cnt[wave * Ck + j], rank = __popcll(m & below);
      out[at + rank] = make_uint2((uint32_t)n, mask);
      if (rank == __popcll(m) - 1) {  // (the last lane's query is in the last block)
        cnt[wave * Ck + j] = at + rank + 1;
        atomicMax(&lastb[j], b);
      }
    }
    wave_lds_fence();  // the place is read by the next slot
  });
  __syncthreads();
  // the last wave's places are the ends
  uint2* tab = chains + (size_t)hq * ((size_t)(N - Bs) * r + Cq) + first + i;
  int k = begin.x, at = begin.y;
  for (int j = jlo; j < jhi; ++j) {
    const int end = cnt[(NW - 1) * Ck + j];
    if (end > at) tab[k++] = make_uint2((uint32_t)j | ((uint32_t)lastb[j] << 16), (uint32_t)at);
    at = end;
  }
  if (tid == 64 * NW - 1) {
    tab[k] = make_uint2(0u, (uint32_t)at);
    head_of[(size_t)hq * Cq + i] = make_int2(k | (odd ? 1 << 16 : 0), first);
  }
}

// S workgroups of one wave or four per (head, query cluster); a wave takes P chains at a time, and where there are fewer such groups than
// waves, the waves of a workgroup share a group.  All rows (s_k, the cells' gradients, the queries') come and go whole, through LDS.
template <int D, int P, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, D == 64 ? 3 : 2))) k_chain_grads(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ s_mu,
    const float* __restrict__ s_k, const bf16_t* __restrict__ s_v, const float* __restrict__ LSE, const float* __restrict__ delta,
    const uint2* __restrict__ chains, const uint2* __restrict__ lists, const int2* __restrict__ head_of, float* __restrict__ G_c,
    bf16_t* __restrict__ G_k, bf16_t* __restrict__ G_v, int h0, int N, int Bs, int nb, int Cq, int Ck, int r, int S, int share, float scale) {
  constexpr int ET = 16;  // queries per tile
  constexpr int MT = D / 16, KS = D / 32, CPR = D / 8, RPL = 64 / CPR, NIT = ET / RPL;  // rows per load instruction
  constexpr int NA = 16 / P;  // columns (key blocks) of a chain
  __shared__ __attribute__((aligned(16))) bf16_t tile[NW][2][ET * D];   // rows of a tile's queries, of their gradients
  __shared__ __attribute__((aligned(16))) bf16_t cells[NW][2][ET * D];  // s_k of the columns' cells (fp32), then their gradients
  __shared__ __attribute__((aligned(16))) float2 tsc[NW][ET];    // (LSE, delta) of a tile's queries
  __shared__ __attribute__((aligned(16))) uint32_t tum[NW][ET];  // the columns they add to
  __shared__ float red[NW][2][64];
  static_assert(sizeof(tile[0]) >= MT * 4 * 64 * 4, "one of a wave's two accumulators fits its row tiles");

  // all workgroups of a query cluster on one XCD (x % 8; the grid's x extent is a multiple of 8): its L2 keeps the rows
  const int i = blockIdx.x % 8 + 8 * (blockIdx.x / 8 / S), sub = blockIdx.x / 8 % S;
  if (i >= Cq) return;
  const int hl = blockIdx.y, hq = h0 + hl, NBm = nb - 1;
  const int2 head = head_of[(size_t)hq * Cq + i];
  const int nch = head.x & 0xffff, ng = (nch + P - 1) / P;
  const int wpc = NW == 1 ? 1 : ng <= share ? 4 : ng <= 2 * share ? 2 : 1;  // waves per group of chains
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), part_w = wave % wpc;
  const uint2* tab = chains + (size_t)hq * ((size_t)(N - Bs) * r + Cq) + head.y + i;
  const uint2* ents = lists + (size_t)hq * N * r + head.y;
  const float* qci = qc + ((size_t)hq * Cq + i) * D;
  const size_t hn = (size_t)hq * N;
  const bf16_t *Qh = Q + hn * D, *gOh = dO + hn * D;
  const float *Lh = LSE + hn, *dh = delta + hn;
  const size_t cell0 = ((size_t)hl * NBm * Cq + i) * Ck;  // cell (a, i, j) is cell0 + a Cq Ck + j
  const uint32_t ablock = (uint32_t)Cq * Ck;
  bf16_t *qt = tile[wave][0], *gt = tile[wave][1], *ck_ = cells[wave][0], *cv_ = cells[wave][1];
  const uint32_t cat = __builtin_amdgcn_readfirstlane(lds_addr(ck_));

  for (int g0 = sub * (NW / wpc); g0 < ng; g0 += S * (NW / wpc)) {
    // made anew for every group: as invariants, places in LDS and elements of the centroid would fill the registers
    int lane = threadIdx.x % 64;
    asm volatile("" : "+v"(lane));
    const int c16 = lane % 16, g = lane / 16;  // this lane's column: chain c16 / NA of the group, key block c16 % NA
    const int k0 = P * (g0 + wave / wpc);
    const uint2 t0 = tab[min(k0, nch)], t1 = tab[min(k0 + 1, nch)], t2 = P == 2 ? tab[min(k0 + 2, nch)] : t1;
    const int elo = t0.y, emid = t1.y, ehi = t2.y;
    // the key blocks in front of a chain's last query are the cells that received anything
    const int j0 = t0.x & 0xffff, am0 = k0 < nch ? min((int)(t0.x >> 16), NBm) : 0;
    const int j1 = P == 2 && k0 + 1 < nch ? t1.x & 0xffff : j0, am1 = P == 2 && k0 + 1 < nch ? min((int)(t1.x >> 16), NBm) : 0;
    // cell of a column (one that received nothing: the chain's first) and whether it received anything
    auto cell_of = [&](int c) {
      const int x = c % NA;
      return (x < (c < NA ? am0 : am1) ? (uint32_t)x * ablock : 0u) + (uint32_t)(c < NA ? j0 : j1);
    };
    auto live_of = [&](int c) { return c % NA < (c < NA ? am0 : am1); };
    const size_t cell = cell0 + cell_of(c16);
    const bool live = live_of(c16);
    f32x4_t gk[MT], gv[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < 4; ++t) { gk[m][t] = 0.f; gv[m][t] = 0.f; }
    float gc = 0.f, dsum = 0.f, ogc = 0.f;
    if (elo + part_w * ET < ehi) {
      // rows of a tile's queries, whole rows per load instruction
      bf16x8_t qr[NIT], gr[NIT];
      uint32_t um_next = 0;
      float2 sc_next;
      uint2 ent = ents[min(elo + part_w * ET + c16, ehi - 1)];
      auto load_tile = [&](int e0) {
        const int e = e0 + c16;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const uint32_t o = (uint32_t)__shfl((int)ent.x, it * RPL + lane / CPR, 16) * D + lane % CPR * 8;
          qr[it] = *reinterpret_cast<const bf16x8_t*>(Qh + o);
          gr[it] = *reinterpret_cast<const bf16x8_t*>(gOh + o);
        }
        sc_next = make_float2(Lh[ent.x], dh[ent.x]);
        um_next = e < ehi ? (P == 2 && e >= emid ? (ent.y & 0xffu) << 8 : ent.y & 0xffffu) : 0u;
        ent = ents[min(e + ET * wpc, ehi - 1)];
      };
      // the summaries of the columns' cells; a chunk of 16 bytes of s_k lies at its place xor the row
      lds_read();
#pragma unroll
      for (int it = 0; it < 2 * NIT; ++it) {
        const int row = it * (RPL / 2) + lane / (2 * CPR), chunk = (lane % (2 * CPR)) ^ row;
        far_rows_to_lds(cat + 1024 * it, reinterpret_cast<const char*>(s_k) + (cell0 + cell_of(row)) * D * 4 + chunk * 16);
      }
      const float mu = s_mu[cell];
      bf16x8_t vb[KS];
#pragma unroll
      for (int x = 0; x < KS; ++x) vb[x] = *reinterpret_cast<const bf16x8_t*>(s_v + cell * D + 32 * x + 8 * g);
      if (part_w == 0) ogc = G_c[cell];
      load_tile(elo + part_w * ET);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      wave_lds_fence();

      bf16x8_t kb[3][KS];
      float ck = 0.f;  // the centroid's share scale * qc_i . k-bar of the scores
#pragma unroll
      for (int x = 0; x < KS; ++x) {
        const float* krow = reinterpret_cast<const float*>(ck_) + c16 * D;
        const float4 k0_ = *reinterpret_cast<const float4*>(krow + 4 * ((8 * x + 2 * g) ^ c16)), k1_ = *reinterpret_cast<const float4*>(krow + 4 * ((8 * x + 2 * g + 1) ^ c16));
        const float v[8] = {k0_.x, k0_.y, k0_.z, k0_.w, k1_.x, k1_.y, k1_.z, k1_.w};
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
      // the gradients of the cells, on their way during the tiles
      lds_read();
      if (part_w == 0) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int row = it * RPL + lane / CPR;
          const size_t o = (cell0 + cell_of(row)) * D * 2 + (tile_at<D>(row, lane % CPR) - row * D) * 2;
          far_rows_to_lds(cat + 1024 * it, reinterpret_cast<const char*>(G_k) + o);
          far_rows_to_lds(cat + ET * D * 2 + 1024 * it, reinterpret_cast<const char*>(G_v) + o);
        }
      }

      for (int e0 = elo + part_w * ET; e0 < ehi; e0 += ET * wpc) {
        f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
        wave_lds_fence();  // the previous tile's LDS rows are read
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int at = tile_at<D>(it * RPL + lane / CPR, lane % CPR);
          *reinterpret_cast<bf16x8_t*>(qt + at) = qr[it];
          *reinterpret_cast<bf16x8_t*>(gt + at) = gr[it];
        }
        if (lane < ET) { tsc[wave][lane] = sc_next; tum[wave][lane] = um_next; }
        wave_lds_fence();
        if (e0 + ET * wpc < ehi) load_tile(e0 + ET * wpc);
#pragma unroll
        for (int x = 0; x < KS; ++x) {
          const bf16x8_t qv = tile_row<D>(qt, c16, 4 * x + g);
#pragma unroll
          for (int z = 0; z < 3; ++z) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qv, kb[z][x], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_row<D>(gt, c16, 4 * x + g), vb[x], dp, 0, 0, 0);
        }
        // rows 4 g + t of the tile: queries; this lane's column: a cell
        const uint4 um4 = *reinterpret_cast<const uint4*>(&tum[wave][4 * g]);
        const float4 a4 = *reinterpret_cast<const float4*>(&tsc[wave][4 * g]), b4 = *reinterpret_cast<const float4*>(&tsc[wave][4 * g + 2]);
        const uint32_t use[4] = {um4.x, um4.y, um4.z, um4.w};
        const float ls[4] = {a4.x, a4.z, b4.x, b4.z}, de[4] = {a4.y, a4.w, b4.y, b4.w};
        float pr[4], dl[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float sv = fmaf(scale, s[t], -ck);
          pr[t] = ((use[t] >> c16) & 1u) ? __expf(sv + mu - ls[t]) : 0.f;  // an empty cell has mu = -inf: p = 0
          dl[t] = pr[t] * (dp[t] - de[t]);
          gc += dl[t] * (1.f - sv) - pr[t] * dp[t];
          dsum += dl[t];
        }
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
          const s16x4_t qa = tile_tr4<D>(qt, 4 * g + c16 / 4, 16 * m + 4 * (c16 % 4));
          const s16x4_t ga = tile_tr4<D>(gt, 4 * g + c16 / 4, 16 * m + 4 * (c16 % 4));
#pragma unroll
          for (int z = 0; z < 3; ++z) {
            gk[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qa, df[z], gk[m], 0, 0, 0);
            gv[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ga, pf[z], gv[m], 0, 0, 0);
          }
        }
      }
      gc += __shfl_xor(gc, 16, 64);
      gc += __shfl_xor(gc, 32, 64);
      dsum += __shfl_xor(dsum, 16, 64);
      dsum += __shfl_xor(dsum, 32, 64);
    }
    if (NW > 1 && wpc > 1) {  // every wave of the workgroup has one group at most: its waves' sums are added in wave order
      float* mine = reinterpret_cast<float*>(qt) + lane;
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
            const float* oth = reinterpret_cast<const float*>(tile[wave + o][0]) + lane;
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
    if (part_w != 0 || elo >= ehi) continue;
    // added to the rows of component 1
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_lds_fence();
    if (g == 0 && live) G_c[cell] = ogc + gc;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const float4 c4 = *reinterpret_cast<const float4*>(qci + 16 * m + 4 * g);
      const float q4[4] = {c4.x, c4.y, c4.z, c4.w};
      const int at = tile_at<D>(c16, 2 * m + g / 2) + 4 * (g % 2);
      float ok4[4], ov4[4];
      ld4(ck_, at, ok4);
      ld4(cv_, at, ov4);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        ok4[t] += scale * fmaf(-dsum, q4[t], gk[m][t]);
        ov4[t] += gv[m][t];
      }
      st4(ck_, at, ok4);
      st4(cv_, at, ov4);
    }
    wave_lds_fence();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int row = it * RPL + lane / CPR, at = tile_at<D>(row, lane % CPR);
      const size_t o = (cell0 + cell_of(row)) * D + lane % CPR * 8;
      const bf16x8_t wk = *reinterpret_cast<const bf16x8_t*>(ck_ + at), wv = *reinterpret_cast<const bf16x8_t*>(cv_ + at);
      if (live_of(row)) {
        *reinterpret_cast<bf16x8_t*>(G_k + o) = wk;
        *reinterpret_cast<bf16x8_t*>(G_v + o) = wv;
      }
    }
  }
}

// The queries that k_chain_grads keeps out, one by one: a workgroup per (head, query cluster) looks through the cluster's LSE
// and delta, and its waves share the chains of a query that is not finite (a chain has one wave: a cell one owner).  A kernel
// of its own, because the registers for it cost k_chain_grads 11 % (16 heads of 64k tokens, 256 x 1024 clusters); where every
// query is finite, it ends at the flag that the lists were left (bf16 inputs: 10 us there, 5 at 12 heads of 6k with 23 x 71 clusters) or reads LSE
// and delta (fp32 inputs).
constexpr int kOddWaves = 16;
template <typename T, int D>
__global__ void __launch_bounds__(64 * kOddWaves) k_chain_odd(
    const T* __restrict__ Q, const T* __restrict__ dO, const float* __restrict__ qc, const float* __restrict__ s_mu,
    const float* __restrict__ s_k, const T* __restrict__ s_v, const int32_t* __restrict__ perm_q, const int32_t* __restrict__ off_q,
    const float* __restrict__ LSE, const float* __restrict__ delta, const int32_t* __restrict__ slotinfo, float* __restrict__ G_c,
    T* __restrict__ G_k, T* __restrict__ G_v, const int2* __restrict__ head_of, int h0, int N, int nb, int Cq, int Ck, int r, float scale) {
  if (head_of && !(head_of[(size_t)(h0 + blockIdx.y) * Cq + blockIdx.x].x >> 16)) return;  // the lists were made without seeing one
  constexpr int Z = 4;  // queries per thread and round
  __shared__ unsigned long long odd[Z][kOddWaves];
  __shared__ int cum[65], seg[64];  // as in k_chain_lists
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
int launch(const MuseDims& d, const T* Q, const T* dO, const float* qc, const float* LSE, FFWorkspace& w, int h0, int hn,
           hipStream_t st) {
  const int cq8 = (d.Cq + 7) / 8 * 8;
  const int2* looked = nullptr;
  if constexpr (sizeof(T) == 2) {
    // The waves of a workgroup share a group of chains where a query cluster has no more groups than `share`, with which the grid
    // would just fill the device (it decides the order of the sums: it is taken from all heads of the call, not from the heads of this
    // chunk, so that the bits do not depend on the size of the workspace).  A quarter of the key clusters is enough, but where that leaves a
    // quarter of the device idle, every group may have a workgroup.  us without / with that, where there are few query clusters:
    //   1 head of 64k, 16 x 128       241 / 133     1 of 16k, D = 128, 4 x 256, r = 16   140 / 91     1 of 16k, 8 x 128   36 / 24
    //   1 of 4.6k, D = 128, 3 x 56     90 / 51      2 of 16k, 4 x 64                      90 / 53     1 of 8k, 4 x 256    30 / 22
    // and 26 / 32 for 4 heads of 8.5k with 15 x 112, which fill it without.
    const int groups = d.nb <= 9 ? (d.Ck + 1) / 2 : d.Ck;
    const long long clusters = (long long)d.Cq * d.B * d.Hq;
    int share = 1;
    while (share < (d.Ck + 3) / 4 && share * clusters < 2048) share *= 2;
    while (share < groups && share * clusters < 1536) share *= 2;
    // With enough query clusters a workgroup is one wave, up to 64 of them per cluster: a place is free again as soon as its wave
    // has ended.  us with 1, 4, 16, 64 such workgroups / 1, 4, 16 of four waves:
    //   16 heads of 64k, 256 x 1024   1841, 1080, 916, 891 / 1132, 1002, 1034       12 of 6k, 23 x 71   365, 133, 85, 86 / 136, 93, 90
    //   16 heads of 64k, 128 x 128    1210, 652, 502, 481 / 673, 606, 651           8 of 16k, 64 x 256  479, 175, 86, 77 / 170, 90, 85
    //   32 of 32k, D = 128, 128 x 512 4136, 3437, 3332, 3339 / 3478, 3529, 3700     1 of 16k, 16 x 1024 1308, 368, 128, 59 / 611, 169, 67, shared 34
    // (few query clusters with few chains share theirs: us one / shared 143 / 45 at 2 heads of 8k, D = 128, 16 x 16, 115 / 37 at one of 16k, 8 x 16)
    const bool one = share <= 8 && share * clusters >= 1536;
    const int S = one ? std::min(64, (d.Ck + 1) / 2) : std::max(share, std::min(16, (d.Ck + 7) / 8));
    // waves: most where there are few clusters, else one for 64 of a cluster's queries or two for 256
    const int nw = clusters <= 512 ? kListWaves : d.N / d.Cq > 256 ? 8 : 4;
    const size_t lds = (size_t)(nw + 1) * d.Ck * 4;
    looked = w.head_of;
    const int bits = std::max(5, 32 - __builtin_clz(d.Ck - 1 | 1));
    static_assert(MUSE_MAX_CLUSTERS <= 1 << 11, "bits of a cluster's number");
    auto sort = [&](auto* kernel) -> int {
      if (lds > 64 * 1024) MUSE_HIP_CHECK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (kListWaves + 1) * MUSE_MAX_CLUSTERS * 4));
      MuseProf prof_("k_chain_lists", st);
      hipLaunchKernelGGL(kernel, dim3(d.Cq, hn), dim3(64 * nw), lds, st, w.perm_q, w.off_q, LSE, w.delta, w.slotinfo, w.chains, w.lists, w.head_of, h0, d.N, d.Bs, d.nb,
                         d.Cq, d.Ck, d.r);
      MUSE_LAUNCH_CHECK();
      return MUSE_OK;
    };
    auto sort_v = [&](auto v4) -> int {
      constexpr bool V = decltype(v4)::value;
      switch (bits) {
        case 5: return sort(k_chain_lists<V, 5>);
        case 6: return sort(k_chain_lists<V, 6>);
        case 7: return sort(k_chain_lists<V, 7>);
        case 8: return sort(k_chain_lists<V, 8>);
        case 9: return sort(k_chain_lists<V, 9>);
        case 10: return sort(k_chain_lists<V, 10>);
        default: return sort(k_chain_lists<V, 11>);
      }
    };
    // without the lists the next kernel must not run
    if (const int rc = d.r % 4 == 0 ? sort_v(std::true_type()) : sort_v(std::false_type())) return rc;
    auto go = [&](auto* kernel) { MuseProf prof_("k_chain_grads", st); hipLaunchKernelGGL(kernel, dim3((unsigned)(cq8 * S), hn), dim3(one ? 64 : 256), 0, st, Q, dO, qc, w.s_mu,
                       w.s_k, (const T*)w.s_v, LSE, w.delta, w.chains, w.lists, w.head_of, w.g_s_c, (T*)w.g_s_k, (T*)w.g_s_v, h0, d.N, d.Bs, d.nb, d.Cq, d.Ck,
                       d.r, S, share, d.scale); };
    if (d.nb <= 9) one ? go(k_chain_grads<D, 2, 1>) : go(k_chain_grads<D, 2, 4>);
    else one ? go(k_chain_grads<D, 1, 1>) : go(k_chain_grads<D, 1, 4>);
  } else {
    // S: the chains of a 32-cluster word are spread over S workgroups until the grid can fill the device (a workgroup
    // stages its cluster's queries, so more than that only repeats the staging).  S decides which chains share a wave and how
    // many waves share a chain, and with that the order of the sums: as above.
    const int W = (d.Ck + 31) / 32;
    int S = 1;
    while (S < 16 && (long long)W * S * d.Cq * d.B * d.Hq < 2048) S *= 2;
    const uint32_t pattern = S == 1 ? 0xffffffffu : S == 2 ? 0x55555555u : S == 4 ? 0x11111111u : S == 8 ? 0x01010101u : 0x00010001u;
    auto go = [&](auto* kernel) { MuseProf prof_("k_chain_grads", st); hipLaunchKernelGGL(kernel, dim3((unsigned)(cq8 * W * S), hn), dim3(256), 0, st, Q, dO, qc, w.s_mu, w.s_k,
                       (const T*)w.s_v, w.perm_q, w.off_q, LSE, w.delta, w.selmask, w.slotinfo, w.chainmask, w.g_s_c,
                       (T*)w.g_s_k, (T*)w.g_s_v, h0, d.N, d.nb, d.Cq, d.Ck, d.r, S, pattern, d.scale); };
    if (d.nb <= 9) go(k_chain_grads_f32<D, 2>);
    else go(k_chain_grads_f32<D, 1>);
  }
  MuseProf prof_("k_chain_odd", st);
  hipLaunchKernelGGL((k_chain_odd<T, D>), dim3(d.Cq, hn), dim3(64 * kOddWaves), 0, st, Q, dO, qc, w.s_mu, w.s_k, (const T*)w.s_v, w.perm_q,
                     w.off_q, LSE, w.delta, w.slotinfo, w.g_s_c, (T*)w.g_s_k, (T*)w.g_s_v, looked, h0, d.N, d.nb, d.Cq, d.Ck, d.r, d.scale);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

}  // namespace

template <typename T>
int muse_launch_chain_grads(const MuseDims& d, const T* Q, const T* dO, const float* qc, const float* LSE, FFWorkspace& w,
                            int h0, int hn, hipStream_t st) {
  return d.D == 64 ? launch<T, 64>(d, Q, dO, qc, LSE, w, h0, hn, st) : launch<T, 128>(d, Q, dO, qc, LSE, w, h0, hn, st);
}
template int muse_launch_chain_grads<float>(const MuseDims&, const float*, const float*, const float*, const float*, FFWorkspace&, int, int, hipStream_t);
template int muse_launch_chain_grads<bf16_t>(const MuseDims&, const bf16_t*, const bf16_t*, const float*, const float*, FFWorkspace&, int, int, hipStream_t);
