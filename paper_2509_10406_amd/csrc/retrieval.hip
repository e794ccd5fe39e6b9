// Exact retrieval (Sec. 3.3): the inverse index "retrieved (key cluster, key block) pair -> queries" and
// the merge of the per-pair forward partial states into the far-field state of every query.
//
//   hits[hk][pair_off[hk][b'*Ck + j] ...]  the queries of all heads of the KV group that retrieved the
//                                           pair, ascending (head, position): x = n | g << 22, y = slot*k2e + u
// Ordered lists (ballot ranks, no atomics on the order) keep every later sum reproducible.
#include "ff_common.h"

namespace {

// The hit lists are built by a counting sort whose order is fixed by construction.  The queries with a far field
// (positions Bs .. N-1) of every query head are cut into SEG slices of whole 64-query chunks, with one counter per pair in LDS.
// Pass 1 (k_hit_counts) leaves the counts per (kv head, head of the group x slice, pair); k_pair_totals,
// k_pair_scan and k_seg_offsets turn them into list starts (pair-major, then head of the group, then slice);
// pass 2 (k_hit_lists) starts from those and writes the hits, with the slot index the pair has in the query's
// exported selections: one wave walks a slice's chunks, and for a selection slot of a chunk the lanes that name the same pair are
// found by ballots over the bits of its number and ranked by lane, so a list is ascending in (head of the group, chunk, slot,
// position) without any atomic deciding an order.
// us of the two passes, with eight waves per slice that shared the pairs and went through the distinct ones of a chunk one by
// one, in both passes / now: 222 + 327 / 36 + 129 at 16 heads of 64k with 256 x 1024 clusters, 245 + 298 / 29 + 75 with 128 x 128, 440 +
// 667 / 67 + 201 at 32 heads of 32k with 128 x 512 and r = 16, 17 + 28 / 7 + 12 at 12 heads of 6k.  With the most pairs there can be (15 blocks
// x 2048 clusters, 120 KB of counters: one wave of the second pass on a CU), the two together: 55 / 51 at one head of 8k, 192 / 189 at one
// of 64k, 647 / 519 at 16 heads of 16k, 2929 / 1235 there with r = 32 and k2 = 2, 1704 / 846 at 16 heads of 64k.
constexpr int kHitWaves = 8;   // of the workgroup that counts
constexpr int kHitSlots = 8;   // selection slots requested together

struct HitSlice {
  int hq, hk, g, c0, c1;  // query head, its kv head and number in the group; chunks
  size_t sbase;           // the slice's counters
};
__device__ __forceinline__ HitSlice hit_slice(int N, int Bs, int Hq, int Hkv, int npair, int SEG, int cps) {
  HitSlice x;
  const int G_ = Hq / Hkv, s = blockIdx.x, chunks = (N - Bs + 63) / 64;
  x.hq = blockIdx.y;
  x.g = (x.hq % Hq) % G_;
  x.hk = (x.hq / Hq) * Hkv + (x.hq % Hq) / G_;
  x.c0 = s * cps;
  x.c1 = min((s + 1) * cps, chunks);
  x.sbase = ((size_t)x.hk * G_ * SEG + (size_t)x.g * SEG + s) * npair;
  return x;
}
// the pairs of slots s0 .. of a chunk's queries (slot s: retrieved cluster s / k2e, its block s % k2e), -1 where there is none
// (selections are trusted inputs; one outside the table is dropped rather than indexed)
__device__ __forceinline__ void load_pairs(int (&pair)[kHitSlots], const int32_t* __restrict__ selc, const int32_t* __restrict__ selb,
                                           size_t qn, bool valid, int s0, int r, int k2e, int Ck, int npair) {
  const int R2 = r * k2e;
  int j[kHitSlots], bp[kHitSlots];
#pragma unroll
  for (int u = 0; u < kHitSlots; ++u) {
    const int s = min(s0 + u, R2 - 1);
    j[u] = selc[qn * r + s / k2e];
    bp[u] = selb[qn * R2 + s];
  }
#pragma unroll
  for (int u = 0; u < kHitSlots; ++u) {
    const int p = bp[u] * Ck + j[u];
    pair[u] = valid && s0 + u < R2 && j[u] >= 0 && j[u] < Ck && bp[u] >= 0 && bp[u] < 16 && p < npair ? p : -1;
  }
}

__global__ void __launch_bounds__(64 * kHitWaves) k_hit_counts(const int32_t* __restrict__ selc, const int32_t* __restrict__ selb,
                                                               int32_t* __restrict__ seg_cnt, int N, int Bs, int Ck, int r, int k2e,
                                                               int Hq, int Hkv, int npair, int SEG, int cps) {
  extern __shared__ int cur[];
  const HitSlice sl = hit_slice(N, Bs, Hq, Hkv, npair, SEG, cps);
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  for (int p = threadIdx.x; p < npair; p += 64 * kHitWaves) cur[p] = 0;
  __syncthreads();
  for (int c = sl.c0 + wave; c < sl.c1; c += kHitWaves) {
    const int n = Bs + 64 * c + lane;
    const size_t qn = (size_t)sl.hq * N + min(n, N - 1);
    for (int s0 = 0; s0 < r * k2e; s0 += kHitSlots) {
      int pair[kHitSlots];
      load_pairs(pair, selc, selb, qn, n < N, s0, r, k2e, Ck, npair);
#pragma unroll
      for (int u = 0; u < kHitSlots; ++u)
        if (pair[u] >= 0) atomicAdd(&cur[pair[u]], 1);
    }
  }
  __syncthreads();
  for (int p = threadIdx.x; p < npair; p += 64 * kHitWaves) seg_cnt[sl.sbase + p] = cur[p];
}

__global__ void __launch_bounds__(64) k_hit_lists(const int32_t* __restrict__ selc, const int32_t* __restrict__ selb,
                                                  const int32_t* __restrict__ seg_off, uint2* __restrict__ hits, size_t hit_cap, int N,
                                                  int Bs, int Ck, int r, int k2e, int Hq, int Hkv, int npair, int SEG, int cps) {
  extern __shared__ int cur[];  // per pair: next list position
  const HitSlice sl = hit_slice(N, Bs, Hq, Hkv, npair, SEG, cps);
  const int lane = threadIdx.x, bits = 32 - __clz(npair - 1 > 0 ? npair - 1 : 1);
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int p0 = 0; p0 < npair; p0 += 64 * 8) {
    int v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = seg_off[sl.sbase + min(p0 + 64 * u + lane, npair - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p0 + 64 * u + lane < npair) cur[p0 + 64 * u + lane] = v[u];
  }
  wave_lds_fence();
  uint2* out = hits + (size_t)sl.hk * hit_cap;
  const int R2 = r * k2e, per = (R2 + kHitSlots - 1) / kHitSlots, total = (sl.c1 - sl.c0) * per;
  int next[kHitSlots];
  auto load = [&](int x) {  // the x-th group of slots of the slice
    const int n = Bs + 64 * (sl.c0 + x / per) + lane;
    load_pairs(next, selc, selb, (size_t)sl.hq * N + min(n, N - 1), n < N, x % per * kHitSlots, r, k2e, Ck, npair);
  };
  if (total > 0) load(0);
  for (int x = 0; x < total; ++x) {
    int pair[kHitSlots];
#pragma unroll
    for (int u = 0; u < kHitSlots; ++u) pair[u] = next[u];
    if (x + 1 < total) load(x + 1);
    const int n = Bs + 64 * (sl.c0 + x / per) + lane, s0 = x % per * kHitSlots;
#pragma unroll
    for (int u = 0; u < kHitSlots; ++u) {
      const bool hit = pair[u] >= 0;
      unsigned long long same = __ballot(hit);
      if (same == 0ull) continue;
      for (int bit = 0; bit < bits; ++bit) {
        const bool one = (pair[u] >> bit) & 1;
        const unsigned long long ones = __ballot(one);
        same &= one ? ones : ~ones;
      }
      if (hit) {
        const int base = cur[pair[u]], rank = __popcll(same & below), count = __popcll(same);
        out[base + rank] = make_uint2((uint32_t)n | ((uint32_t)sl.g << 22), (uint32_t)(s0 + u));
        if (rank == count - 1) cur[pair[u]] = base + count;
      }
      wave_lds_fence();
    }
  }
}

// The two passes over the segment counters: 64 pairs (lanes) per workgroup, its 16 waves share the segments.  (A thread
// per pair walked all segments, up to 2048 of them, one after the other: 0.38 + 0.22 ms at 4 heads of 29k tokens, D = 128,
// one KV head; 0.03 ms each now.)
constexpr int kSegWaves = 16;
// pair_cnt[hk][p] = hits of pair p over all (head of the group, slice) segments
__global__ void __launch_bounds__(64 * kSegWaves) k_pair_totals(const int32_t* __restrict__ seg_cnt, int32_t* __restrict__ pair_cnt,
                                                                 int npair, int SEGT) {
  __shared__ int part[kSegWaves][64];
  const int hk = blockIdx.y, lane = threadIdx.x % 64, wave = threadIdx.x / 64, p = blockIdx.x * 64 + lane;
  const int per = (SEGT + kSegWaves - 1) / kSegWaves, g0 = wave * per, g1 = g0 + per < SEGT ? g0 + per : SEGT;
  const int32_t* c = seg_cnt + (size_t)hk * SEGT * npair + (p < npair ? p : npair - 1);
  int tot = 0;
#pragma unroll 8
  for (int gs = g0; gs < g1; ++gs) tot += c[(size_t)gs * npair];
  part[wave][lane] = tot;
  __syncthreads();
  if (wave == 0 && p < npair) {
    for (int w = 1; w < kSegWaves; ++w) tot += part[w][lane];
    pair_cnt[(size_t)hk * (npair + 1) + p] = tot;
  }
}

// seg_off[hk][gs][p] = pair_off[hk][p] + hits of pair p in the segments before gs
__global__ void __launch_bounds__(64 * kSegWaves) k_seg_offsets(const int32_t* __restrict__ seg_cnt, const int32_t* __restrict__ pair_off,
                                                                 int32_t* __restrict__ seg_off, int npair, int SEGT) {
  __shared__ int part[kSegWaves][64];
  const int hk = blockIdx.y, lane = threadIdx.x % 64, wave = threadIdx.x / 64, p = blockIdx.x * 64 + lane;
  const int per = (SEGT + kSegWaves - 1) / kSegWaves, g0 = wave * per, g1 = g0 + per < SEGT ? g0 + per : SEGT;
  const size_t base = (size_t)hk * SEGT * npair + (p < npair ? p : npair - 1);
  int tot = 0;
#pragma unroll 8
  for (int gs = g0; gs < g1; ++gs) tot += seg_cnt[base + (size_t)gs * npair];
  part[wave][lane] = tot;
  __syncthreads();
  if (p >= npair) return;
  int run = pair_off[(size_t)hk * (npair + 1) + p];
  for (int w = 0; w < wave; ++w) run += part[w][lane];
#pragma unroll 8
  for (int gs = g0; gs < g1; ++gs) {
    seg_off[base + (size_t)gs * npair] = run;
    run += seg_cnt[base + (size_t)gs * npair];
  }
}

// Work items of the per-pair retrieval kernels: a pair's hit tiles (32 hits each) are cut into runs of kRunTiles, so
// a heavy pair becomes many equal items and a light one a single item (no empty slices, no tails).
//   run_map[hk][run_off[hk][p] + u] = (p, first hit of run u, end of the run)
// The items of the key/value gradient kernel are (pair, hit slice), c3_slices of them per pair that has hits.
__host__ __device__ inline int pair_runs(int hits) { return ((hits + 31) / 32 + kRunTiles - 1) / kRunTiles; }
__host__ __device__ inline int pair_slices(int hits, C3Cut cut) { return hits > 0 ? c3_slices(hits, cut) : 0; }
__global__ void __launch_bounds__(256) k_pair_items(const int32_t* __restrict__ pair_off, const int32_t* __restrict__ run_off,
                                                     const int32_t* __restrict__ c3_off, int4* __restrict__ run_map,
                                                     int2* __restrict__ c3_map, int npair, size_t run_cap, C3Cut cut) {
  const int hk = blockIdx.y, p = blockIdx.x * 256 + threadIdx.x;
  if (p >= npair) return;
  const size_t at = (size_t)hk * (npair + 1) + p;
  const int lo = pair_off[at], hi = pair_off[at + 1];
  if (run_map) {
    int4* run = run_map + (size_t)hk * run_cap + run_off[at];
    for (int u = 0, h = lo; h < hi; ++u, h += 32 * kRunTiles)
      run[u] = make_int4(p, h, h + 32 * kRunTiles < hi ? h + 32 * kRunTiles : hi, 0);
  }
  int2* sl = c3_map + (size_t)hk * run_cap + c3_off[at];
  for (int u = 0; u < pair_slices(hi - lo, cut); ++u) sl[u] = make_int2(p, u);
}

// exclusive prefixes, per kv head, of the pairs' hits, runs and slices (entry n: the totals)
__global__ void __launch_bounds__(1024) k_pair_scan(const int32_t* __restrict__ cnt, int32_t* __restrict__ pair_off,
                                                     int32_t* __restrict__ run_off, int32_t* __restrict__ c3_off, int n, C3Cut cut) {
  __shared__ int wsum[3][16];
  const int hk = blockIdx.x, lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  const size_t base = (size_t)hk * (n + 1);
  const int per = (n + 1023) / 1024;
  int mine[3] = {0, 0, 0};
  for (int u = 0; u < per; ++u) {
    const int i = threadIdx.x * per + u;
    const int c = i < n ? cnt[base + i] : 0;
    mine[0] += c; mine[1] += pair_runs(c); mine[2] += pair_slices(c, cut);
  }
  int run[3];
#pragma unroll
  for (int z = 0; z < 3; ++z) {
    int incl = mine[z];
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(incl, d, 64);
      if (lane >= d) incl += v;
    }
    if (lane == 63) wsum[z][wave] = incl;
    run[z] = incl - mine[z];
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 3; ++z)
    for (int w = 0; w < wave; ++w) run[z] += wsum[z][w];
  for (int u = 0; u < per; ++u) {
    const int i = threadIdx.x * per + u;
    if (i >= n) break;
    const int c = cnt[base + i];
    pair_off[base + i] = run[0]; run_off[base + i] = run[1]; c3_off[base + i] = run[2];
    run[0] += c; run[1] += pair_runs(c); run[2] += pair_slices(c, cut);
  }
  if (threadIdx.x == 1023) { pair_off[base + n] = run[0]; run_off[base + n] = run[1]; c3_off[base + n] = run[2]; }
}

// far-field state of every query  <-  state (+) partial states of its retrieved pairs.
// D/4 lanes per query, each owning 4 dims; part rows are [D], and (max, sum) of all rows follow them.
__global__ void __launch_bounds__(256) k_merge_ret(const int32_t* __restrict__ selb, const float* __restrict__ part,
                                                    const float* __restrict__ part_ml, float* __restrict__ ff_acc, float* __restrict__ ff_ml, size_t nq,
                                                    int N, int Bs, int D, int R2) {
  const int LPQ = D / 4;
  size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  size_t q = t / LPQ;
  const int c = (int)(t % LPQ);
  if (q >= nq) return;
  if ((int)(q % N) < Bs) return;  // first block: no far field
  float m = ff_ml[q * 2], l = ff_ml[q * 2 + 1];
  float4 a = *reinterpret_cast<float4*>(ff_acc + q * D + 4 * c);
  if (!(l > 0.f)) { m = MUSE_NEG_INF; l = 0.f; a = make_float4(0.f, 0.f, 0.f, 0.f); }
  auto fold = [&](float pm, float pl, const float4 pa) {
    const float mn = fmaxf(m, pm);
    const float ca = __expf(m - mn), cb = __expf(pm - mn);
    l = l * ca + pl * cb;
    a.x = a.x * ca + pa.x * cb; a.y = a.y * ca + pa.y * cb;
    a.z = a.z * ca + pa.z * cb; a.w = a.w * ca + pa.w * cb;
    m = mn;
  };
  for (int s0 = 0; s0 < R2; s0 += 8) {
    // eight of the query's partial states are requested together and folded in slot order
    float2 ml[8];
    float4 pa[8];
#pragma unroll
    for (int su = 0; su < 8; ++su) {
      const size_t at = q * R2 + (s0 + su < R2 ? s0 + su : 0);
      const bool ok = s0 + su < R2 && selb[at] >= 0;
      ml[su] = ok ? *reinterpret_cast<const float2*>(part_ml + 2 * at) : make_float2(0.f, 0.f);
      pa[su] = ok ? *reinterpret_cast<const float4*>(part + at * D + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int su = 0; su < 8; ++su)
      if (ml[su].y > 0.f) fold(ml[su].x, ml[su].y, pa[su]);
  }
  *reinterpret_cast<float4*>(ff_acc + q * D + 4 * c) = a;
  if (c == 0) { ff_ml[q * 2] = m; ff_ml[q * 2 + 1] = l; }
}

}  // namespace

int muse_ff_build_inverse_index(const MuseDims& d, const int32_t* selc, const int32_t* selb, FFWorkspace& w, hipStream_t st) {
  const int HQ = d.B * d.Hq, HK = d.B * d.Hkv, N = d.N, NBm = d.nb - 1;
  const int SEG = ff_hit_segments(d), SEGT = (d.Hq / d.Hkv) * SEG, npair = NBm * d.Ck;
  const int chunks = (N - d.Bs + 63) / 64, cps = (chunks + SEG - 1) / SEG;
  const size_t lds = (size_t)npair * sizeof(int);
  static_assert((size_t)15 * MUSE_MAX_CLUSTERS * sizeof(int) <= 128 * 1024, "the pair counters of the largest accepted shape fit the LDS");
  static bool attr_set = false;
  if (!attr_set) {
    MUSE_HIP_CHECK(hipFuncSetAttribute((const void*)k_hit_counts, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    MUSE_HIP_CHECK(hipFuncSetAttribute((const void*)k_hit_lists, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    attr_set = true;
  }
  const dim3 g(SEG, HQ), gs((npair + 63) / 64, HK);
  { MuseProf prof_("k_hit_counts", st); hipLaunchKernelGGL(k_hit_counts, g, dim3(64 * kHitWaves), lds, st, selc, selb, w.seg_cnt, N, d.Bs, d.Ck, d.r, d.k2e, d.Hq, d.Hkv, npair, SEG, cps); }
  { MuseProf prof_("k_pair_totals", st); hipLaunchKernelGGL(k_pair_totals, gs, dim3(64 * kSegWaves), 0, st, w.seg_cnt, w.pair_cnt, npair, SEGT); }
  { MuseProf prof_("k_pair_scan", st); hipLaunchKernelGGL(k_pair_scan, dim3(HK), dim3(1024), 0, st, w.pair_cnt, w.pair_off, w.run_off, w.c3_off, npair, ff_c3_cut(d)); }
  { MuseProf prof_("k_seg_offsets", st); hipLaunchKernelGGL(k_seg_offsets, gs, dim3(64 * kSegWaves), 0, st, w.seg_cnt, w.pair_off, w.seg_off, npair, SEGT); }
  { MuseProf prof_("k_hit_lists", st); hipLaunchKernelGGL(k_hit_lists, g, dim3(64), lds, st, selc, selb, w.seg_off, w.hits, w.hit_cap, N, d.Bs, d.Ck, d.r, d.k2e, d.Hq, d.Hkv, npair, SEG, cps); }
  { MuseProf prof_("k_pair_items", st); hipLaunchKernelGGL(k_pair_items, dim3((npair + 255) / 256, HK), dim3(256), 0, st, w.pair_off, w.run_off, w.c3_off, w.run_map, w.c3_map, npair, w.run_cap, ff_c3_cut(d)); }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_merge_ret(const MuseDims& d, const int32_t* selb, const float* part, float* ff_acc, float* ff_ml,
                          hipStream_t st) {
  const size_t nq = (size_t)d.B * d.Hq * d.N;
  const size_t threads = nq * (d.D / 4);
  { MuseProf prof_("k_merge_ret", st); hipLaunchKernelGGL(k_merge_ret, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, selb, part, part + nq * d.r * d.k2e * d.D, ff_acc, ff_ml, nq, d.N, d.Bs, d.D, d.r * d.k2e); }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
