// The per-query-tile far-field forward for bf16 inputs: cluster scores (Eq. 7), the r retrieved clusters and the monopole
// attention over all other clusters (component 1) as a partial softmax state.
#include "ff_common.h"
#include "lds_tile.h"

namespace {

// The scores run on the 16-bit matrix cores without losing the precision that decides selections: k-bar is stored as a bf16 plane
// plus an fp16 plane of the remainder (together 19 significant bits or more), the query operand is the bf16 query itself (as fp16 it is
// exact from 2^-17 to 65504; larger entries make infinite scores), and the query centroid's share of q~ . k-bar is a per-cell scalar
// c = scale * qc_i . k-bar, the weighted mean of the tilt logits that the kernel which wrote the planes has at hand:
//   score = scale * q . (hi + mid) + (mu-bar - c).
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;

// top RCAP of two lists sorted from the largest down, into a
template <int RCAP>
__device__ __forceinline__ void merge_lists(float (&a)[RCAP], const float (&b)[RCAP]) {
#pragma unroll
  for (int k = 0; k < RCAP; ++k) a[k] = fmaxf(a[k], b[RCAP - 1 - k]);  // the largest RCAP of both, falling then rising
#pragma unroll
  for (int s = RCAP / 2; s >= 1; s /= 2)
#pragma unroll
    for (int k = 0; k < RCAP; ++k)
      if ((k & s) == 0) {
        const float hi = fmaxf(a[k], a[k + s]), lo = fminf(a[k], a[k + s]);
        a[k] = hi;
        a[k + s] = lo;
      }
}

// LDS of one wave: NB tiles (32 rows of a plane or of the values), at the end its 32 x D sums in their place; the scalars of two
// tiles; its list (kLate: in the place of the second value tile, which is asked for when the lists are read); what it tells the others
template <int D, int RCAP, int NB>
struct WaveLds {
  static constexpr bool kLate = D == 128 && RCAP == 32;
  static constexpr int kTile = 32 * D * 2, kMus = NB * kTile, kEnd = kMus + 2 * 256, kList = kLate ? kTile : kEnd;
  static constexpr int kMax = kLate ? kEnd : kEnd + RCAP * 128, kCnt = kMax + 128, kSum = kCnt + 128, kBytes = kSum + 128;
  static_assert(NB >= 2, "the sums take two tiles");
};
constexpr int kFfWaves = 8;  // most waves of a workgroup

// The end of a phase: LDS is written; what is on its way from memory stays on its way.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void all_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// what is read from LDS is in registers, and its place may be written
__device__ __forceinline__ void lds_read() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// W waves (the workgroup) share a tile of up to 32 queries of one (spatial block b >= 1, query cluster i); wave w takes the
// tiles w, w + W, .. of 32 clusters, TPW at most, and keeps their scores in registers: what decides the selection (both planes
// of k-bar) is read once, the values once, 6 D + 4 bytes per cell.
//   scores     both planes of a tile come straight to LDS, the next tiles (NB = 4) or the next one (NB = 2) on their way while
//              this one is scored; a lane keeps the RCAP largest of its scores sorted
//   selection  the waves exchange their lists, every wave merges all of them, so that it knows the r largest scores of a query:
//              a cluster that reaches the last of them is selected, and its place is the number of larger ones.  Where two
//              scores are equal the places are given out one by one, lowest cluster first.
//   softmax    over the others, against the maximum of all waves, and P V, the first value tiles on their way since the scores
//              were made; the waves' sums meet in LDS.  A weight enters as two bf16 terms (16 bits and more): the largest of
//              those that stay behind a selection would be what bf16 rounds worst.  The second term costs 3 % of the kernel (2608 -> 2689 us
//              at 16 heads of 64k, 0.3 % of the layer; 2473 -> 2545 at 32 of 32k, D = 128), and O is closer to its value in 64 bits
//              (4096 tokens, 16 x 256 clusters, r = 8: 2.07e-3 and 2.01e-3 of the norm).  With few query clusters the
//              summaries come from the L2 and it is 7 % (16 heads of 46k, 9 x 771: 1027 -> 1096).
// Bound by the summaries' way from memory: 12.2 GB fetched and written at 16 heads of 64k with 256 x 1024 clusters, 4.5 TB/s; without the
// selection (insertion and places) it took 2577 us instead of 2614.  With six and eight tiles per wave most forms spill 2 to 7
// vector registers, the one with six tiles and lists of 32 at D = 64 17.  (The times below are with weights of one term.)  The kernel before this one was a wave per tile that read the bf16
// plane of k-bar for a bound of the scores and then everything (8 D + 8 bytes), left tiles with many candidates to a second launch, and
// needed the largest key norm of every head.  us, before (with its second launch) / now: 3270 / 2614 there, 6550 / 4930 at 32
// heads, 585 / 300 with 128 x 128, 139 / 102 at 8 heads of 16k with 64 x 256, 67 / 38 at 12 of 6k with 23 x 71, 4040 / 2745 at 32 of 32k
// with D = 128, 128 x 512 and r = 16, 670 / 312 there with 64 x 64 and r = 4, 215 / 58 at one of 8k with 8 x 2048.
template <int D, int RCAP, int TPW, int NB, int OCC>
__global__ void __launch_bounds__(64 * kFfWaves) __attribute__((amdgpu_waves_per_eu(OCC, OCC))) k_farfield_tiles(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ A_kb, const uint16_t* __restrict__ A_km,
    const float* __restrict__ A_c, const bf16_t* __restrict__ A_v, const int32_t* __restrict__ perm_q,
    const int32_t* __restrict__ off_q, const int32_t* __restrict__ tile_off, float* __restrict__ ff_acc,
    float* __restrict__ ff_ml, int32_t* __restrict__ selc, int h0, int N, int nb, int Cq, int Ck, int r, float scale) {
  constexpr int DT = D / 32, KS = D / 16, CPR = D / 8, NIT = 32 * CPR / 64;
  using L = WaveLds<D, RCAP, NB>;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int W = blockDim.x / 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int hq = h0 + blockIdx.z, b = blockIdx.y + 1, NBm = nb - 1;
  const int lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  unsigned char* my = lds + wave * L::kBytes;
  const uint32_t at = __builtin_amdgcn_readfirstlane(lds_addr(my));

  // Workgroups go to the 8 XCDs round-robin by their linear id and the grid's x extent is a multiple of 8, so
  // x % 8 is the XCD: each XCD takes a contiguous run of the tiles, and the tiles of one (block, query cluster)
  // group, which stream the same cells at about the same time, share its L2.
  const int32_t* to = tile_off + ((size_t)hq * nb + b) * (Cq + 1);
  const int ntl = to[Cq], run = (ntl + 7) / 8;
  const int tile = (blockIdx.x % 8) * run + blockIdx.x / 8;
  if ((int)blockIdx.x / 8 >= run || tile >= ntl) return;
  // the query cluster of the tile: the last with to[i] <= tile, by all lanes in two steps (a bisection is a chain of eight loads)
  const int step = (Cq + 63) / 64;
  const int first = __popcll(__ballot(lane * step < Cq && to[min(lane * step, Cq - 1)] <= tile)) - 1;
  const int i = first * step + __popcll(__ballot(lane < step && first * step + lane < Cq && to[min(first * step + lane, Cq - 1)] <= tile)) - 1;

  const size_t acell = (((size_t)blockIdx.z * NBm + (b - 1)) * Cq + i) * Ck;
  const bf16_t* Ah = A_kb + acell * D;
  const bf16_t* Am = reinterpret_cast<const bf16_t*>(A_km) + acell * D;
  const bf16_t* Av = A_v + acell * D;
  const float* Ac = A_c + acell;
  auto tile_j0 = [&](int t) { return 32 * (wave + W * t); };
  // a number that is made anew where it is used: as an invariant, what is derived from it for every score would be kept in registers
  auto opaque = [](int x) {
    asm volatile("" : "+v"(x));
    return x;
  };
  // 32 rows straight to LDS, which takes 16 bytes per lane in order: the swizzle of tile_at is in the source.  Rows past the
  // last cluster repeat it (what is waited for by count is always asked for).
  auto bring_rows = [&](const bf16_t* plane, int j0, int buf) {
    const int row0 = opaque(lane / CPR);
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int row = it * (64 / CPR) + row0, chunk = (tile_at<D>(row, lane % CPR) - row * D) / 8;
      rows_to_lds(at + buf * L::kTile + 1024 * it, (uint32_t)(min(j0 + row, Ck - 1) * D + chunk * 8) * 2, plane);
    }
  };
  constexpr int kPlanes = 2 * NIT + 1, kValues = NIT;  // loads of a score tile and of a value tile
  auto bring = [&](int t) {  // score tile t of this wave into its pair of buffers
    const int p = NB == 4 ? t % 2 : 0;
    bring_rows(Ah, tile_j0(t), 2 * p);
    bring_rows(Am, tile_j0(t), 2 * p + 1);
    words_to_lds(at + L::kMus + 256 * p, (uint32_t)min(tile_j0(t) + opaque(col), Ck - 1) * 4, Ac);
  };
  auto bring_v = [&](int t) { bring_rows(Av, tile_j0(t), t % NB); };
  bring(0);

  const int32_t* oq = off_q + (size_t)hq * ((size_t)nb * Cq + 1);
  const int qlo = oq[b * Cq + i], qhi = oq[b * Cq + i + 1], tt = tile - to[i];
  int pos = qlo + 32 * tt + col;
  const bool valid = pos < qhi;
  pos = valid ? pos : qlo + 32 * tt;
  const int n = perm_q[(size_t)hq * N + pos];

  f32x16_t S[TPW];
  float m = MUSE_NEG_INF;
  {
    float list[RCAP];  // the largest scores of this lane's clusters, then of the query's
#pragma unroll
    for (int k = 0; k < RCAP; ++k) list[k] = MUSE_NEG_INF;
    {
      bf16x8_t qb[KS];  // the query as the bf16 operand: dims 16 ks + 8 half .. + 7
      const bf16_t* qrow = Q + ((size_t)hq * N + n) * D + 8 * half;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qb[ks] = *reinterpret_cast<const bf16x8_t*>(qrow + 16 * ks);
      if (NB == 4 && TPW > 1) bring(1);
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        // behind tile t are on their way: tile t + 1, or behind the last but one the first two value tiles
        if constexpr (NB == 2) all_but<0>();
        else if (t + 1 < TPW) all_but<kPlanes>();
        else if (TPW > 1) all_but<2 * kValues>();
        else all_but<0>();
        wave_lds_fence();
        const int p = NB == 4 ? t % 2 : 0, j0 = tile_j0(t);
        const bf16_t* th = reinterpret_cast<const bf16_t*>(my + 2 * p * L::kTile);
        const bf16_t* tm = reinterpret_cast<const bf16_t*>(my + (2 * p + 1) * L::kTile);
        const float* mus = reinterpret_cast<const float*>(my + L::kMus + 256 * p);
        f32x16_t acc = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {  // the planes take turns in the sum: its order decides between clusters of nearly equal scores
          uint4 raw = __builtin_bit_cast(uint4, qb[ks]);
          asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w));  // the conversion stays here: the copy's registers would spill
          const bf16x8_t q = __builtin_bit_cast(bf16x8_t, raw);
          f16x8_t qh;
#pragma unroll
          for (int e = 0; e < 8; ++e) qh[e] = (_Float16)(float)q[e];
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(th, col, 2 * ks + half), qb[ks], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, tile_row<D>(tm, col, 2 * ks + half)), qh, acc, 0, 0, 0);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 m4 = *reinterpret_cast<const float4*>(&mus[8 * g + 4 * half]);
          const float c4[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[4 * g + u] = fmaf(scale, acc[4 * g + u], c4[u]);
        }
        lds_read();
        if (NB == 4 ? t + 2 < TPW : t + 1 < TPW) {
          bring(NB == 4 ? t + 2 : t + 1);
        } else {  // the values, two tiles at a time
          const int v0 = NB == 4 && t + 1 == TPW && TPW > 1 ? 2 : 0;
          if (v0 < TPW) bring_v(v0);
          if (v0 + 1 < TPW && !L::kLate) bring_v(v0 + 1);
        }
        if (j0 + 32 > Ck) {
          const int left = opaque(Ck - j0 - 4 * half);
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[e] = 8 * (e / 4) + e % 4 < left ? acc[e] : MUSE_NEG_INF;
        }
        S[t] = acc;
        if (r > 0 && j0 < Ck) {  // insertion into the sorted list: new l_k = med3(x, l_{k-1}, l_k), new l_0 = max(x, l_0)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float x = acc[e];
#pragma unroll
            for (int k = RCAP - 1; k > 0; --k) list[k] = __builtin_amdgcn_fmed3f(x, list[k - 1], list[k]);
            list[0] = fmaxf(list[0], x);
          }
        }
      }
    }
    // the query's r-th largest score; not a number: none is taken out (no score compares with it, one that is infinite neither)
    float thr = __builtin_nanf("");
    if (r > 0) {
      float other[RCAP];
#pragma unroll
      for (int k = 0; k < RCAP; ++k) other[k] = __shfl_xor(list[k], 32, 64);
      merge_lists(list, other);
      if (W > 1) {  // every wave merges all lists: the lower half of a query those of even waves, the upper half the others
        float* mine = reinterpret_cast<float*>(my + L::kList);
        if (half == 0) {
#pragma unroll
          for (int k = 0; k < RCAP; ++k) mine[32 * k + col] = list[k];
        }
        lds_barrier();
        auto fetch = [&](float (&x)[RCAP], int w) {
          const float* in = reinterpret_cast<const float*>(lds + w * L::kBytes + L::kList);
#pragma unroll
          for (int k = 0; k < RCAP; ++k) x[k] = in[32 * k + col];
        };
        fetch(list, half);
        for (int w = 2 + half; w < W; w += 2) {
          fetch(other, w);
          merge_lists(list, other);
        }
#pragma unroll
        for (int k = 0; k < RCAP; ++k) other[k] = __shfl_xor(list[k], 32, 64);
        merge_lists(list, other);
      }
#pragma unroll
      for (int k = 0; k < RCAP; ++k)
        if (k == r - 1) thr = list[k];
      bool tied = false;
#pragma unroll
      for (int k = 1; k < RCAP; ++k) tied |= k < r && list[k] == list[k - 1] && list[k] > MUSE_NEG_INF;
      thr = fmaxf(thr, -3.4028234e38f);  // fewer than r clusters with a finite score: every one of them is selected
      // the place of a selected cluster is the number of larger scores
      int32_t* out = selc + ((size_t)hq * N + n) * r;
      int cnt = 0;
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const int jt = opaque(tile_j0(t) + 4 * half);
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (S[t][e] >= thr) {
            int place = 0;
#pragma unroll
            for (int k = 0; k < RCAP; ++k) place += list[k] > S[t][e];
            if (valid) out[place] = jt + 8 * (e / 4) + e % 4;
            ++cnt;
          }
      }
      cnt += __shfl_xor(cnt, 32, 64);
      if (W > 1) {
        if (half == 0) reinterpret_cast<int*>(my + L::kCnt)[col] = cnt;
        lds_barrier();
        cnt = 0;
        for (int w = 0; w < W; ++w) cnt += reinterpret_cast<const int*>(lds + w * L::kBytes + L::kCnt)[col];
      }
      if (__ballot(tied || cnt > r)) {
        // Two clusters of a query score the same (every wave sees it): the places are given out anew, one by one, the largest
        // score behind the last one's, and of the clusters that have it the one with the lowest number.
        all_but<0>();
        lds_barrier();
        float ps = __builtin_huge_valf();
        int pj = -1;
        for (int place = 0; place < r; ++place) {
          float s = MUSE_NEG_INF;
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
            const int jt = opaque(tile_j0(t) + 4 * half);
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (S[t][e] < ps || (S[t][e] == ps && jt + 8 * (e / 4) + e % 4 > pj)) s = fmaxf(s, S[t][e]);
          }
          s = fmaxf(s, __shfl_xor(s, 32, 64));
          if (half == 0) reinterpret_cast<float*>(my + L::kMax)[col] = s;
          lds_barrier();
          for (int w = 0; w < W; ++w) s = fmaxf(s, reinterpret_cast<const float*>(lds + w * L::kBytes + L::kMax)[col]);
          int j = 0x7fffffff;
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
            const int jt = opaque(tile_j0(t) + 4 * half);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int je = jt + 8 * (e / 4) + e % 4;
              if (S[t][e] == s && (s < ps || je > pj)) j = min(j, je);
            }
          }
          j = min(j, __shfl_xor(j, 32, 64));
          if (half == 0) reinterpret_cast<int*>(my + L::kCnt)[col] = j;
          lds_barrier();
          for (int w = 0; w < W; ++w) j = min(j, reinterpret_cast<const int*>(lds + w * L::kBytes + L::kCnt)[col]);
          if (s == MUSE_NEG_INF) continue;  // no cluster with a finite score is left
          ps = s;
          pj = j;
          if (valid && threadIdx.x < 32) out[place] = j;
        }
        lds_barrier();
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
          const int jt = opaque(tile_j0(t) + 4 * half);
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (S[t][e] > ps || (S[t][e] == ps && jt + 8 * (e / 4) + e % 4 <= pj)) S[t][e] = MUSE_NEG_INF;
        }
        thr = __builtin_nanf("");
      }
    }
    if (L::kLate && TPW > 1) bring_v(1);
    // the selected ones leave the softmax
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        S[t][e] = S[t][e] >= thr ? MUSE_NEG_INF : S[t][e];
        m = fmaxf(m, S[t][e]);
      }
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if (W > 1) {
      if (half == 0) reinterpret_cast<float*>(my + L::kMax)[col] = m;
      lds_barrier();
      for (int w = 0; w < W; ++w) m = fmaxf(m, reinterpret_cast<const float*>(lds + w * L::kBytes + L::kMax)[col]);
    }
  }

  // ---- the softmax over the others, P V: every wave against the same maximum ----
  const float mref = m == MUSE_NEG_INF ? 0.f : m;
  float l = 0.f;
  f32x16_t o[DT];
#pragma unroll
  for (int x = 0; x < DT; ++x) o[x] = zero16();
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      S[t][e] = __expf(S[t][e] - mref);
      l += S[t][e];
    }
    constexpr int kAhead = NB < TPW ? NB : TPW;
    if (t + kAhead <= TPW) all_but<(kAhead - 1) * kValues>();
    else if (t + 2 == TPW) all_but<kValues>();
    else if (t + 3 == TPW) all_but<2 * kValues>();
    else all_but<0>();
    wave_lds_fence();
    const bf16_t* vt = reinterpret_cast<const bf16_t*>(my + t % NB * L::kTile);
#pragma unroll
    for (int G = 0; G < 2; ++G) {
      const bf16x8_t pf = pack8(S[t], 2 * G, 2 * G + 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) S[t][8 * G + e] -= (float)pf[e];  // what the rounding left
      const bf16x8_t pr = pack8(S[t], 2 * G, 2 * G + 1);
#pragma unroll
      for (int x = 0; x < DT; ++x) {
        const bf16x8_t v = tile_cols<D>(vt, 16 * G, x, lane);
        o[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pf, o[x], 0, 0, 0);
        o[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pr, o[x], 0, 0, 0);
      }
    }
    if (t + NB < TPW) {
      lds_read();
      bring_v(t + NB);
    }
  }
  l += __shfl_xor(l, 32, 64);
  float* sums = reinterpret_cast<float*>(my);  // [query][16-byte chunk, by an xor of query bits]
  constexpr int CPQ = D / 4;
  wave_lds_fence();
#pragma unroll
  for (int x = 0; x < DT; ++x)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(sums + col * D + (((8 * x + 2 * g + half) ^ (col % CPQ)) << 2)) =
          make_float4(o[x][4 * g], o[x][4 * g + 1], o[x][4 * g + 2], o[x][4 * g + 3]);
  if (half == 0) {
    reinterpret_cast<float*>(my + L::kSum)[col] = l;
    reinterpret_cast<int*>(my + L::kCnt)[col] = valid ? n : -1;
  }
  lds_barrier();
  for (int u = threadIdx.x; u < 32 * CPQ; u += 64 * W) {
    const int q = u / CPQ, c = u % CPQ, nq = reinterpret_cast<const int*>(lds + L::kCnt)[q];
    if (nq < 0) continue;
    const float* in = reinterpret_cast<const float*>(lds) + q * D + ((c ^ (q % CPQ)) << 2);
    float4 a = *reinterpret_cast<const float4*>(in);
    for (int w = 1; w < W; ++w) {
      const float4 z = *reinterpret_cast<const float4*>(in + w * (L::kBytes / 4));
      a.x += z.x; a.y += z.y; a.z += z.z; a.w += z.w;
    }
    *reinterpret_cast<float4*>(ff_acc + ((size_t)hq * N + nq) * D + 4 * c) = a;
  }
  if (threadIdx.x < 32 && valid) {
    float sum = 0.f;
    for (int w = 0; w < W; ++w) sum += reinterpret_cast<const float*>(lds + w * L::kBytes + L::kSum)[col];
    *reinterpret_cast<float2*>(ff_ml + ((size_t)hq * N + n) * 2) = make_float2(m, sum);
  }
}

template <int D, int RCAP, int TPW, int NB, int OCC>
int launch(const MuseDims& d, const void* Q, const FFWorkspace& w, int32_t* selc, int h0, int hn, hipStream_t st) {
  constexpr int kBytes = WaveLds<D, RCAP, NB>::kBytes;
  const int W = ((d.Ck + 31) / 32 + TPW - 1) / TPW;
  auto* kernel = k_farfield_tiles<D, RCAP, TPW, NB, OCC>;
  static_assert(kBytes * kFfWaves <= 160 * 1024, "a workgroup's LDS");
  static bool attr_set = false;
  if (!attr_set) {
    MUSE_HIP_CHECK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kFfWaves * kBytes));
    attr_set = true;
  }
  {
    MuseProf prof_("k_farfield_fwd", st);
    hipLaunchKernelGGL(kernel, dim3((unsigned)ff_tile_grid_x(d), d.nb - 1, hn), dim3(64 * W), W * kBytes, st, (const bf16_t*)Q,
                       (const bf16_t*)w.A_kb, (const uint16_t*)w.A_km, w.A_c, (const bf16_t*)w.A_v, w.perm_q, w.off_q, w.tile_off, w.ff_acc, w.ff_ml,
                       selc, h0, d.N, d.nb, d.Cq, d.Ck, d.r, d.scale);
  }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

// Tiles of clusters per wave.  The waves of a workgroup pass three barriers, so few waves with many tiles each waste the least,
// up to four of them (one for each SIMD; eight only where eight tiles do not reach).  At D = 64 a small problem (less than 8192
// waves, 8 per SIMD) takes fewer tiles per wave.  us with 1, 2, 4, 6 and 8 tiles per wave (D = 64; heads, tokens, query x key clusters, r):
//   16, 32k, 64 x 128, 8   201, 171, 179, 219, 284      4, 16k, 32 x 128, 8     40, 47, 67, 90, 102
//   16, 32k, 64 x 256, 8   408, 294, 281, 361, 332      4, 16k, 32 x 256, 8     71, 64, 79, 105, 122
//   16, 32k, 64 x 512, 9     -   -   604, 645, 676      4, 16k, 32 x 512, 8    120, 83, 79, 103, 124
//   16, 32k, 64 x 768, 8     -   -  1175, 664, 882      1, 16k, 32 x 256, 8     27, 22, 24, 29, 30
//   16, 64k, 256 x 1024, 8   -   -  3086, 3728, 2614    1, 16k, 32 x 1024, 8     -   -  55, 69, 53
// D = 128:
//   32, 32k, 64 x 64, 4    400, 312, 383, 462, 570      16, 32k, 64 x 384, 8   722, 1100, 742, 627, 724
//   16, 32k, 64 x 128, 8   386, 279, 268, 313, 376      32, 32k, 128 x 512, 16   -  3854, 2782, 3193, 2745
//   16, 32k, 64 x 256, 8   887, 536, 438, 523, 473      8, 32k, 64 x 1024, 8     -   -   943, 1094, 812
int tiles_per_wave(const MuseDims& d) {
  const int ntile = (d.Ck + 31) / 32;
  if (d.D == 128) return ntile <= 2 ? ntile : ntile <= 8 ? 4 : ntile <= 12 ? 6 : 8;
  const long long tiles = (long long)d.B * d.Hq * (d.nb - 1) * (d.Bs / 32 + d.Cq / 2);
  int t = ntile <= 4 ? 1 : ntile <= 8 ? 2 : ntile <= 16 ? 4 : ntile <= 24 ? 6 : 8;
  while (t < 4 && t < ntile && tiles * ((ntile + 2 * t - 1) / (2 * t)) >= 8192) t *= 2;
  return t;
}

template <int D, int RCAP>
int launch_tpw(const MuseDims& d, const void* Q, const FFWorkspace& w, int32_t* selc, int h0, int hn, hipStream_t st) {
  switch (tiles_per_wave(d)) {
    case 1: return launch<D, RCAP, 1, 2, D == 64 ? 4 : 2>(d, Q, w, selc, h0, hn, st);
    case 2: return launch<D, RCAP, 2, 2, D == 64 ? 4 : 2>(d, Q, w, selc, h0, hn, st);
    case 4: return launch<D, RCAP, 4, 2, D == 64 ? 3 : 2>(d, Q, w, selc, h0, hn, st);
    case 6: return launch<D, RCAP, 6, 2, D == 64 ? 3 : 2>(d, Q, w, selc, h0, hn, st);
    default: return launch<D, RCAP, 8, D == 64 && RCAP < 32 ? 4 : 2, 2>(d, Q, w, selc, h0, hn, st);
  }
}

}  // namespace

int muse_launch_farfield_tiles(const MuseDims& d, const void* Q, const FFWorkspace& w, int32_t* selc, int h0, int hn, hipStream_t st) {
  static_assert(MUSE_MAX_CLUSTERS <= 32 * 8 * kFfWaves, "eight tiles per wave reach the largest accepted Ck");
  if (d.D == 64) return d.r <= 8 ? launch_tpw<64, 8>(d, Q, w, selc, h0, hn, st) : d.r <= 16 ? launch_tpw<64, 16>(d, Q, w, selc, h0, hn, st) : launch_tpw<64, 32>(d, Q, w, selc, h0, hn, st);
  return d.r <= 8 ? launch_tpw<128, 8>(d, Q, w, selc, h0, hn, st) : d.r <= 16 ? launch_tpw<128, 16>(d, Q, w, selc, h0, hn, st) : launch_tpw<128, 32>(d, Q, w, selc, h0, hn, st);
}
