// Far-field stages (Sec. 3.1-3.3): workspace layout and fp32-MFMA helpers shared by the forward and
// backward translation units.
//
// fp32 MFMA (v_mfma_f32_32x32x2_f32) conventions used throughout:
//   - accumulator element e = 4g+t of lane l is row 8g + 4(l/32) + t, column l%32;
//   - an operand lane supplies one value per instruction: its k-slot is l/32.
//   "Row pattern": operand X[row = l%32][c], contraction over the contiguous index c.  A lane loads
//   float4 groups X[row][8u + 4(l/32) .. +3]; instruction (u,t) uses element t, i.e. half h
//   contributes c = 8u + 4h + t.  Two row-pattern operands pair up consistently.
//   "Column pattern": A[m][k] = X[k][m] read as X[k0 + 8g + 4(l/32) + t][m0 + l%32] (coalesced over
//   lanes), pairing with a B operand taken straight from an accumulator (its rows are 8g+4h+t).
#pragma once
#include <utility>

#include "common.h"

__device__ __forceinline__ f32x16_t mfma32(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}

// acc += X[row][.] (row pattern, `row` already offset by 4*(l/32)) times the row-pattern operand b
template <int D>
__device__ __forceinline__ f32x16_t mfma_rows(f32x16_t acc, const float* __restrict__ row, const float (&b)[D / 8][4]) {
#pragma unroll
  for (int u = 0; u < D / 8; ++u) {
    float4 a = *reinterpret_cast<const float4*>(row + 8 * u);
    acc = mfma32(a.x, b[u][0], acc);
    acc = mfma32(a.y, b[u][1], acc);
    acc = mfma32(a.z, b[u][2], acc);
    acc = mfma32(a.w, b[u][3], acc);
  }
  return acc;
}

// One tile of 32 accumulated key summaries as the score MFMAs consume it: the lane's row-pattern groups
// of k-bar and its 16 mu-bar values.  Loading is separate from use so that every load of a tile is in
// flight before the first MFMA waits on one.
template <int D>
struct KTile {
  float4 a[D / 8];
  float mu[16];
};

template <int D>
__device__ __forceinline__ void load_ktile(KTile<D>& kt, const float* __restrict__ Amu, const float* __restrict__ Ak,
                                           int j0, int Ck, int col, int half) {
  int c = j0 + col;
  c = c < Ck ? c : Ck - 1;
  const float* row = Ak + (size_t)c * D + 4 * half;
#pragma unroll
  for (int u = 0; u < D / 8; ++u) kt.a[u] = *reinterpret_cast<const float4*>(row + 8 * u);
  if ((Ck & 3) == 0) {  // rows 8g + 4 half + t, t = 0..3, are one aligned float4
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      int base = j0 + 8 * g + 4 * half;
      base = base < Ck ? base : Ck - 4;
      const float4 m4 = *reinterpret_cast<const float4*>(Amu + base);
      kt.mu[4 * g] = m4.x; kt.mu[4 * g + 1] = m4.y; kt.mu[4 * g + 2] = m4.z; kt.mu[4 * g + 3] = m4.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      int jr = j0 + 8 * (e / 4) + 4 * half + (e % 4);
      kt.mu[e] = Amu[jr < Ck ? jr : Ck - 1];
    }
  }
}

// scores^T of 32 key clusters (rows) x 32 queries (columns) against accumulated summaries, Eq. 7:
// accumulator preloaded with mu-bar, then += k-bar . q~
template <int D>
__device__ __forceinline__ f32x16_t score_ktile(const KTile<D>& kt, int j0, int Ck, const float (&qt)[D / 8][4], int half) {
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int jr = j0 + 8 * (e / 4) + 4 * half + (e % 4);
    acc[e] = jr < Ck ? kt.mu[e] : MUSE_NEG_INF;
  }
#pragma unroll
  for (int u = 0; u < D / 8; ++u) {
    acc = mfma32(kt.a[u].x, qt[u][0], acc);
    acc = mfma32(kt.a[u].y, qt[u][1], acc);
    acc = mfma32(kt.a[u].z, qt[u][2], acc);
    acc = mfma32(kt.a[u].w, qt[u][3], acc);
  }
  return acc;
}

template <int D>
__device__ __forceinline__ f32x16_t score_tile(const float* __restrict__ Amu, const float* __restrict__ Ak, int j0,
                                               int Ck, const float (&qt)[D / 8][4], int col, int half) {
  KTile<D> kt;
  load_ktile<D>(kt, Amu, Ak, j0, Ck, col, half);
  return score_ktile<D>(kt, j0, Ck, qt, half);
}

// bf16 MFMA (v_mfma_f32_32x32x16_bf16) helpers.  pack8: accumulator rows 4*g0..+3 and 4*g1..+3 of a lane
// become the 8 k-slots of a B (or A) operand; the matching other operand must use the same row order.
__device__ __forceinline__ bf16x8_t pack8(const f32x16_t& s, int g0, int g1) {
  bf16x8_t r;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    r[t] = (__bf16)s[4 * g0 + t];
    r[4 + t] = (__bf16)s[4 * g1 + t];
  }
  return r;
}

// The queries of the kernels that read the retrieved chains' summaries per query (k_comp2_fwd, k_comp2_bwd_dq), 16 lanes per query:
// this group's place in the bucketed order (block by block, cluster by cluster), negative: none.  Workgroups go to the 8 XCDs
// round-robin.  A block's queries are cut into runs of up to 16 workgroups, eight or a multiple of eight of them; an XCD takes
// a run of the last block, the same one of the block before, and so on, then its next run.  So the queries that it has at one
// time are of a few clusters, whatever their block, and read the same rows, and the last blocks, whose queries have the most work, go
// first.  (Clusters lie at about the same share of every block; nothing but speed depends on it.)  Which XCD has the first run
// changes with the head, or the runs left over at the end would all be the first XCDs'.
// us of k_comp2_fwd / k_comp2_bwd_dq with other orders: block by block in runs of 32, which leaves the last XCDs idle at every head's end / the same
// with that turn, from the last block / exactly cluster by cluster, an eighth per XCD, for which a place takes two more round trips / now:
//   32 heads of 64k, rotary rows, 256 x 1024      3125 / 3108, 3113 / 3085, 2890 / 3024, 2779 / 2945
//   32 heads of 32k, D = 128, 128 x 512, r = 16   3760 / 4113, 3606 / 4081, 3507 / 4044, 3371 / 3973
//   16 heads of 64k, 256 x 1024; 128 x 128        1156 / 1164, 1094 / 1149, 1125 / 1187, 1040 / 1115; 907 / 1006, 862 / 996, 921 / 1032, 825 / 977
//   8 heads of 16k; 12 of 6k; 4 fp32 of 8k        87 / 91, 77 / 80, 88 / 89, 75 / 79; 71 / 97, 50 / 75, 55 / 77, 49 / 71; 149 / 146, 132 / 128, 130 / 127, 121 / 118
// Runs of 32 in the first three: 2900 / 3018, 3612 / 4092, 1071 / 1143; of 8: 2843 / 2951, 3509 / 3955, 1084 / 1126 (of 16 on that box 2820 /
// 2952, 3435 / 3998, 1054 / 1122).
static inline __host__ __device__ int far_run(int Bs) {  // workgroups of a run: at most 16, as many runs for every XCD
  const int wgs = (Bs + 15) / 16, turns = (wgs + 127) / 128;
  return (wgs + 8 * turns - 1) / (8 * turns);
}
__device__ __forceinline__ int far_position(int Bs, int nb) {
  const int run = far_run(Bs), g = blockIdx.x / 8 / run, k = g / (nb - 1) * 8 + (blockIdx.x + blockIdx.y) % 8;
  const int at = (k * run + blockIdx.x / 8 % run) * 16 + threadIdx.x / 16;
  return at < Bs ? (nb - 1 - g % (nb - 1)) * Bs + at : -1;
}

// What a 16-lane group does with one value per key block, eight of them at a time: the dims' partial sums of all eight meet in
// the lane of the block (value u in lanes u and u + 8; three exchanges that halve the values and one addition, where a sum for
// every lane takes four for each value), the scalars of a block are worked out there once, and go back by a broadcast.
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float xor4_of(float v) {  // row_shl:4 into the even quads, row_shr:4 into the odd ones
  const int x = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0x5, false), x, 0x114, 0xf, 0xa, false));
}
__device__ __forceinline__ float sums_to_lanes(const float (&v)[8]) {  // added up in the order of group_sum
  const bool l4 = threadIdx.x & 4, l2 = threadIdx.x & 2, l1 = threadIdx.x & 1;
  float t[4], w[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) t[k] = (l1 ? v[2 * k + 1] : v[2 * k]) + dpp_of<0xB1>(l1 ? v[2 * k] : v[2 * k + 1]);  // quad_perm [1,0,3,2]
#pragma unroll
  for (int k = 0; k < 2; ++k) w[k] = (l2 ? t[2 * k + 1] : t[2 * k]) + dpp_of<0x4E>(l2 ? t[2 * k] : t[2 * k + 1]);  // quad_perm [2,3,0,1]
  const float x = (l4 ? w[1] : w[0]) + xor4_of(l4 ? w[0] : w[1]);
  return x + dpp_of<0x128>(x);  // row_ror:8
}
__device__ __forceinline__ float max_of_8(float x) {
  x = fmaxf(x, dpp_of<0x141>(x));
  x = fmaxf(x, dpp_of<0xB1>(x));
  return fmaxf(x, dpp_of<0x4E>(x));
}
__device__ __forceinline__ float sum_of_8(float x) {
  x += dpp_of<0x141>(x);
  x += dpp_of<0xB1>(x);
  return x + dpp_of<0x4E>(x);
}
// the lanes 0 .. 7 of the group where x holds
__device__ __forceinline__ unsigned lanes_of_8(bool x) { return (unsigned)(__ballot(x) >> (threadIdx.x % 64 / 16 * 16)) & 0xffu; }
// f(u, the value of lane u) for u < n; u is a constant
template <int n, typename F, int... U>
__device__ __forceinline__ void each_lane_(float x, F f, std::integer_sequence<int, U...>) {
  (f(U, dpp_of<0x150 + U>(x)), ...);  // row_newbcast
}
template <int n, typename F>
__device__ __forceinline__ void each_lane(float x, F f) {
  each_lane_<n>(x, f, std::make_integer_sequence<int, n>());
}

constexpr int kMaxCk = 2304;  // key clusters a kernel can index in LDS
static_assert(kMaxCk >= MUSE_MAX_CLUSTERS, "the host accepts more clusters than the kernels index");
constexpr int kKeys = 4;      // retrieved keys that the per-query kernels of fp32 inputs request together
constexpr int kRunTiles = 4;  // hit tiles (of 32) per work item of the retrieval forward / dq pair kernels
constexpr int kC3Slices = 8;  // most waves that share the hits of one retrieved pair in the key/value gradients
// hit slices of a pair in the key/value gradient kernels of the retrieval: one per `tiles` tiles of 32 hits, `most` at most
struct C3Cut {
  int tiles, most;
};
__host__ __device__ inline int c3_slices(int nhits, C3Cut cut) {
  const int nt = (nhits + 31) / 32;
  const int s = nt / cut.tiles;
  return s < 1 ? 1 : (s > cut.most ? cut.most : s);
}
// bytes of the far-field state of all queries, of the retrieval's partial rows per (query, slot), and of the partial
// dK | dV rows of one hit slice
static inline size_t ff_state_bytes(const MuseDims& d) { return (size_t)d.B * d.Hq * d.N * (d.D + 2) * 4; }
// The chain gradients' lists (backward, bf16 inputs) lie where that backward reads nothing.  Over the far-field state: the chains, r at most
// per query behind the first block and an end per query cluster, and a head per query cluster.  Over the maxima and sums behind the
// retrieval's partial rows: the entries, r per query.
static inline size_t ff_chains(const MuseDims& d) { return (size_t)d.B * d.Hq * ((size_t)(d.N - d.Bs) * d.r + d.Cq); }
static inline size_t ff_chain_bytes(const MuseDims& d) { return (ff_chains(d) + (size_t)d.B * d.Hq * d.Cq) * 8; }
static inline size_t ff_chain_list_bytes(const MuseDims& d) { return (size_t)d.B * d.Hq * d.N * d.r * 8; }
static inline size_t ff_ret_rows_bytes(const MuseDims& d) { return (size_t)d.B * d.Hq * d.N * (d.r > 0 ? d.r : 1) * d.k2e * d.D * 4; }
static inline size_t ff_ret_part_bytes(const MuseDims& d) {
  const size_t ml = ff_ret_rows_bytes(d) / d.D * 2;
  return ff_ret_rows_bytes(d) + (ml > ff_chain_list_bytes(d) ? ml : ff_chain_list_bytes(d));
}
static inline size_t ff_c3_slice_bytes(const MuseDims& d) { return (size_t)d.B * d.Hkv * d.N * 2 * d.D * 4; }
// Tiles per slice.  A further slice costs a partial row of dK and dV per key of the pair, written and read again (16 D bytes;
// the gathered rows of a tile of bf16 hits are 128 D: one tile's worth at 8 keys, eight at 64), so where the problem fills the
// device with long slices (4096 of them), they are long: at
// 16 heads of 64k tokens with 128 x 128 clusters 16 tiles against 4 take 1.22 + 0.16 ms (kernel + reduction) against
// 1.55 + 0.39, at 12 heads of 6k 4 tiles are what keeps the device busy.
// fp32 inputs have no partial rows per (query, slot): the slices take the room that bf16 inputs need for them and that of the
// forward's far-field state, which the backward does not read, and no more.
static inline C3Cut ff_c3_cut(const MuseDims& d) {
  const size_t tiles = (size_t)d.B * d.Hq * d.N * (d.r > 0 ? d.r : 1) * d.k2e / 32 / 4096;
  const size_t later = d.dtype == MUSE_DTYPE_BF16 ? kC3Slices - 1 : (ff_state_bytes(d) + ff_ret_part_bytes(d)) / ff_c3_slice_bytes(d);
  return {tiles < 4 ? 4 : tiles > 16 ? 16 : (int)tiles, later < kC3Slices - 1 ? 1 + (int)later : kC3Slices};
}

struct FFWorkspace {
  // all heads
  int32_t *perm_k, *off_k, *perm_q, *off_q, *tile_off;
  void *Ks, *Vs;      // keys / values in bucketed order, input dtype
  float *ff_acc, *ff_ml;  // contiguous: [HQ,N,D] then [HQ,N,2]
  // backward only, all heads
  float* delta;
  uint32_t* selmask;   // [HQ][W][N] by bucketed query position
  int32_t* slotinfo;   // [HQ][N][r] by bucketed query position: cluster | retrieved-block mask << 16
  int32_t* pair_off;             // inverse index of the retrieval: (kv head, key block, key cluster) -> hits
  int32_t* pair_cnt;             // hits per pair, [HK][pairs + 1]
  int32_t* run_off;              // [HK][pairs + 1]: first work item of every pair, [pairs] = their number
  int4* run_map;                 // [HK][run_cap]: (pair, first hit, end) of a work item; bf16 inputs
  int32_t* c3_off;               // [HK][pairs + 1]: first (pair, hit slice) item of every pair, [pairs] = their number
  int2* c3_map;                  // [HK][run_cap]: (pair, slice) items of the key/value gradient kernel
  size_t run_cap;                // work items per kv head the map can hold
  int32_t *seg_cnt, *seg_off;    // its construction: counts / list starts [HK][head of the group x query slice][pair]
  uint2* hits;                   // x = n | g << 22 (query position, head inside the KV group), y = slot*k2e + u
  size_t hit_cap;                // hits per kv head
  float* ret_part;               // bf16 inputs, per (query, slot, u): forward partial rows [D], then (max, sum) [2] of all rows; or dq partial rows [D]
  uint2 *chains, *lists;         // lists of the chain gradients, bf16 inputs: in ff_acc and behind the rows of ret_part
  int2* head_of;                 // [HQ][Cq]: in ff_acc
  float *dKs, *dVs;            // fp32 gradients in bucketed key order
  float* c3_part;              // r > 0: [slices - 1][HK][N][2][D] partial dK | dV rows of the later hit slices of a pair (fp32: over ff_acc)
  float *dQacc, *dKacc, *dVacc;  // fp32 gradients in sequence order (alias the outputs when they are fp32)
  float* dQff;                   // r > 0: component 1's part of dQ, which k_comp2_bwd_dq adds to dQacc with its own (r = 0: k_ff_bwd_dq adds it, unused)
  void* qcb;                     // bf16 [hc][Cq padded to 32][D]: scaled query centroids of a head chunk
  // per chunk of `hc` query heads
  float* L;
  uint32_t* chainmask;  // [hc][Cq][ceil(Ck/32)]: key clusters retrieved by some query of the query cluster
  uint32_t* chainmaskT;  // [hc][Ck][ceil(Cq/32)]: the same bits, key-cluster-major
  // Value summaries and cell gradients are stored in the input type.  The accumulated k-bar decides
  // selections: fp32 inputs keep it in fp32 (A_k); bf16 inputs keep a bf16 plane A_kb (also the operand of the
  // gradient contractions), an fp16 plane A_km of the remainder and the scalar A_c = mu-bar - scale * qc_i . k-bar
  // per cell.
  float *s_mu, *s_k, *A_mu, *A_k, *A_c;
  void *s_v, *A_v, *A_kb, *A_km;
  float* g_s_c;
  void *g_s_k, *g_s_v;
  float *g_A_c, *g_A_k, *g_A_v;  // gradients of the accumulated cells; fp32 inputs (bf16: never leave the kernel)
  // dipole correction (MUSE_FLAG_DIPOLE): untilted covariances [HK][nb-1][Ck][D][D] (all heads) and the merged
  // matrices [hc][nb-1][Cq][D][D] of a head chunk
  float *dip_cov, *dip_cbar;
  int hc;
};

static inline size_t ff_al(size_t x) { return (x + 255) & ~(size_t)255; }

// query-range slices per head when the hit lists of the retrieval are built: enough (slice, head) waves to fill
// the device, every slice a whole number of 64-query chunks
static inline int ff_hit_segments(const MuseDims& d) {
  const int HQ = d.B * d.Hq, chunks = (d.N - d.Bs + 63) / 64;
  int seg = (2048 + HQ - 1) / HQ;
  seg = seg > chunks ? chunks : seg;
  return seg < 1 ? 1 : seg;
}
// most work items (runs of kRunTiles hit tiles inside one pair) a kv head can have
static inline size_t ff_run_cap(const MuseDims& d) {
  size_t NBm = d.nb > 1 ? d.nb - 1 : 1, R2 = (size_t)(d.r > 0 ? d.r : 1) * d.k2e;
  size_t npair = NBm * d.Ck, hits = (size_t)(d.Hq / d.Hkv) * d.N * R2;
  return (hits / 32 + npair) / kRunTiles + npair + 1;
}
// the forward of fp32 inputs reads the retrieved keys per query, without the inverse index
static inline bool ff_has_index(const MuseDims& d, bool bwd) { return bwd || d.dtype == MUSE_DTYPE_BF16; }
// bytes of the far-field state and of what the backward keeps in the same place: the slices' partial rows (fp32 inputs) or the chains
static inline size_t ff_acc_bytes(const MuseDims& d, bool bwd) {
  const size_t a = ff_state_bytes(d), c3 = (ff_c3_cut(d).most - 1) * ff_c3_slice_bytes(d);
  const size_t later = d.dtype == MUSE_DTYPE_FP32 ? c3 : ff_chain_bytes(d);
  return bwd && d.r > 0 && d.nb > 1 && later > a ? later : a;
}
// bytes of the segment counters of the inverse index
static inline size_t ff_segcnt_bytes(const MuseDims& d) {
  size_t HK = (size_t)d.B * d.Hkv, NBm = d.nb > 1 ? d.nb - 1 : 1;
  return HK * (d.Hq / d.Hkv) * ff_hit_segments(d) * NBm * d.Ck * 4;
}

// bytes of the all-heads part / of one query head of the chunked part
// x extent of the forward tile kernels' grid: the tiles of a (head, block) pair, rounded up to the 8 XCDs
static inline size_t ff_tile_grid_x(const MuseDims& d) { return (size_t)(d.Bs / 32 + d.Cq + 1 + 7) / 8 * 8; }
// the grid of far_position (nb > 1)
static inline dim3 far_grid(const MuseDims& d, int hn) {
  const int round = 16 * 8 * far_run(d.Bs);  // queries of a block in a run for every XCD
  return dim3((d.Bs + round - 1) / round * 8 * (d.nb - 1) * far_run(d.Bs), hn);
}
static inline size_t ff_fixed_bytes(const MuseDims& d, bool bwd) {
  size_t HQ = (size_t)d.B * d.Hq, HK = (size_t)d.B * d.Hkv, N = d.N, D = d.D;
  size_t es = d.dtype == MUSE_DTYPE_BF16 ? 2 : 4;
  size_t W = (d.Ck + 31) / 32, NBm = d.nb > 1 ? d.nb - 1 : 1, R2 = (size_t)(d.r > 0 ? d.r : 1) * d.k2e;
  size_t b = ff_al(HK * N * 4) + ff_al(HK * ((size_t)d.nb * d.Ck + 1) * 4) + ff_al(HQ * N * 4) +
             ff_al(HQ * ((size_t)d.nb * d.Cq + 1) * 4) + ff_al(HQ * d.nb * ((size_t)d.Cq + 1) * 4) +
             2 * ff_al(HK * N * D * es) + ff_al(ff_acc_bytes(d, bwd));
  // inverse index of the retrieval and, for bf16 inputs, its per-(query, slot) partial results
  if (ff_has_index(d, bwd))
    b += 4 * ff_al(HK * ((size_t)d.nb * d.Ck + 1) * 4) + 2 * ff_al(ff_segcnt_bytes(d)) +
         ff_al(HK * ff_run_cap(d) * 8) + ff_al(HQ * N * R2 * 8);
  if (es == 2) b += ff_al(HK * ff_run_cap(d) * 16) + ff_al(ff_ret_part_bytes(d));
  if (bwd) {
    b += ff_al(HQ * N * 4) + ff_al(HQ * N * W * 4) + ff_al(HQ * N * (size_t)(d.r > 0 ? d.r : 1) * 4) + 2 * ff_al(HK * N * D * 4) +
         ff_al(HQ * N * D * 4) + ff_al(HQ * D * (size_t)((d.Cq + 31) / 32 * 32) * 2);
    if (d.grad_dtype != MUSE_DTYPE_FP32) b += ff_al(HQ * N * D * 4) + 2 * ff_al(HK * N * D * 4);
    if (es == 2 && d.r > 0 && d.nb > 1) b += ff_al((kC3Slices - 1) * ff_c3_slice_bytes(d));
  }
  if (d.dipole) b += ff_al(HK * NBm * d.Ck * D * D * 4);
  return b;
}

static inline size_t ff_head_bytes(const MuseDims& d, bool bwd) {
  size_t cells = (size_t)(d.nb > 1 ? d.nb - 1 : 1) * d.Cq * d.Ck, D = d.D;
  size_t es = d.dtype == MUSE_DTYPE_BF16 ? 2 : 4;
  size_t b = ff_al((size_t)d.Cq * d.N * 4) + ff_al((size_t)d.Cq * ((d.Ck + 31) / 32) * 4) + ff_al((size_t)d.Ck * ((d.Cq + 31) / 32) * 4) + 2 * ff_al(cells * 4) + ff_al(cells * D * 4) + 2 * ff_al(cells * D * es);
  b += es == 2 ? 2 * ff_al(cells * D * 2) + ff_al(cells * 4) : ff_al(cells * D * 4);
  if (bwd) b += (es == 2 ? 1 : 2) * (ff_al(cells * 4) + 2 * ff_al(cells * D * es));
  if (d.dipole) b += ff_al((size_t)(d.nb > 1 ? d.nb - 1 : 1) * d.Cq * D * D * 4);
  return b;
}

// farfield.hip
int muse_ff_carve(const MuseDims& d, bool bwd, void* ws, size_t ws_bytes, FFWorkspace* w, void* dQ, void* dK, void* dV);
template <typename T>
int muse_ff_prepare(const MuseDims& d, const T* K, const T* V, const int32_t* aq, const int32_t* ak, FFWorkspace& w,
                    hipStream_t st);
template <typename T>
int muse_ff_summaries(const MuseDims& d, const float* qc, FFWorkspace& w, int h0, int hn, hipStream_t st);
// farfield_tiles.hip: the far-field forward's tile kernel of bf16 inputs
int muse_launch_farfield_tiles(const MuseDims& d, const void* Q, const FFWorkspace& w, int32_t* selc, int h0, int hn,
                               hipStream_t st);
template <typename T>
int muse_ff_block_summaries(const MuseDims& d, const int32_t* selc, FFWorkspace& w, int h0, int hn, bool cleared, hipStream_t st);  // cleared: w.chainmask is all zeros

// cell_grads.hip: component 1 of the per-block cell gradients, bf16 inputs, of the query heads [h0, h0+hn)
int muse_launch_ff_bwd_cells_mx(const MuseDims& d, const void* Q, const void* dO, const float* qc, const float* LSE,
                                FFWorkspace& w, int h0, int hn, hipStream_t st);
// chain_grads.hip: component 2 of the per-block cell gradients of the query heads [h0, h0+hn)
template <typename T>
int muse_launch_chain_grads(const MuseDims& d, const T* Q, const T* dO, const float* qc, const float* LSE, FFWorkspace& w,
                            int h0, int hn, hipStream_t st);

// retrieval_kv.hip
int muse_launch_c3_pairs(const MuseDims& d, const void* Q, const void* dO, const float* LSE, FFWorkspace& w, hipStream_t st);
// adds the partial rows of the later hit slices of every pair to dKs, dVs
int muse_launch_c3_reduce(const MuseDims& d, FFWorkspace& w, hipStream_t st);
// retrieval_fp32.hip
int muse_launch_c3_pairs_f32(const MuseDims& d, const float* Q, const float* dO, const float* LSE, FFWorkspace& w, hipStream_t st);
// retrieval_q.hip
int muse_launch_ret_fwd_pairs(const MuseDims& d, const void* Q, const void* Ks, const void* Vs, const int32_t* off_k,
                              const int32_t* run_off, const int4* run_map, size_t run_cap, const uint2* hits,
                              size_t hit_cap, float* part, hipStream_t st);
int muse_launch_ret_bwd_dq_pairs(const MuseDims& d, const void* Q, const void* dO, const void* Ks, const void* Vs,
                                 const float* LSE, const float* delta, const int32_t* off_k, const int32_t* run_off,
                                 const int4* run_map, size_t run_cap, const uint2* hits, size_t hit_cap, float* dqpart,
                                 hipStream_t st);
// attn_mfma.hip
int muse_launch_cells_to_keys_mx(const MuseDims& d, const void* Ks, const void* Vs, const float* qc, void* qcb,
                                 const float* L, const float* s_mu, const float* G_c, const void* G_k, const void* G_v,
                                 const int32_t* off_k, const int32_t* perm_k, float* dKs, float* dVs, float* dK, float* dV, int h0, int hn,
                                 hipStream_t st);
// dipole.hip: dipole correction of the monopole-only mode (App. B), forward
template <typename T>
int muse_dipole_covariances(const MuseDims& d, FFWorkspace& w, hipStream_t st);
template <typename T>
int muse_dipole_apply(const MuseDims& d, const T* Q, const float* qc, const int32_t* aq, FFWorkspace& w, int h0, int hn,
                      hipStream_t st);
// retrieval.hip: ordered hit lists and work items from the exported selections; merge of the forward partials
int muse_ff_build_inverse_index(const MuseDims& d, const int32_t* selc, const int32_t* selb, FFWorkspace& w, hipStream_t st);
int muse_launch_merge_ret(const MuseDims& d, const int32_t* selb, const float* part, float* ff_acc, float* ff_ml,
                          hipStream_t st);
