// bf16 causal attention on MFMA (Sec. 3, Eq. 1-2; Sec. 3.3 "Local attention"): keys restricted to
// the query's own spatial block of size Bs (Bs = N gives exact attention).  The two backward
// kernels (dQ per query tile, dK/dV per key tile; no atomics) in tiles of 128 rows, for short blocks and few
// tiles; attn_bwd.hip has the others, and says where the line is.  The forward is in attn_fwd.hip.
//
// Tiling for 64-wide waves and v_mfma_f32_32x32x16_bf16:
//   - a wave owns 32 queries (dQ) or 32 keys (dK/dV) as the N-columns of the MFMA, so every
//     per-row softmax quantity lives in one lane (two lanes: the two halves hold different K-rows);
//   - scores are produced transposed (S^T = K Q^T in dQ, S = Q K^T in dK/dV) so that their
//     accumulator layout IS the B-operand layout of the following contraction: probabilities go
//     from registers straight back into the matrix cores, never through LDS;
//   - accumulator element e of lane l is row 8*(e/4) + 4*(l/32) + e%4, column l%32; an operand
//     lane holds 8 consecutive k for k-slot-half l/32.  For the second contraction the 8 k-slots of
//     half h over 16 keys are keys {4h..4h+3} and {8+4h..8+4h+3}: a permutation applied to both
//     operands, which a contraction does not see.
#include "ff_common.h"
#include "flash_tile.h"
#include "lds_tile.h"

namespace {

constexpr int BN = 64;  // rows staged in LDS per step

// Staging of a tile through registers, so that the global loads of the next tile are in flight while the current one is
// consumed: fetch_rows into registers, commit_rows from registers into LDS.  The registers are named members,
// not an array: an array that is passed around and read through pointer casts ends up in memory (the compiler
// parks it in LDS), and the wait for its loads then comes right after they are issued.
struct TileRegs {
  uint4 a, b, c, d;
};

// Transposed tile in operand order.  The second contraction of the backward kernels takes, for lane half h and the
// 16 rows r0 .. r0+15 of the staged tile, the rows r0 + {4h .. 4h+3} and r0 + {8+4h .. 8+4h+3} as its 8 k-slots.
// Stored in that order (inside every group of 16 rows the bits 2 and 3 of the row index change places) an operand
// is one 16-byte read instead of two 8-byte ones; an LDS instruction costs about the same whatever its width, and
// LDS instructions, not bytes, are what these kernels run out of.  Rows are padded to a multiple of 16 bytes.
constexpr int TPAD16 = 8;
__device__ __forceinline__ int tr_pos(int row) { return (row & ~12) | ((row & 4) << 1) | ((row & 8) >> 1); }
// rows 2r and 2r+1 (chunk cc of each) into the row-major tile, and their 8 columns into the transposed tile as
// 4-byte stores of two neighbouring rows (they stay neighbours in operand order)
template <int D, int ROWS>
__device__ __forceinline__ void commit_pair(const uint4 a, const uint4 b, int r, int cc, bf16_t (*rm)[D + 8],
                                            bf16_t (*tr)[ROWS + TPAD16]) {
  *reinterpret_cast<uint4*>(&rm[2 * r][cc * 8]) = a;
  *reinterpret_cast<uint4*>(&rm[2 * r + 1][cc * 8]) = b;
  const uint32_t wa[4] = {a.x, a.y, a.z, a.w}, wb[4] = {b.x, b.y, b.z, b.w};
  const int pos = tr_pos(2 * r);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    *reinterpret_cast<uint32_t*>(&tr[cc * 8 + 2 * i][pos]) = __builtin_amdgcn_perm(wb[i], wa[i], 0x05040100u);
    *reinterpret_cast<uint32_t*>(&tr[cc * 8 + 2 * i + 1][pos]) = __builtin_amdgcn_perm(wb[i], wa[i], 0x07060302u);
  }
}
// the operand of lane half `half` over the 16 rows starting at r0 (a multiple of 16)
template <int W>
__device__ __forceinline__ bf16x8_t ld_tr16(const bf16_t (*tr)[W], int d, int r0, int half) {
  return *reinterpret_cast<const bf16x8_t*>(&tr[d][r0 + 8 * half]);
}

// Which row pair and which 16-byte chunk the c-th of a tile's (ROWS / 2) x (D / 8) staging units is: consecutive
// lanes take consecutive pairs of one chunk.  The 4-byte transposed stores of 32 lanes then fall into 32 different
// banks; the 16-byte row stores (lanes 288 bytes apart) pay a two-way conflict, 14 % of their time in a
// microbenchmark, where a mapping that spares them doubles the time of the transposed stores.
template <int D, int ROWS>
__device__ __forceinline__ void pair_unit(int c, int& pr, int& pc) {
  pr = c % (ROWS / 2);
  pc = c / (ROWS / 2);
}

// A tile as it lies: chunk c = thread + 256 i is chunk c % (D / 8) of row c / (D / 8), so a load instruction takes whole rows,
// and the tile in LDS (lds_tile.h) serves rows and transposed operands alike.
template <int D>
__device__ __forceinline__ uint4 fetch_row_chunk(const bf16_t* __restrict__ src, int r0, int N, int i) {
  const int c = threadIdx.x + 256 * i;
  return *reinterpret_cast<const uint4*>(src + (size_t)min(r0 + c / (D / 8), N - 1) * D + c % (D / 8) * 8);
}
template <int D>
__device__ __forceinline__ void fetch_rows(const bf16_t* __restrict__ src, int r0, int N, TileRegs& r) {
  static_assert(BN * (D / 8) / 256 == (D == 64 ? 2 : 4), "chunks per thread");
  r.a = fetch_row_chunk<D>(src, r0, N, 0);
  r.b = fetch_row_chunk<D>(src, r0, N, 1);
  if constexpr (D == 128) {
    r.c = fetch_row_chunk<D>(src, r0, N, 2);
    r.d = fetch_row_chunk<D>(src, r0, N, 3);
  }
}
template <int D>
__device__ __forceinline__ void commit_row_chunk(const uint4 v, int i, bf16_t* tile) {
  const int c = threadIdx.x + 256 * i;
  *reinterpret_cast<uint4*>(tile + tile_at<D>(c / (D / 8), c % (D / 8))) = v;
}
template <int D>
__device__ __forceinline__ void commit_rows(const TileRegs& r, bf16_t* tile) {
  commit_row_chunk<D>(r.a, 0, tile);
  commit_row_chunk<D>(r.b, 1, tile);
  if constexpr (D == 128) {
    commit_row_chunk<D>(r.c, 2, tile);
    commit_row_chunk<D>(r.d, 3, tile);
  }
}

// dQ.  The matrix pipe is 0.53 to 0.57 busy at D = 64 (0.50 at D = 128), the vector pipe 0.68; what the matrix pipe waits for is the
// vector work between S and dQ and the LDS reads in front of it (no bank conflicts), which three (D = 128: two) waves per SIMD
// cover in part.  Keys lie in LDS once, row-major, for
// both contractions; with a transposed copy (4-byte stores in row pairs, half of the LDS-active cycles in bank conflicts) and
// two barriers per step it took, us before -> after, 989 -> 927 for exact attention of 32 heads of 8k, D = 128, 482 -> 460 at
// 8 heads of 16k, 1821 -> 1779 at 16 heads of 64k in blocks of 8192, 3560 -> 3376 at 32; same bits.
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, D == 64 ? 3 : 2))) k_flash_bwd_dq(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                                       const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
                                                       const float* __restrict__ LSE, const float* __restrict__ delta,
                                                       float* __restrict__ dQ, int N, int Bs, int Hq, int Hkv,
                                                       int nbatch, float scale, float scale_log2e) {
  constexpr int KS = D / 16, DT = D / 32;
  __shared__ __attribute__((aligned(256))) bf16_t ks[2][BN * D];
  __shared__ __attribute__((aligned(256))) bf16_t vs[2][BN * D];
  const FlashTile ft = flash_tile(N, Bs, Hq, nbatch);
  if (!ft.ok) return;
  const int hq = ft.h, b = ft.b, hk = hq / (Hq / Hkv);
  const size_t qh = ((size_t)b * Hq + hq) * N, kh = ((size_t)b * Hkv + hk) * N;
  const int q0 = (ft.blk * ft.tpg + ft.tpg - 1 - ft.t) * 128;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const int nq = q0 + 32 * wave + col;
  const int nqc = nq < N ? nq : N - 1;
  const int myb = (nqc / Bs) * Bs;

  bf16x8_t qf[KS], gf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    qf[s] = *reinterpret_cast<const bf16x8_t*>(Q + (qh + nqc) * D + 16 * s + 8 * half);
    gf[s] = *reinterpret_cast<const bf16x8_t*>(dO + (qh + nqc) * D + 16 * s + 8 * half);
  }
  const float lse2 = LSE[qh + nqc] * 1.4426950408889634f, dl = delta[qh + nqc];
  const bool unaligned = (Bs % 128) != 0;
  f32x16_t dq[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[t][e] = 0.f;

  const int kbeg = (q0 / Bs) * Bs, kend = min(q0 + 128, N);
  const bf16_t *Kh = K + kh * D, *Vh = V + kh * D;
  // two tiles in LDS, a third on its way in registers: a step has one barrier, the next tile is written in its middle
  TileRegs kreg, vreg;
  fetch_rows<D>(Kh, kbeg, N, kreg);
  fetch_rows<D>(Vh, kbeg, N, vreg);
  commit_rows<D>(kreg, ks[0]);
  commit_rows<D>(vreg, vs[0]);
  fetch_rows<D>(Kh, kbeg + BN, N, kreg);
  fetch_rows<D>(Vh, kbeg + BN, N, vreg);
  int buf = 0;
  for (int k0 = kbeg; k0 < kend; k0 += BN, buf ^= 1) {
    __syncthreads();
    const bool live = k0 <= q0 + 32 * wave + 31;  // wave-uniform
    const bool edge = unaligned || k0 + BN - 1 > q0 + 32 * wave || k0 + BN > N;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      if (kt == 1) {  // past the end: some row of the sequence that nobody reads
        commit_rows<D>(kreg, ks[buf ^ 1]);
        commit_rows<D>(vreg, vs[buf ^ 1]);
        fetch_rows<D>(Kh, k0 + 2 * BN, N, kreg);
        fetch_rows<D>(Vh, k0 + 2 * BN, N, vreg);
      }
      if (!live) continue;
      f32x16_t s, dp;
#pragma unroll
      for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
      for (int x = 0; x < KS; ++x) {
        bf16x8_t a = tile_row<D>(ks[buf], 32 * kt + col, 2 * x + half);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[x], s, 0, 0, 0);
        bf16x8_t av = tile_row<D>(vs[buf], 32 * kt + col, 2 * x + half);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, gf[x], dp, 0, 0, 0);
      }
      if (edge) {  // wave-uniform: only tiles on the diagonal or at the sequence end hold masked entries
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          int kg = k0 + 32 * kt + 8 * (e / 4) + 4 * half + (e % 4);
          if (kg > nq || kg < myb) s[e] = MUSE_NEG_INF;  // p = 0
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p = fast_exp2(fmaf(s[e], scale_log2e, -lse2));
        s[e] = p * (dp[e] - dl);
      }
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        bf16x8_t df = pack8(s, 2 * G, 2 * G + 1);
#pragma unroll
        for (int t = 0; t < DT; ++t) {
          bf16x8_t a = tile_cols<D>(ks[buf], 32 * kt + 16 * G, t, lane);
          dq[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, df, dq[t], 0, 0, 0);
        }
      }
    }
  }
  if (nq >= N) return;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // every query row belongs to exactly one tile: the row is written, not added to
      *reinterpret_cast<float4*>(dQ + (qh + nq) * D + 32 * t + 8 * g + 4 * half) =
          make_float4(scale * dq[t][4 * g + 0], scale * dq[t][4 * g + 1], scale * dq[t][4 * g + 2], scale * dq[t][4 * g + 3]);
    }
}

// dK/dV for D = 128 in short blocks.  One wave with dK and dV of its 32 keys needs 128 accumulator registers beside 64 of keys and values:
// one wave per SIMD, and nothing runs while it waits.  So two waves share 32 keys: wave w computes P = exp2(c (Q K^T - LSE))
// and dV += P^T dO, wave w + 4 (on the same SIMD) dP = dO V^T and, a step behind, dS = P dP and dK += dS^T Q; P passes
// between them through LDS in fp32, one barrier per step of 32 queries.  A step's rows are staged once, row-major for both
// operand forms (lds_tile.h): Q in three buffers (next, current, the one dK still reads), dO in two.  The accumulators of S
// and dP start at -LSE / scale and -delta.  The query heads of the group follow one another in one sequence of steps.
// Matrix pipe 0.45 busy, LDS 0.4, vector 0.4: the three share the time between barriers.  One wave per 32 keys and SIMD with
// 32 queries staged per two barriers took 1.75 ms at 32 heads of 8k tokens (8 KV heads, exact attention), this 1.39;
// 3.57 -> 2.82 ms at 32k tokens in blocks of 4096.  One wave per SIMD with the next scores issued between the vector
// instructions of the current ones took 1.51, this kernel with each role pipelined over two steps 2.09 (spills).
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) k_flash_bwd_dkv128(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
    const float* __restrict__ LSE, const float* __restrict__ delta, float* __restrict__ dK, float* __restrict__ dV, int N,
    int Bs, int Hq, int Hkv, int nbatch, float scale, float scale_log2e) {
  constexpr int D = 128, KS = D / 16, DT = D / 32, BQ = 32, kTile = BQ * D;
  __shared__ __attribute__((aligned(16))) bf16_t qs[3][kTile];
  __shared__ __attribute__((aligned(16))) bf16_t gs[3][kTile];     // two buffers and a tile of zeros
  __shared__ __attribute__((aligned(16))) float4 px[2][4][4][64];  // P of a step: [wave pair][4 rows][lane]
  __shared__ __attribute__((aligned(16))) float seeds[3][2][BQ];   // -LSE / scale, -delta; zeros
  const FlashTile ft = flash_tile(N, Bs, Hkv, nbatch);
  if (!ft.ok) return;
  const int hk = ft.h, b = ft.b, G_ = Hq / Hkv;
  const size_t kh = ((size_t)b * Hkv + hk) * N;
  const int k0 = (ft.blk * ft.tpg + ft.t) * 128;  // the first key tiles of a block see the most queries
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, col = lane % 32, half = lane / 32;
  const int kw = w % 4;
  const bool second = w >= 4;  // dP and dK
  const int mk = k0 + 32 * kw + col;
  const int mkc = mk < N ? mk : N - 1;
  const int nlen = min((mkc / Bs + 1) * Bs, N) - mk;  // the key's queries are mk .. mk + nlen - 1
  const int qend = min((min(k0 + 127, N - 1) / Bs + 1) * Bs, N);
  const int nq = (qend - k0 + BQ - 1) / BQ, nt = G_ * nq;  // steps per query head, steps of the group
  // a tile of 128 keys inside one block with every row in range: only the diagonal needs a mask
  const bool aligned = (Bs % 128) == 0 && k0 + 128 <= N;
  const float seed = -1.4426950408889634f / scale_log2e;

  bf16x8_t kv[KS];
#pragma unroll
  for (int x = 0; x < KS; ++x) kv[x] = *reinterpret_cast<const bf16x8_t*>((second ? V : K) + (kh + mkc) * D + 16 * x + 8 * half);
  f32x16_t acc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) acc[t] = zero16();

  uint4 qr, gr;  // this thread's chunk of row tid / 16 of a coming step
  float lr = 0.f;
  const int sr = tid / 16, sc = tid % 16;
  const size_t qh0 = ((size_t)b * Hq + (size_t)hk * G_) * N;
  const bf16_t *qp = Q + qh0 * D + 8 * sc, *gp = dO + qh0 * D + 8 * sc;
  const float* lp = ((tid / BQ) % 2 ? delta : LSE) + qh0;
  int fq = k0;  // first query of the next step to fetch
  auto fetch = [&]() {
    const int row = min(fq + sr, N - 1);
    qr = *reinterpret_cast<const uint4*>(qp + (size_t)row * D);
    gr = *reinterpret_cast<const uint4*>(gp + (size_t)row * D);
    lr = lp[min(fq + tid % BQ, N - 1)];
    fq += BQ;
    if (fq >= qend) {  // on to the next query head
      fq = k0;
      qp += (size_t)N * D;
      gp += (size_t)N * D;
      lp += N;
    }
  };
  auto commit = [&](int bq, int bg) {
    const int at = tile_at<D>(sr, sc);
    *reinterpret_cast<uint4*>(qs[bq] + at) = qr;
    *reinterpret_cast<uint4*>(gs[bg] + at) = gr;
    if (tid < 2 * BQ) seeds[bg][tid / BQ][tid % BQ] = lr * (tid < BQ ? seed : -1.f);
  };
  // 32 staged rows times the wave's keys or values
  auto scores = [&](const bf16_t* rows, const float* sd) {
    f32x16_t s;
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const float4 x = *reinterpret_cast<const float4*>(sd + 8 * gq + 4 * half);
      s[4 * gq + 0] = x.x; s[4 * gq + 1] = x.y; s[4 * gq + 2] = x.z; s[4 * gq + 3] = x.w;
    }
#pragma unroll
    for (int x = 0; x < KS; ++x) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(rows, col, 2 * x + half), kv[x], s, 0, 0, 0);
    return s;
  };
  const int rr = 4 * half + (lane % 16) / 4, cc = 16 * ((lane / 16) % 2) + 4 * (lane % 4);
  auto grads = [&](const bf16_t* rows, const f32x16_t& p) {  // acc += rows^T p
#pragma unroll
    for (int G = 0; G < 2; ++G) {
      const bf16x8_t pf = pack8(p, 2 * G, 2 * G + 1);
#pragma unroll
      for (int t = 0; t < DT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            tr_join(tile_tr4<D>(rows, 16 * G + rr, 32 * t + cc), tile_tr4<D>(rows, 16 * G + rr + 8, 32 * t + cc)), pf, acc[t], 0, 0, 0);
    }
  };
  f32x16_t dp = zero16();
  auto finish = [&](const bf16_t* rows, int bp) {  // dS of a step from its P and dP, into dK
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const float4 p = px[bp][kw][gq][lane];
      dp[4 * gq] *= p.x; dp[4 * gq + 1] *= p.y; dp[4 * gq + 2] *= p.z; dp[4 * gq + 3] *= p.w;
    }
    grads(rows, dp);
  };
  *reinterpret_cast<uint4*>(gs[2] + 8 * tid) = make_uint4(0u, 0u, 0u, 0u);
  if (tid < 2 * BQ) seeds[2][tid / BQ][tid % BQ] = 0.f;
  fetch();
  commit(0, 0);
  __syncthreads();
  if (nt > 1) fetch();
  int bq = 0, q0 = k0;
  for (int T = 0; T < nt; ++T) {
    const int bn = bq == 2 ? 0 : bq + 1, bl = bq == 0 ? 2 : bq - 1, bg = T & 1;
    if (T + 1 < nt) commit(bn, bg ^ 1);  // buffers last read before the previous barrier
    if (T + 2 < nt) fetch();
    // A step whose queries all precede the wave's keys reads the zeros: P is zero there, and a row that is not finite must
    // not reach the keys as 0 * inf.  (Left out by a branch, the step cost 1.6 % of exact attention at 8k tokens.)  The step
    // before this one was the last of a query head where this is its first.
    const int bz = q0 + BQ > k0 + 32 * kw ? bg : 2;
    if (!second) {
      f32x16_t s = scores(qs[bq], seeds[bg][0]);
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = fast_exp2(s[e] * scale_log2e);
      if (!aligned || q0 < k0 + 32 * kw + 32) {
        const int nm = q0 + 4 * half - mk;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = (unsigned)(nm + 8 * (e / 4) + e % 4) < (unsigned)nlen ? s[e] : 0.f;
      }
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) px[bg][kw][gq][lane] = make_float4(s[4 * gq], s[4 * gq + 1], s[4 * gq + 2], s[4 * gq + 3]);
      grads(gs[bz], s);
    } else {
      if (T > 0) finish(q0 == k0 || q0 > k0 + 32 * kw ? qs[bl] : gs[2], bg ^ 1);
      dp = scores(gs[bz], seeds[bz][1]);
    }
    __syncthreads();
    bq = bn;
    q0 = q0 + BQ < qend ? q0 + BQ : k0;
  }
  if (second) finish(qs[bq == 0 ? 2 : bq - 1], (nt - 1) & 1);
  if (mk >= N) return;
  float* out = (second ? dK : dV) + (kh + mk) * D;
  const float mul = second ? scale : 1.f;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      // every key row belongs to exactly one tile (the query heads of the group are summed in registers)
      *reinterpret_cast<float4*>(out + 32 * t + 8 * g + 4 * half) =
          make_float4(mul * acc[t][4 * g + 0], mul * acc[t][4 * g + 1], mul * acc[t][4 * g + 2], mul * acc[t][4 * g + 3]);
}

// dK/dV of the block diagonal for D = 64, arranged in phases so that a wave never waits for LDS right before a
// matrix instruction, and with the fewest vector instructions per score.  For a tile of 32 queries:
//   A  8 MFMAs   S = Q K^T and dP = dO V^T.  Their accumulators start at -LSE / scale and -delta (read from LDS
//                straight into the accumulator registers), so the probability is exp2(c S) and dS = P dP with no
//                further subtraction;
//   B  vector    P, dS, conversion to bf16 operands; the causal mask only on the tiles the diagonal crosses;
//   C  8 MFMAs   dV += P^T dO, dK += dS^T Q.
// The transposed operands of C are requested before B, the accumulator seeds and row operands of the next tile
// during C, so each request is in flight across a whole phase.  Two staged tiles of 64 queries: while one is
// consumed the next is written into the other (in the middle of the tile, when its global loads have landed) and
// the one after that is requested from memory, so a tile costs one barrier.  With two waves per SIMD the vector
// phase of one wave runs beside the matrix phases of the other.
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) k_flash_bwd_dkv_p(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ delta,
    float* __restrict__ dK, float* __restrict__ dV, int N, int Bs, int Hq, int Hkv, int nbatch, float scale,
    float scale_log2e) {
  constexpr int KS = D / 16, DT = D / 32;
  constexpr int BQ = 64, NQT = BQ / 32;
  __shared__ __attribute__((aligned(16))) bf16_t qs[2][BQ][D + 8];
  __shared__ __attribute__((aligned(16))) bf16_t gs[2][BQ][D + 8];
  __shared__ __attribute__((aligned(16))) bf16_t qt_[2][D][BQ + TPAD16];
  __shared__ __attribute__((aligned(16))) bf16_t gt_[2][D][BQ + TPAD16];
  __shared__ __attribute__((aligned(16))) float lse_s[2][BQ];  // -LSE / scale
  __shared__ __attribute__((aligned(16))) float dl_s[2][BQ];   // -delta
  const FlashTile ft = flash_tile(N, Bs, Hkv, nbatch);
  if (!ft.ok) return;
  const int hk = ft.h, b = ft.b, G_ = Hq / Hkv;
  const size_t kh = ((size_t)b * Hkv + hk) * N;
  const int k0 = (ft.blk * ft.tpg + ft.t) * 128;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const int mk = k0 + 32 * wave + col;
  const int mkc = mk < N ? mk : N - 1;
  const int myend = min((mkc / Bs + 1) * Bs, N);
  const int qend = min((min(k0 + 127, N - 1) / Bs + 1) * Bs, N);
  // a tile of 128 keys inside one block with every row in range: only the diagonal needs a mask
  const bool aligned = (Bs % 128) == 0 && k0 + 128 <= N;
  const float seed = -1.4426950408889634f / scale_log2e;
  static_assert(BQ / 2 * (D / 8) == 256, "one pair of rows and one 16-byte chunk per thread");
  int pr_, pc_;  // row pair and chunk this thread stages
  pair_unit<D, BQ>(threadIdx.x, pr_, pc_);

  bf16x8_t kf[KS], vf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    kf[s] = *reinterpret_cast<const bf16x8_t*>(K + (kh + mkc) * D + 16 * s + 8 * half);
    vf[s] = *reinterpret_cast<const bf16x8_t*>(V + (kh + mkc) * D + 16 * s + 8 * half);
  }
  f32x16_t dk[DT], dv[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[t][e] = 0.f; dv[t][e] = 0.f; }

  int cur = 0;  // the staged tile being consumed; the other one is written meanwhile: one barrier per tile
  for (int g = 0; g < G_; ++g) {
    const size_t qh = ((size_t)b * Hq + (size_t)hk * G_ + g) * N;
    uint4 qa, qb, ga, gb;  // rows 2r and 2r+1 of a coming tile, chunk cc, of Q and dO
    float lreg = 0.f, dreg = 0.f;
    auto fetch = [&](int q0) {
      int r0 = q0 + 2 * pr_, r1 = r0 + 1;
      r0 = r0 < N ? r0 : N - 1;
      r1 = r1 < N ? r1 : N - 1;
      qa = *reinterpret_cast<const uint4*>(Q + (qh + r0) * D + 8 * pc_);
      qb = *reinterpret_cast<const uint4*>(Q + (qh + r1) * D + 8 * pc_);
      ga = *reinterpret_cast<const uint4*>(dO + (qh + r0) * D + 8 * pc_);
      gb = *reinterpret_cast<const uint4*>(dO + (qh + r1) * D + 8 * pc_);
      if (threadIdx.x < BQ) {
        int n = q0 + threadIdx.x;
        n = n < N ? n : N - 1;
        lreg = LSE[qh + n];
        dreg = delta[qh + n];
      }
    };
    auto commit = [&](int buf) {
      commit_pair<D, BQ>(qa, qb, pr_, pc_, qs[buf], qt_[buf]);
      commit_pair<D, BQ>(ga, gb, pr_, pc_, gs[buf], gt_[buf]);
      if (threadIdx.x < BQ) {
        lse_s[buf][threadIdx.x] = lreg * seed;
        dl_s[buf][threadIdx.x] = -dreg;
      }
    };
    if (k0 < qend) {
      fetch(k0);
      commit(cur);  // every wave is past the barrier that ended the last tile of the previous head
      __syncthreads();
      if (k0 + BQ < qend) fetch(k0 + BQ);
    }
    for (int q0 = k0; q0 < qend; q0 += BQ) {
      const bool skip = q0 + BQ - 1 < k0 + 32 * wave;  // every query of the tile precedes this wave's keys
      bf16_t (*qsc)[D + 8] = qs[cur];
      bf16_t (*gsc)[D + 8] = gs[cur];
      bf16_t (*qtc)[BQ + TPAD16] = qt_[cur];
      bf16_t (*gtc)[BQ + TPAD16] = gt_[cur];
      const float* lsc = lse_s[cur];
      const float* dlc = dl_s[cur];
      f32x16_t s, dp;
      bf16x8_t aq[KS], ag[KS];
      auto seed_acc = [&](int qt) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const float4 l4 = *reinterpret_cast<const float4*>(&lsc[32 * qt + 8 * gq + 4 * half]);
          const float4 d4 = *reinterpret_cast<const float4*>(&dlc[32 * qt + 8 * gq + 4 * half]);
          s[4 * gq + 0] = l4.x; s[4 * gq + 1] = l4.y; s[4 * gq + 2] = l4.z; s[4 * gq + 3] = l4.w;
          dp[4 * gq + 0] = d4.x; dp[4 * gq + 1] = d4.y; dp[4 * gq + 2] = d4.z; dp[4 * gq + 3] = d4.w;
        }
      };
      auto load_rows = [&](int qt, int part) {  // half of the row operands of a tile
#pragma unroll
        for (int x = part * (KS / 2); x < (part + 1) * (KS / 2); ++x) {
          aq[x] = *reinterpret_cast<const bf16x8_t*>(&qsc[32 * qt + col][16 * x + 8 * half]);
          ag[x] = *reinterpret_cast<const bf16x8_t*>(&gsc[32 * qt + col][16 * x + 8 * half]);
        }
      };
      auto tile = [&](int qt) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < KS; ++x) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[x], kf[x], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ag[x], vf[x], dp, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        bf16x8_t tq[2][DT], tg[2][DT];
#pragma unroll
        for (int G = 0; G < 2; ++G)
#pragma unroll
          for (int t = 0; t < DT; ++t) {
            tg[G][t] = ld_tr16(gtc, 32 * t + col, 32 * qt + 16 * G, half);
            tq[G][t] = ld_tr16(qtc, 32 * t + col, 32 * qt + 16 * G, half);
          }
        __builtin_amdgcn_sched_barrier(0);
        if (aligned && q0 + 32 * qt >= k0 + 32 * wave + 32) {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float p = fast_exp2(s[e] * scale_log2e);
            s[e] = p;
            dp[e] = p * dp[e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int n = q0 + 32 * qt + 8 * (e / 4) + 4 * half + e % 4;
            float p = fast_exp2(s[e] * scale_log2e);
            p = (n < mk || n >= myend) ? 0.f : p;
            s[e] = p;
            dp[e] = p * dp[e];
          }
        }
        bf16x8_t pf[2], df[2];
#pragma unroll
        for (int G = 0; G < 2; ++G) {
          pf[G] = pack8(s, 2 * G, 2 * G + 1);
          df[G] = pack8(dp, 2 * G, 2 * G + 1);
        }
        if (qt + 1 < NQT) seed_acc(qt + 1);
#pragma unroll
        for (int G = 0; G < 2; ++G) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int t = 0; t < DT; ++t) {
            dv[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tg[G][t], pf[G], dv[t], 0, 0, 0);
            dk[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tq[G][t], df[G], dk[t], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (qt + 1 < NQT) load_rows(qt + 1, G);  // the operands just consumed leave room for these
        }
      };
      if (!skip) {
        seed_acc(0);
        load_rows(0, 0);
        load_rows(0, 1);
        tile(0);
      }
      if (q0 + BQ < qend) {  // the next tile into the other buffer, the one after it into the registers
        commit(cur ^ 1);
        if (q0 + 2 * BQ < qend) fetch(q0 + 2 * BQ);
      }
      if (!skip) tile(1);
      __syncthreads();
      cur ^= 1;
    }
  }
  if (mk >= N) return;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      size_t o = (kh + mk) * D + 32 * t + 8 * g + 4 * half;
      *reinterpret_cast<float4*>(dK + o) =
          make_float4(scale * dk[t][4 * g + 0], scale * dk[t][4 * g + 1], scale * dk[t][4 * g + 2], scale * dk[t][4 * g + 3]);
      *reinterpret_cast<float4*>(dV + o) = make_float4(dv[t][4 * g + 0], dv[t][4 * g + 1], dv[t][4 * g + 2], dv[t][4 * g + 3]);
    }
}

// ------------------------------------------------------------------------------------------
// Summary gradients -> keys and values for bf16 inputs: one wave per (kv head, key block b', key
// cluster j); the keys of the segment are the MFMA columns, 32 query clusters at a time the rows.
//   W[i,m] = exp(L[i,m] - mu[i]),  T[i,m] = G_c[i] + G_k[i].k_m + G_v[i].v_m
//   dv_m += sum_i W G_v[i],  dk_m += sum_i W G_k[i] + (W T) qbar_i
// G and qbar are rounded to bf16 for the matrix cores (gradients only); qbar comes from a bf16 copy qcb[head][i][d] (scale
// folded in, i padded to a multiple of 32 with zeros).  A tile of gradient rows and centroids goes to LDS row-major, whole
// rows per load instruction, and serves the row operands of T and, through transposed reads, the contractions over i.
// Bound by the gradient rows, D x 2 bytes each at a stride of Ck rows.  Row operands read straight from memory touched 32 rows
// with every instruction, centroids and rows were transposed with 2-byte stores: 3.10 ms at 16 heads of 64k with 256 x 1024
// clusters (9.2 GB) against 2.29, 2.77 against 1.86 at 32 heads of 32k, D = 128, 128 x 512 clusters (since the rows are added to the block
// diagonal's here, which saves passes of their own, 2.36 and 1.95).  Three waves per SIMD at
// D = 64, and a second tile in flight, spill (4.6 and 3.2 ms).
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_qc_rows(const float* __restrict__ qc, bf16_t* __restrict__ qcb, int D, int Cq, int CqP,
                                                 float scale) {
  const int h = blockIdx.y;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= D * CqP) return;
  qcb[(size_t)h * D * CqP + t] = f32_to_bf16_bits(t / D < Cq ? scale * qc[(size_t)h * Cq * D + t] : 0.f);
}

template <int D, bool HERE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1, D == 64 ? 2 : 1))) k_cells_to_keys_mx(const bf16_t* __restrict__ Ks, const bf16_t* __restrict__ Vs,
                                                          const bf16_t* __restrict__ qcb, const float* __restrict__ L,
                                                          const float* __restrict__ s_mu, const float* __restrict__ G_c,
                                                          const bf16_t* __restrict__ G_k, const bf16_t* __restrict__ G_v,
                                                          const int32_t* __restrict__ off_k, const int32_t* __restrict__ perm_k, float* __restrict__ dKs,
                                                          float* __restrict__ dVs, float* __restrict__ dK, float* __restrict__ dV, int h0, int N, int nb, int Cq, int CqP,
                                                          int Ck, int Hq, int Hkv, int frozen) {
  constexpr int KS = D / 16, DT = D / 32, CPR = D / 8, NIT = 32 * CPR / 64;
  __shared__ __attribute__((aligned(16))) bf16_t gks[32 * D];
  __shared__ __attribute__((aligned(16))) bf16_t gvs[32 * D];
  __shared__ __attribute__((aligned(16))) bf16_t qs[32 * D];
  __shared__ __attribute__((aligned(16))) float mus[32];
  __shared__ __attribute__((aligned(16))) float gcs[32];
  const int G_ = Hq / Hkv;
  const int hkl = blockIdx.z;
  const int hq0 = h0 + hkl * G_;
  const int hk = (hq0 / Hq) * Hkv + (hq0 % Hq) / G_;
  // x % 8 is the XCD a workgroup lands on (the grid's x extent is a multiple of 8): each XCD takes a run of
  // consecutive key clusters, whose per-cell scalars share 32-byte sectors, so a sector is fetched by one L2
  const int run = gridDim.x / 8;
  const int bp = blockIdx.y, j = (blockIdx.x % 8) * run + blockIdx.x / 8, NBm = nb - 1;
  if (j >= Ck) return;
  const int lane = threadIdx.x, col = lane % 32, half = lane / 32;
  const int32_t* ok = off_k + (size_t)hk * ((size_t)nb * Ck + 1);
  const int klo = ok[bp * Ck + j], khi = ok[bp * Ck + j + 1];
  for (int m0 = klo; m0 < khi; m0 += 32) {
    const int pm = m0 + col;
    const bool mvalid = pm < khi;
    const int pmc = mvalid ? pm : m0;
    bf16x8_t kb[KS], vb[KS];  // the lane's key and value
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      kb[x] = *reinterpret_cast<const bf16x8_t*>(Ks + ((size_t)hk * N + pmc) * D + 16 * x + 8 * half);
      vb[x] = *reinterpret_cast<const bf16x8_t*>(Vs + ((size_t)hk * N + pmc) * D + 16 * x + 8 * half);
    }
    f32x16_t dk[DT], dv[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) { dk[t][e] = 0.f; dv[t][e] = 0.f; }
    // Tiles of 32 query clusters of one head of the group: the gradient rows and the centroids, whole rows per load
    // instruction (a lane that reads its own operand straight from memory touches 32 rows with every instruction), the rows'
    // scalars, the logits of the lane's key against the 16 query clusters of its accumulator rows.
    const int nti = (Cq + 31) / 32, ntile = G_ * nti;
    for (int tile = 0; tile < ntile; ++tile) {
      const int hl = hkl * G_ + tile / nti, i0 = tile % nti * 32;
      // uniform bases, the lanes' offsets take 32 bits
      const size_t cell0 = (((size_t)hl * NBm + bp) * Cq + i0) * Ck + j;
      const bf16_t *gkp = G_k + cell0 * D, *gvp = G_v + cell0 * D, *qp = qcb + ((size_t)hl * CqP + i0) * D;
      const float *mup = s_mu + cell0, *gcp = G_c + cell0, *Lp = L + ((size_t)hl * Cq + i0) * N;
      bf16x8_t gk[NIT], gv[NIT], gq[NIT];
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int row = it * (64 / CPR) + lane / CPR, cc = lane % CPR;
        const uint32_t o = (uint32_t)(min(row, Cq - 1 - i0) * Ck * D + cc * 8);
        gk[it] = *reinterpret_cast<const bf16x8_t*>(gkp + o);
        gv[it] = *reinterpret_cast<const bf16x8_t*>(gvp + o);
        gq[it] = *reinterpret_cast<const bf16x8_t*>(qp + (uint32_t)(row * D + cc * 8));
      }
      const uint32_t oc = (uint32_t)(min(col, Cq - 1 - i0) * Ck);
      const float mu_l = mup[oc], gc_l = gcp[oc];
      float lg[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) lg[e] = Lp[(uint32_t)(min(8 * (e / 4) + 4 * half + (e % 4), Cq - 1 - i0) * N + pmc)];
      wave_lds_fence();  // the previous tile's operand reads are done
      if (half == 0) { mus[col] = mu_l; gcs[col] = gc_l; }
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int at = tile_at<D>(it * (64 / CPR) + lane / CPR, lane % CPR);
        *reinterpret_cast<bf16x8_t*>(gks + at) = gk[it];
        *reinterpret_cast<bf16x8_t*>(gvs + at) = gv[it];
        *reinterpret_cast<bf16x8_t*>(qs + at) = gq[it];
      }
      wave_lds_fence();
      f32x16_t tacc, wv;
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const float4 m4 = *reinterpret_cast<const float4*>(&mus[8 * gq + 4 * half]);
        const float4 c4 = *reinterpret_cast<const float4*>(&gcs[8 * gq + 4 * half]);
        const float mv[4] = {m4.x, m4.y, m4.z, m4.w}, cv[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = 4 * gq + u;
          const bool iv = i0 + 8 * gq + 4 * half + u < Cq;
          tacc[e] = cv[u];
          wv[e] = (iv && mvalid) ? __expf(lg[e] - mv[u]) : 0.f;
        }
      }
      // frozen aggregation weights: nothing flows through W (the T term and its contraction with qbar drop out)
      if (!frozen) {
#pragma unroll
        for (int x = 0; x < KS; ++x) {
          tacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(gks, col, 2 * x + half), kb[x], tacc, 0, 0, 0);
          tacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_row<D>(gvs, col, 2 * x + half), vb[x], tacc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) tacc[e] = (wv[e] > 0.f && !frozen) ? wv[e] * tacc[e] : 0.f;
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        bf16x8_t wf = pack8(wv, 2 * G, 2 * G + 1);
        bf16x8_t tf = pack8(tacc, 2 * G, 2 * G + 1);
#pragma unroll
        for (int t = 0; t < DT; ++t) {
          const bf16x8_t ak = tile_cols<D>(gks, 16 * G, t, lane);
          const bf16x8_t av = tile_cols<D>(gvs, 16 * G, t, lane);
          dv[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, wf, dv[t], 0, 0, 0);
          dk[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak, wf, dk[t], 0, 0, 0);
          if (!frozen) dk[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_cols<D>(qs, 16 * G, t, lane), tf, dk[t], 0, 0, 0);
        }
      }
    }
    if (mvalid) {
      // HERE: with the retrieval's rows (bucketed) to the block diagonal's (in the sequence's order); else to the former (the two are bodies
      // of their own: one for both made the former 5 to 20 % slower)
      const size_t from = ((size_t)hk * N + pm) * D;
      if constexpr (HERE) {
        const size_t to = ((size_t)hk * N + perm_k[(size_t)hk * N + pm]) * D;
        const float *fk = dKs, *fv = dVs;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int gg = 0; gg < 4; ++gg) {
            const int d = 32 * t + 8 * gg + 4 * half;
            const float4 a = *reinterpret_cast<const float4*>(fk + from + d), c = *reinterpret_cast<const float4*>(fv + from + d);
            float4 k = *reinterpret_cast<float4*>(dK + to + d), v = *reinterpret_cast<float4*>(dV + to + d);
            k.x += a.x + dk[t][4 * gg]; k.y += a.y + dk[t][4 * gg + 1]; k.z += a.z + dk[t][4 * gg + 2]; k.w += a.w + dk[t][4 * gg + 3];
            v.x += c.x + dv[t][4 * gg]; v.y += c.y + dv[t][4 * gg + 1]; v.z += c.z + dv[t][4 * gg + 2]; v.w += c.w + dv[t][4 * gg + 3];
            *reinterpret_cast<float4*>(dK + to + d) = k;
            *reinterpret_cast<float4*>(dV + to + d) = v;
          }
      } else {
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int gg = 0; gg < 4; ++gg) {
            const int d = 32 * t + 8 * gg + 4 * half;
            float4 a = *reinterpret_cast<float4*>(dKs + from + d), c = *reinterpret_cast<float4*>(dVs + from + d);
            a.x += dk[t][4 * gg]; a.y += dk[t][4 * gg + 1]; a.z += dk[t][4 * gg + 2]; a.w += dk[t][4 * gg + 3];
            c.x += dv[t][4 * gg]; c.y += dv[t][4 * gg + 1]; c.z += dv[t][4 * gg + 2]; c.w += dv[t][4 * gg + 3];
            *reinterpret_cast<float4*>(dKs + from + d) = a;
            *reinterpret_cast<float4*>(dVs + from + d) = c;
          }
      }
    }
  }
}

}  // namespace

int muse_launch_cells_to_keys_mx(const MuseDims& d, const void* Ks, const void* Vs, const float* qc, void* qcb,
                                 const float* L, const float* s_mu, const float* G_c, const void* G_k, const void* G_v,
                                 const int32_t* off_k, const int32_t* perm_k, float* dKs, float* dVs, float* dK, float* dV, int h0, int hn,
                                 hipStream_t st) {
  const int CqP = (d.Cq + 31) / 32 * 32;
  // qcb holds the scaled centroids of the chunk's heads [h0, h0 + hn)
  { MuseProf prof_("k_qc_rows", st); hipLaunchKernelGGL(k_qc_rows, dim3((d.D * CqP + 255) / 256, hn), dim3(256), 0, st, qc + (size_t)h0 * d.Cq * d.D, (bf16_t*)qcb, d.D, d.Cq, CqP, d.scale); }
  dim3 g((d.Ck + 7) / 8 * 8, d.nb - 1, hn / (d.Hq / d.Hkv));
  auto go = [&](auto* kernel) {
    MuseProf prof_("k_cells_to_keys_mx", st);
    hipLaunchKernelGGL(kernel, g, dim3(64), 0, st, (const bf16_t*)Ks, (const bf16_t*)Vs, (const bf16_t*)qcb, L, s_mu, G_c, (const bf16_t*)G_k, (const bf16_t*)G_v,
                       off_k, perm_k, dKs, dVs, dK, dV, h0, d.N, d.nb, d.Cq, CqP, d.Ck, d.Hq, d.Hkv, d.frozen_weights ? 1 : 0);
  };
  if (d.D == 64) dK ? go(k_cells_to_keys_mx<64, true>) : go(k_cells_to_keys_mx<64, false>);
  else dK ? go(k_cells_to_keys_mx<128, true>) : go(k_cells_to_keys_mx<128, false>);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

// attn_bwd.hip: the kernels of 256 rows per workgroup, and where they are the better ones
bool muse_attn_dq_wide(const MuseDims& d, int Bs);
bool muse_attn_dkv_wide(const MuseDims& d, int Bs);
bool muse_attn_rows_to_lds(const void* Q, const void* K, const void* V, const void* dO);
int muse_launch_attn_dq_wide(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                             const float* delta, void* dQ, hipStream_t st);
int muse_launch_attn_dkv_wide(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                              const float* delta, void* dK, void* dV, hipStream_t st);

int muse_launch_attn_bwd_mfma(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V,
                              const void* dO, const float* LSE, const float* delta, float* dQacc,
                              float* dKacc, float* dVacc, hipStream_t st) {
  const dim3 gq = flash_grid(d.N, Bs, d.Hq, d.B), gk = flash_grid(d.N, Bs, d.Hkv, d.B);
  float sl = d.scale * 1.4426950408889634f;
  const bf16_t *q = (const bf16_t*)Q, *k = (const bf16_t*)K, *v = (const bf16_t*)V, *g = (const bf16_t*)dO;
  const bool to_lds = muse_attn_rows_to_lds(Q, K, V, dO);
  if (to_lds && muse_attn_dq_wide(d, Bs)) {
    if (int rc = muse_launch_attn_dq_wide(d, Bs, Q, K, V, dO, LSE, delta, dQacc, st)) return rc;
  } else {
    MuseProf prof_("k_flash_bwd_dq", st);
    if (d.D == 64) hipLaunchKernelGGL(k_flash_bwd_dq<64>, gq, dim3(256), 0, st, q, k, v, g, LSE, delta, dQacc, d.N, Bs, d.Hq, d.Hkv, d.B, d.scale, sl);
    else hipLaunchKernelGGL(k_flash_bwd_dq<128>, gq, dim3(256), 0, st, q, k, v, g, LSE, delta, dQacc, d.N, Bs, d.Hq, d.Hkv, d.B, d.scale, sl);
  }
  if (to_lds && muse_attn_dkv_wide(d, Bs)) return muse_launch_attn_dkv_wide(d, Bs, Q, K, V, dO, LSE, delta, dKacc, dVacc, st);
  {
    MuseProf prof_("k_flash_bwd_dkv", st);
    if (d.D == 64) hipLaunchKernelGGL(k_flash_bwd_dkv_p<64>, gk, dim3(256), 0, st, q, k, v, g, LSE, delta, dKacc, dVacc, d.N, Bs, d.Hq, d.Hkv, d.B, d.scale, sl);
    else hipLaunchKernelGGL(k_flash_bwd_dkv128, gk, dim3(512), 0, st, q, k, v, g, LSE, delta, dKacc, dVacc, d.N, Bs, d.Hq, d.Hkv, d.B, d.scale, sl);
  }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
