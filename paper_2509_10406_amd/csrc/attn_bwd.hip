// bf16 causal attention, backward, for blocks long enough to fill tiles of 256 rows (keys restricted to the query's own spatial
// block of size Bs; Bs = N gives exact attention).  attn_mfma.hip has the kernels for the rest and the layouts both share.
//
// What bounds these kernels: the matrix instructions (32 cycles each), the vector work on a score (exponential 8.5 cycles, the rest
// 4.6 each, measured), and the LDS reads of the operands, each of which is about as long as the others if a wave has 32 rows of
// its own.  So a wave has 64 rows (units a and b of 32), which halves the LDS reads per matrix instruction, in one wave per SIMD with
// all 512 registers, and does the overlapping itself.  A "part" of the loop holds three independent things:
//   the scores S and dP of the unit after next, the vector work of the next one, the gradients of the last one:
//   A(i): S, dP of (b, i)      P, dS of (a, i)      gradients of (b, i - 1)
//   B(i): S, dP of (a, i + 1)  P, dS of (b, i)      gradients of (a, i)
// for the tiles i of 32 staged rows: behind every matrix instruction stand one score's vector work and the LDS reads of operands
// that are taken most of a part later (fixed with scheduling barriers; the compiler keeps the order).  Staged rows go from memory
// to LDS without registers, a step (two tiles) or two ahead, one request behind every third or fourth matrix instruction: in a
// row they hold the wave until memory has taken them.  One barrier per step.
//   The accumulated gradients live in accumulation registers (the asm below), scores and operands in vector registers (the
// compiler is told to let the other matrix instructions write there: left to itself it puts all results into accumulation
// registers and moves every score out again, 200 moves in 64 matrix instructions).
// Measured, us, 128 rows per workgroup and 32 per wave -> this: dK/dV 640 -> 465 at 8 heads of 16k, 200 -> 135 at 32 heads of 4k,
// 82 -> 52 at 128 heads of 1k; dQ 440 -> 370, 150 -> 104, 51 -> 41; dQ at D = 128 791 -> 641 at 32 heads of 8k, 241 -> 175 of 4k; dK/dV
// at D = 128 (before: 32 keys and one matrix phase per wave) 1210 -> 1012, 339 -> 287, 149 -> 120 at 128 heads of 1k.  Cycles
// per step (of 2048 in matrix instructions) 3050 for dK/dV, of 1536 2420 for dQ (D = 128: of 3072 4380).  The clock is below its 2.4
// GHz meanwhile: 1.7 to 1.8 in the first passes after a pause (GRBM_GUI_ACTIVE over the time), 2.0 where calls follow one another (2.2
// for dK/dV at D = 128): the times above are of calls in a row, a single pass takes 10 to 35 % longer.
#include <type_traits>

#include "ff_common.h"
#include "flash_tile.h"
#include "lds_tile.h"

namespace {

constexpr int TR = 256;  // rows of a workgroup's tile: keys (dK / dV) or queries (dQ)
constexpr int BN = 64;   // rows staged per step
constexpr int TR128 = 128;  // keys of a workgroup's tile of dK / dV at D = 128

using lds_frag = __attribute__((address_space(3))) const bf16x8_t*;
using lds_f4 = __attribute__((address_space(3))) const f32x4_t*;
using lds_tr = __attribute__((address_space(3))) s16x4_t*;

__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
__device__ __forceinline__ void group_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// acc += a b with acc in accumulation registers.  The compiler does not know this for a matrix instruction: the operands are written
// at least a matrix instruction earlier, and acc_settle stands behind the last one of a sequence, in front of any reader.
__device__ __forceinline__ void mfma_acc(f32x16_t& acc, bf16x8_t a, bf16x8_t b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// dK and dV at D = 64: a wave owns 64 keys, tiles of queries are staged, from the keys' own to the block's last (query heads of the
// group one after the other).  The accumulators of S and dP start at -LSE / scale and -delta (from LDS), so P = exp2(c S), dS = P dP.
// Queries past the block's end start at -inf: P is zero there.
// Three buffers: in step i, tile i + 1 has to be complete at the barrier in the middle (A(i + 1) reads its rows in the second half),
// behind that barrier nobody reads tile i - 1 any more and i + 2 goes there.
template <typename OT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) k_flash_bwd_dkv_wide(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
    const float* __restrict__ LSE, const float* __restrict__ delta, OT* __restrict__ dK, OT* __restrict__ dV, int N,
    int Bs, int Hq, int Hkv, int nbatch, int chunk, float scale, float scale_log2e) {
  constexpr int D = 64, KS = D / 16, DT = D / 32, NB = 3, kTile = BN * D, kB = kTile * 2, LAG = 8, CPR = D / 8, NCH = BN * CPR / 256;
  __shared__ __attribute__((aligned(256))) bf16_t tiles[2][NB][kTile];  // Q, dO
  __shared__ __attribute__((aligned(256))) float seeds[NB][4][BN];      // -LSE / scale, -delta, and the same again (waves 2 and 3)
  const int tpg = (Bs + TR - 1) / TR;
  const FlashTile ft = flash_tile_of(tpg, N / Bs, Hkv, nbatch, tpg, chunk);
  if (!ft.ok) return;
  const int hk = ft.h, b = ft.b, G_ = Hq / Hkv;
  const size_t kh = ((size_t)b * Hkv + hk) * N, qh0 = ((size_t)b * Hq + (size_t)hk * G_) * N;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, col = lane % 32, half = lane / 32;
  const int k0 = ft.blk * Bs + ft.t * TR, bend = (ft.blk + 1) * Bs;
  const int ka = k0 + 64 * wave;  // the wave's keys: ka .. ka + 63
  const int ns = (bend - k0 + BN - 1) / BN;

  bf16x8_t kf[2][KS], vf[2][KS];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      const size_t o = (kh + min(ka + 32 * u + col, bend - 1)) * D + 16 * x + 8 * half;
      kf[u][x] = *reinterpret_cast<const bf16x8_t*>(K + o);
      vf[u][x] = *reinterpret_cast<const bf16x8_t*>(V + o);
    }
  f32x16_t dk[2][DT], dv[2][DT];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int t = 0; t < DT; ++t) dk[u][t] = dv[u][t] = zero16();

  // staging
  const float seed = -1.4426950408889634f / scale_log2e;
  const float smul = wave % 2 == 0 ? seed : -1.f, sdead = wave % 2 == 0 ? seed * __builtin_huge_valf() : 0.f;
  float sv = 0.f;
  const bf16_t *qp = Q + qh0 * D, *gp = dO + qh0 * D;
  const float* sp = (wave % 2 == 0 ? LSE : delta) + qh0;
  // LDS takes the 16-byte chunks of a tile in order of the thread, so the order of the chunks in a row is in the source
  const int srow = tid / CPR, schunk = (tile_at<D>(srow, tid % CPR) - srow * D) / 8;
  const uint32_t lds0 = lds_addr(&tiles[0][0][0]) + wave * 1024;
  int fq = k0, cq = k0, fh = 0;
  auto bring_op = [&](int k, int buf) {  // the k-th of the 2 NCH requests of a tile
    const int u = k / 2;
    const uint32_t off = (uint32_t)(min(fq + BN / NCH * u + srow, bend - 1) * D + 8 * schunk) * 2;
    rows_to_lds(lds0 + (k % 2 * NB + buf) * kB + u * 4096, off, k % 2 ? gp : qp);
  };
  auto bring_end = [&]() {
    sv = sp[min(fq + lane, bend - 1)];
    fq += BN;
    const bool over = fq >= bend;
    const int step = over && ++fh < G_ ? N : 0;  // past the last head: its tiles again, which nobody reads
    fq = over ? k0 : fq;
    qp += (size_t)step * D;
    gp += (size_t)step * D;
    sp += step;
  };
  auto bring = [&](int buf) {
#pragma unroll
    for (int k = 0; k < 2 * NCH; ++k) bring_op(k, buf);
    bring_end();
  };
  auto arrived = [&](int buf) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    seeds[buf][wave][lane] = cq + lane < bend ? sv * smul : sdead;
    cq = cq + BN < bend ? cq + BN : k0;
  };

  // operand addresses of this lane in the first buffer
  const uint32_t rat = lds_addr(&tiles[0][0][tile_at<D>(col, half)]);
  const uint32_t tat = lds_addr(&tiles[0][0][tile_at<D>(4 * half + (lane % 16) / 4, 2 * ((lane / 16) % 2) + (lane % 4) / 2) + 4 * (lane % 2)]);
  const uint32_t sat = lds_addr(&seeds[0][0][4 * half]);
  uint32_t ra_[KS], ta_[4], sa_ = sat;  // where the next operands are read
  auto rows_from = [&](int buf) {
#pragma unroll
    for (int x = 0; x < KS; ++x) ra_[x] = (rat ^ (uint32_t)(x << 5)) + buf * kB;
    sa_ = sat + buf * (4 * BN * 4);
  };
  auto cols_from = [&](int buf) {
#pragma unroll
    for (int x = 0; x < 4; ++x) ta_[x] = (tat ^ (uint32_t)(x << 5)) + buf * kB;
  };

  bf16x8_t rows[2][KS];     // of Q, dO
  bf16x8_t cols[2][2][DT];  // of Q, dO: [16-row group][32 columns]
  f32x16_t sd[2];           // seeds of S, dP
  f32x16_t s[2], dp[2];
  uint32_t pf[2][2][4], df[2][2][4];

  // Operand j of a part (j even: rows, odd: columns), from rows 32 qr / 32 qc of the tile
  auto load_op = [&](int j, int qr, int qc) {
    if (j % 2 == 0) {
      const int x = j / 4, w = (j / 2) % 2;
      rows[w][x] = *(lds_frag)(uintptr_t)(ra_[x] + (w * NB * kB + qr * 32 * D * 2));
    } else {
      const int k = j / 2, G = k / 4, t = (k % 4) / 2, w = 1 - k % 2;
      const uint32_t o = w * NB * kB + (qc * 32 + G * 16) * D * 2;
      cols[w][G][t] = tr_join(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(ta_[2 * t] + o)),
                              __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(ta_[2 * t + 1] + (o + 8 * D * 2))));
    }
  };
  auto load_seed = [&](int w, int g, int qr) {
    const f32x4_t v = *(lds_f4)(uintptr_t)(sa_ + (w * BN + qr * 32 + 8 * g) * 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) sd[w][4 * g + u] = v[u];
  };
  auto mfma_op = [&](int j, int us, int ug, bool sdp, bool grad) {
    if (j % 2 == 0) {
      if (!sdp) return;
      const int x = j / 4;
      if ((j / 2) % 2 == 0)
        s[us] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows[0][x], kf[us][x], x == 0 ? sd[0] : s[us], 0, 0, 0);
      else
        dp[us] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows[1][x], vf[us][x], x == 0 ? sd[1] : dp[us], 0, 0, 0);
    } else {
      if (!grad) return;
      const int k = j / 2, G = k / 4, t = (k % 4) / 2;
      if (k % 2 == 0) {
        const uint4 w = make_uint4(pf[ug][G][0], pf[ug][G][1], pf[ug][G][2], pf[ug][G][3]);
        mfma_acc(dv[ug][t], cols[1][G][t], __builtin_bit_cast(bf16x8_t, w));
      } else {
        const uint4 w = make_uint4(df[ug][G][0], df[ug][G][1], df[ug][G][2], df[ug][G][3]);
        mfma_acc(dk[ug][t], cols[0][G][t], __builtin_bit_cast(bf16x8_t, w));
      }
    }
  };
  auto loads = [&](int c, int qr, int qc) {
    if (c == 2 || c == 4 || c == 6 || c == 8) load_seed(0, c / 2 - 1, qr);
    if (c == 5 || c == 6) load_seed(1, c - 5, qr);
    if (c == 8 || c == 9) load_seed(1, c - 6, qr);
    if (c < 8 && c % 2 == 1) load_op(c / 2, qr, qc);
    if (c >= LAG + 4 && c < LAG + 16) load_op(c - LAG, qr, qc);
  };
  float tm = 0.f;
  auto valu_op = [&](int e, int u, bool mask, int nm) {
    if (e == 0) tm = s[u][0] * scale_log2e;
    float p = fast_exp2(tm);
    if (e < 15) tm = s[u][e + 1] * scale_log2e;
    if (e > 0) dp[u][e - 1] *= s[u][e - 1];
    if (mask) p = nm + 8 * (e / 4) + e % 4 >= 0 ? p : 0.f;
    s[u][e] = p;
    if (e >= 2 && e % 2 == 0) {
      const int i = e / 2 - 1;
      pf[u][i / 4][i % 4] = pack_bf16x2(s[u][e - 2], s[u][e - 1]);
      df[u][i / 4][i % 4] = pack_bf16x2(dp[u][e - 2], dp[u][e - 1]);
    }
    if (e == 15) {
      dp[u][15] *= p;
      pf[u][1][3] = pack_bf16x2(s[u][14], p);
      df[u][1][3] = pack_bf16x2(dp[u][14], dp[u][15]);
    }
  };
  // 16 matrix instructions, one element of the unit `uv` and the reads of the operands that the next part takes behind each
#define DKV_PART(FIRST_HALF, US, UV, SDP, VAL, MASK, GRAD, QR, QC, BRING)                \
  {                                                                                      \
    _Pragma("unroll") for (int j = 0; j < 16; ++j) {                                     \
      mfma_op(j, US, 1 - UV, SDP, GRAD);                                                 \
      __builtin_amdgcn_sched_barrier(0);                                                 \
      if (VAL) valu_op(j, UV, MASK, nm);                                                 \
      loads(FIRST_HALF ? j : 16 + j, QR, QC);                                            \
      if ((BRING) && j % 4 == 1) bring_op(j / 4, nn);                                    \
      __builtin_amdgcn_sched_barrier(0);                                                 \
    }                                                                                    \
  }
  const int nm = 4 * half - col;
  bring(0);
  arrived(0);
  group_barrier();
  bring(1);
  int cur = 0;
  for (int g = 0; g < G_; ++g) {
    int i = 0;
    auto idle = [&]() {
      const int nxt = cur == NB - 1 ? 0 : cur + 1;
      arrived(nxt);
      group_barrier();
      bring(nxt == NB - 1 ? 0 : nxt + 1);
      cur = nxt;
    };
    for (; i < min(wave, ns); ++i) idle();
    if (i < ns) {
      int nxt = cur == NB - 1 ? 0 : cur + 1, nn;
      rows_from(cur);
      cols_from(cur);
#pragma unroll
      for (int q = 0; q < 4; ++q) { load_seed(0, q, 0); load_seed(1, q, 0); }
#pragma unroll
      for (int j = 0; j < 16; j += 2) load_op(j, 0, 0);
#pragma unroll
      for (int j = 0; j < 16; j += 2) mfma_op(j, 0, 1, true, false);
      __builtin_amdgcn_sched_barrier(0);
      DKV_PART(true, 1, 0, false, true, true, false, 1, 0, false)
      DKV_PART(false, 0, 1, true, false, false, true, 1, 0, false)
      arrived(nxt);
      group_barrier();
      nn = nxt == NB - 1 ? 0 : nxt + 1;
      rows_from(nxt);
      DKV_PART(true, 1, 0, true, true, false, false, 0, 1, true)
      bring_end();
      DKV_PART(false, 0, 1, true, true, true, true, 0, 1, false)
      cur = nxt;
      for (++i; i < ns; ++i) {
        nxt = cur == NB - 1 ? 0 : cur + 1;
        cols_from(cur);
        DKV_PART(true, 1, 0, true, true, false, true, 1, 0, false)
        DKV_PART(false, 0, 1, true, true, false, true, 1, 0, false)
        arrived(nxt);
        group_barrier();
        nn = nxt == NB - 1 ? 0 : nxt + 1;
        rows_from(nxt);
        DKV_PART(true, 1, 0, true, true, false, true, 0, 1, true)
        bring_end();
        DKV_PART(false, 0, 1, true, true, false, true, 0, 1, false)
        cur = nxt;
      }
#pragma unroll
      for (int j = 1; j < 16; j += 2) mfma_op(j, 0, 1, false, true);
      acc_settle();
    }
  }
#undef DKV_PART
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing is on its way into LDS that others may own soon
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int mk = ka + 32 * u + col;
    if (mk >= bend) continue;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const size_t o = (kh + mk) * D + 32 * t + 8 * g + 4 * half;
        const f32x16_t &a = dk[u][t], &c = dv[u][t];
        const float k4[4] = {scale * a[4 * g], scale * a[4 * g + 1], scale * a[4 * g + 2], scale * a[4 * g + 3]};
        const float v4[4] = {c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
        st4(dK, o, k4);
        st4(dV, o, v4);
      }
  }
}

// dK and dV at D = 128.  Accumulators of dK and dV and both operands of 64 keys are too many registers for one wave, so two waves
// share 64 keys: one computes P = exp2(c (Q K^T - LSE)) and dV += P^T dO, the other, a step of 32 queries behind, dP = dO V^T,
// dS = P dP and dK += dS^T Q; P passes between them through LDS in fp32, one barrier per step.  Within a wave the same
// three things overlap as above, a step being the parts A and B of one tile.
// At step T: P and dV of tile T, dP and dK of tile T - 1; rows of tile T + 1 are read, T + 2 is on its way, T + 3 is asked for
// (behind the barrier that ends the reads of T - 2): five buffers.  Seeds come in chunks of 256 rows, four buffers: a chunk is
// written at the first step of the chunk two before it, when nobody reads the one before that any more.
template <typename OT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) k_flash_bwd_dkv128_wide(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
    const float* __restrict__ LSE, const float* __restrict__ delta, OT* __restrict__ dK, OT* __restrict__ dV, int N,
    int Bs, int Hq, int Hkv, int nbatch, int chunk, float scale, float scale_log2e) {
  constexpr int D = 128, KS = D / 16, DT = D / 32, BQ = 32, NB = 5, NS = 4, SC = 256, kTile = BQ * D, kB = kTile * 2, NM = 16, LAG = 6;
  __shared__ __attribute__((aligned(256))) bf16_t tiles[2][NB][kTile];       // Q, dO
  __shared__ __attribute__((aligned(256))) float4 px[2][2][2][4][64];        // P: [step parity][wave pair][unit][4 rows][lane]
  __shared__ __attribute__((aligned(256))) float seeds[NS][2][SC];           // -LSE / scale, -delta
  const int tpg = (Bs + TR128 - 1) / TR128;
  const FlashTile ft = flash_tile_of(tpg, N / Bs, Hkv, nbatch, tpg, chunk);
  if (!ft.ok) return;
  const int hk = ft.h, b = ft.b, G_ = Hq / Hkv;
  const size_t kh = ((size_t)b * Hkv + hk) * N, qh0 = ((size_t)b * Hq + (size_t)hk * G_) * N;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, col = lane % 32, half = lane / 32;
  const int pair = wave % 2, role = wave / 2;
  const int k0 = ft.blk * Bs + ft.t * TR128, bend = (ft.blk + 1) * Bs;
  const int ka = k0 + 64 * pair;  // the pair's keys: ka .. ka + 63
  const int ns = (bend - k0 + BQ - 1) / BQ, NT = G_ * ns;

  bf16x8_t kv[2][KS];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int x = 0; x < KS; ++x)
      kv[u][x] = *reinterpret_cast<const bf16x8_t*>((role ? V : K) + (kh + min(ka + 32 * u + col, bend - 1)) * D + 16 * x + 8 * half);
  f32x16_t acc[2][DT];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int t = 0; t < DT; ++t) acc[u][t] = zero16();

  // staged rows
  const bf16_t *qp = Q + qh0 * D, *gp = dO + qh0 * D;
  const int srow = tid / 16, schunk = (tile_at<D>(srow, tid % 16) - srow * D) / 8;
  const uint32_t lds0 = lds_addr(&tiles[0][0][0]) + wave * 1024;
  int fq = k0, fh = 0, fb = 0;
  auto bring_op = [&](int k) {  // the k-th of the four requests of a tile
    const uint32_t off = (uint32_t)(min(fq + 16 * (k / 2) + srow, bend - 1) * D + 8 * schunk) * 2;
    rows_to_lds(lds0 + (k % 2 * NB + fb) * kB + k / 2 * 4096, off, k % 2 ? gp : qp);
  };
  auto bring_end = [&]() {
    fb = fb == NB - 1 ? 0 : fb + 1;
    fq += BQ;
    const bool over = fq >= bend;
    const int step = over && ++fh < G_ ? N : 0;  // past the last head: its tiles again, which nobody reads
    fq = over ? k0 : fq;
    qp += (size_t)step * D;
    gp += (size_t)step * D;
  };
  auto bring = [&]() {
#pragma unroll
    for (int k = 0; k < 4; ++k) bring_op(k);
    bring_end();
  };
  // seeds of a chunk, a row per thread
  const float seed = -1.4426950408889634f / scale_log2e, dead = seed * __builtin_huge_valf();
  const float *lp = LSE + qh0, *ep = delta + qh0;
  int sq = k0, sh = 0, sb = 0;
  float lv, ev;
  auto seeds_fetch = [&]() {
    lv = lp[min(sq + tid, bend - 1)];
    ev = ep[min(sq + tid, bend - 1)];
  };
  auto seeds_commit = [&]() {
    seeds[sb][0][tid] = sq + tid < bend ? lv * seed : dead;
    seeds[sb][1][tid] = -ev;
    sb = (sb + 1) % NS;
    sq += SC;
    const bool over = sq >= bend;
    const int step = over && ++sh < G_ ? N : 0;
    sq = over ? k0 : sq;
    lp += step;
    ep += step;
  };

  const uint32_t rat = lds_addr(&tiles[0][0][tile_at<D>(col, half)]);
  const uint32_t tat = lds_addr(&tiles[0][0][tile_at<D>(4 * half + (lane % 16) / 4, 2 * ((lane / 16) % 2) + (lane % 4) / 2) + 4 * (lane % 2)]);
  const uint32_t sat = lds_addr(&seeds[0][0][4 * half]), pat = lds_addr(&px[0][pair][0][0][lane]);

  auto work = [&](auto role_c) {
    constexpr int R = decltype(role_c)::value;  // 0: P and dV, 1: dP and dK, a step behind
    uint32_t ra_[KS], ta_[2 * DT], sa_, pa_ = pat;
    bf16x8_t rows[KS], cols[2][DT];
    f32x16_t sd, s[2];
    float pv[2][16];
    uint32_t pf[2][2][4];
    auto load_op = [&](int j) {
      if (j % 2 == 0) {
        rows[j / 2] = *(lds_frag)(uintptr_t)(ra_[j / 2] + R * NB * kB);
      } else {
        const int G = j / 2 / DT, t = j / 2 % DT;
        const uint32_t o = (1 - R) * NB * kB + G * 16 * D * 2;
        cols[G][t] = tr_join(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(ta_[2 * t] + o)),
                             __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(ta_[2 * t + 1] + (o + 8 * D * 2))));
      }
    };
    auto load_seed = [&](int g) {
      const f32x4_t v = *(lds_f4)(uintptr_t)(sa_ + (R * SC + 8 * g) * 4);
#pragma unroll
      for (int u = 0; u < 4; ++u) sd[4 * g + u] = v[u];
    };
    auto load_p = [&](int u, int g) {
      const f32x4_t v = *(lds_f4)(uintptr_t)(pa_ + (u * 4 + g) * 1024);
#pragma unroll
      for (int x = 0; x < 4; ++x) pv[u][4 * g + x] = v[x];
    };
    auto mfma_op = [&](int j, int us, int ug, bool score, bool grad) {
      const int x = j / 2;
      if (j % 2 == 0 && score) s[us] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows[x], kv[us][x], x == 0 ? sd : s[us], 0, 0, 0);
      if (j % 2 == 1 && grad) {
        const int G = x / DT, t = x % DT;
        mfma_acc(acc[ug][t], cols[G][t], __builtin_bit_cast(bf16x8_t, make_uint4(pf[ug][G][0], pf[ug][G][1], pf[ug][G][2], pf[ug][G][3])));
      }
    };
    float tm = 0.f;
    const int nm = 4 * half - col;
    auto pack = [&](int u, int k) { pf[u][k / 4][k % 4] = pack_bf16x2(s[u][2 * k], s[u][2 * k + 1]); };
    auto valu_op = [&](int j, int u, bool mask) {
      if constexpr (R == 0) {
        const int e = j;
        if (e == 0) tm = s[u][0] * scale_log2e;
        float p = fast_exp2(tm);
        if (e < 15) tm = s[u][e + 1] * scale_log2e;
        if (mask) p = nm + 8 * (e / 4) + e % 4 >= 0 ? p : 0.f;
        s[u][e] = p;
        if (e >= 2 && e % 2 == 0) pack(u, e / 2 - 1);
        if (e == 15) pack(u, 7);
        if ((e % 4 == 0 && e > 0) || e == 15) {  // four rows of P for the other wave
          const int g = e == 15 ? 3 : e / 4 - 1;
          const f32x4_t v = {s[u][4 * g], s[u][4 * g + 1], s[u][4 * g + 2], s[u][4 * g + 3]};
          *(__attribute__((address_space(3))) f32x4_t*)(uintptr_t)(pa_ + (u * 4 + g) * 1024) = v;
        }
      } else {  // P arrives in the first positions of part A
        if (j >= 6 && j < 14) {
          const int e = 2 * (j - 6);
          s[u][e] *= pv[u][e];
          s[u][e + 1] *= pv[u][e + 1];
        }
        if (j >= 7 && j < 15) pack(u, j - 7);
      }
    };
#define DKV_PART(SECOND, US, UV, SCORE, VAL, MASK, GRAD)                                 \
  {                                                                                      \
    _Pragma("unroll") for (int j = 0; j < NM; ++j) {                                     \
      mfma_op(j, US, 1 - UV, SCORE, GRAD);                                               \
      __builtin_amdgcn_sched_barrier(0);                                                 \
      if (VAL) valu_op(j, UV, MASK);                                                     \
      if (!(SECOND)) {                                                                   \
        if (R == 1 && j < 4) load_p(0, j);                                               \
        if (R == 1 && j >= 12) load_p(1, j - 12);                                        \
        if (j >= 1 && j < 5) load_seed(j - 1);                                           \
        if (j >= LAG) load_op(j - LAG);                                                  \
        if (j % 4 == 1) bring_op(j / 4);                                                 \
      } else if (j < LAG) {                                                              \
        load_op(NM - LAG + j);                                                           \
      }                                                                                  \
      __builtin_amdgcn_sched_barrier(0);                                                 \
    }                                                                                    \
  }
    int T = 0, t0 = 0, cb = 0, nb = 1, ni = 0, nsb = 0;  // step, its tile's number in the head; of tile T - R the buffer and the next one's; of the next tile the number and the seeds
    auto begin = [&]() {
      if (t0 % (SC / BQ) == 0 && T < NT) {  // the first step of a chunk: the one two further on is written
        seeds_commit();
        seeds_fetch();
      }
      ni = ni + 1 == ns ? 0 : ni + 1;
      nsb = ni % (SC / BQ) == 0 ? (nsb + 1) % NS : nsb;
    };
    auto end = [&]() {
      ++T;
      t0 = t0 + 1 == ns ? 0 : t0 + 1;
      cb = nb;
      nb = nb == NB - 1 ? 0 : nb + 1;
      asm volatile("s_waitcnt vmcnt(4)" ::: "memory");  // all but the tile asked for last
      group_barrier();
    };
    auto from = [&](int br) {
#pragma unroll
      for (int x = 0; x < 2 * DT; ++x) ta_[x] = (tat ^ (uint32_t)(x << 5)) + cb * kB;
#pragma unroll
      for (int x = 0; x < KS; ++x) ra_[x] = (rat ^ (uint32_t)(x << 5)) + br * kB;
      sa_ = sat + (uint32_t)(nsb * 2 * SC + ni % (SC / BQ) * BQ) * 4;
      pa_ = pat + (uint32_t)((T - R) & 1) * (2 * 2 * 4 * 64 * 16);
    };
    auto pin = [&](int u) {  // the operands of a part's last elements are made in that part, not behind the next branch
#pragma unroll
      for (int G = 0; G < 2; ++G) asm volatile("" ::"v"(pf[u][G][0]), "v"(pf[u][G][1]), "v"(pf[u][G][2]), "v"(pf[u][G][3]));
    };
    auto idle = [&]() {
      begin();
      bring();
      end();
    };
    if (R == 1) {  // a step behind
      bring();
      if (NT > 0) {
        seeds_commit();
        seeds_fetch();
      }
      ++T;
      t0 = ns == 1 ? 0 : 1;
      asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      group_barrier();
    }
    for (int g = 0; g < G_; ++g) {
      int i = 0;
      for (; i < min(2 * pair, ns); ++i) idle();
      if (i < ns) {
        from(cb);
#pragma unroll
        for (int q = 0; q < 4; ++q) load_seed(q);
#pragma unroll
        for (int j = 0; j < NM; j += 2) load_op(j);
        begin();
#pragma unroll
        for (int j = 0; j < NM; j += 2) mfma_op(j, 0, 1, true, false);
        __builtin_amdgcn_sched_barrier(0);
        from(nb);
        DKV_PART(false, 1, 0, false, true, true, false)
        bring_end();
        DKV_PART(true, 0, 1, true, false, false, true)
        end();
        if (++i < ns) {
          begin();
          from(nb);
          DKV_PART(false, 1, 0, true, true, false, false)
          bring_end();
          DKV_PART(true, 0, 1, true, true, true, true)
          pin(1);
          end();
          for (++i; i < ns; ++i) {
            begin();
            from(nb);
            DKV_PART(false, 1, 0, true, true, false, true)
            bring_end();
            DKV_PART(true, 0, 1, true, true, false, true)
            pin(1);
            end();
          }
#pragma unroll
          for (int j = 1; j < NM; j += 2) mfma_op(j, 0, 1, false, true);
        }
        acc_settle();
      }
    }
    if (R == 0) idle();
#undef DKV_PART
  };
  seeds_fetch();
  seeds_commit();
  seeds_fetch();
  seeds_commit();
  seeds_fetch();
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int x = 0; x < KS; ++x) asm volatile("" ::"a"(kv[u][x]));
  bring();
  bring();
  bring();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  group_barrier();
  if (role == 0) work(std::integral_constant<int, 0>{});
  else work(std::integral_constant<int, 1>{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing is on its way into LDS that others may own soon
  acc_settle();
  OT* out = role ? dK : dV;
  const float mul = role ? scale : 1.f;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int mk = ka + 32 * u + col;
    if (mk >= bend) continue;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16_t& a = acc[u][t];
        const float r4[4] = {mul * a[4 * g], mul * a[4 * g + 1], mul * a[4 * g + 2], mul * a[4 * g + 3]};
        st4(out, (kh + mk) * D + 32 * t + 8 * g + 4 * half, r4);
      }
  }
}

// dQ: a wave owns 64 queries, tiles of keys are staged from the diagonal back to the block's first key: the masked tiles come first,
// in code of their own in front of the loop (behind it, the compiler spilled at D = 128).  Unit a is the later half of the queries:
// in the first step, keys 32 .. 63 meet a alone, keys 0 .. 31 meet a and, masked, b.  Four buffers: the requests of step i for tile
// i + 2 are only waited for in the middle of step i + 1.
template <int D, typename OT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) k_flash_bwd_dq_wide(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
    const float* __restrict__ LSE, const float* __restrict__ delta, OT* __restrict__ dQ, int N, int Bs, int Hq, int Hkv,
    int nbatch, int chunk, float scale, float scale_log2e) {
  constexpr int KS = D / 16, DT = D / 32, NM = 2 * KS + 2 * DT, LAG = NM / 3, CPR = D / 8, NCH = BN * CPR / 256;
  constexpr int NB = 4, kTile = BN * D, kB = kTile * 2;
  __shared__ __attribute__((aligned(256))) bf16_t tiles[2][NB][kTile];  // K, V
  const int tpg = (Bs + TR - 1) / TR;
  const FlashTile ft = flash_tile_of(tpg, N / Bs, Hq, nbatch, tpg, chunk);
  if (!ft.ok) return;
  const int hq = ft.h, b = ft.b, hk = hq / (Hq / Hkv);
  const size_t qh = ((size_t)b * Hq + hq) * N, kh = ((size_t)b * Hkv + hk) * N;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, col = lane % 32, half = lane / 32;
  const int kbeg = ft.blk * Bs, bend = kbeg + Bs, t0 = tpg - 1 - ft.t, q0 = kbeg + t0 * TR;  // long rows first
  const int wa = q0 + 64 * wave;  // the wave's queries: wa .. wa + 63
  const int ns = (min(q0 + TR, bend) - kbeg + BN - 1) / BN;

  bf16x8_t qf[2][KS], gf[2][KS];
  float lse2[2], dl[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const size_t n = qh + min(wa + 32 * (1 - u) + col, bend - 1);
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      qf[u][x] = *reinterpret_cast<const bf16x8_t*>(Q + n * D + 16 * x + 8 * half);
      gf[u][x] = *reinterpret_cast<const bf16x8_t*>(dO + n * D + 16 * x + 8 * half);
    }
    lse2[u] = LSE[n] * 1.4426950408889634f;
    dl[u] = delta[n];
  }
  f32x16_t dq[2][DT];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int t = 0; t < DT; ++t) dq[u][t] = zero16();

  const bf16_t *Kh = K + kh * D, *Vh = V + kh * D;
  const int srow = tid / CPR, schunk = (tile_at<D>(srow, tid % CPR) - srow * D) / 8;
  const uint32_t lds0 = lds_addr(&tiles[0][0][0]) + wave * 1024;
  int fk = kbeg + (ns - 1) * BN;  // from the diagonal to the block's first key
  auto bring_op = [&](int k, int buf) {  // the k-th of the 2 NCH requests of a tile; past the first tile that one again, which nobody reads
    const int u = k / 2;
    const uint32_t off = (uint32_t)(min(max(fk, kbeg) + BN / NCH * u + srow, bend - 1) * D + 8 * schunk) * 2;
    rows_to_lds(lds0 + (k % 2 * NB + buf) * kB + u * 4096, off, k % 2 ? Vh : Kh);
  };
  auto bring = [&](int buf) {
#pragma unroll
    for (int k = 0; k < 2 * NCH; ++k) bring_op(k, buf);
    fk -= BN;
  };
  auto arrived = [&]() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NCH) : "memory"); };  // all but the tile brought last

  const uint32_t rat = lds_addr(&tiles[0][0][tile_at<D>(col, half)]);
  const uint32_t tat = lds_addr(&tiles[0][0][tile_at<D>(4 * half + (lane % 16) / 4, 2 * ((lane / 16) % 2) + (lane % 4) / 2) + 4 * (lane % 2)]);
  uint32_t ra_[KS], ta_[2 * DT];
  auto rows_from = [&](int buf) {
#pragma unroll
    for (int x = 0; x < KS; ++x) ra_[x] = (rat ^ (uint32_t)(x << 5)) + buf * kB;
  };
  auto cols_from = [&](int buf) {
#pragma unroll
    for (int x = 0; x < 2 * DT; ++x) ta_[x] = (tat ^ (uint32_t)(x << 5)) + buf * kB;
  };
  bf16x8_t rows[2][KS], cols[2][DT];
  f32x16_t s[2], dp[2];
  uint32_t df[2][2][4];
  auto load_op = [&](int j, int qr, int qc) {
    if (j % 3 < 2) {
      rows[j % 3][j / 3] = *(lds_frag)(uintptr_t)(ra_[j / 3] + (j % 3 * NB * kB + qr * 32 * D * 2));
    } else {
      const int G = j / 3 / DT, t = j / 3 % DT;
      const uint32_t o = (qc * 32 + G * 16) * D * 2;
      cols[G][t] = tr_join(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(ta_[2 * t] + o)),
                           __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(ta_[2 * t + 1] + (o + 8 * D * 2))));
    }
  };
  auto mfma_op = [&](int j, int us, int ug, bool sdp, bool grad) {
    const int x = j / 3;
    if (j % 3 == 0 && sdp) s[us] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows[0][x], qf[us][x], x == 0 ? zero16() : s[us], 0, 0, 0);
    if (j % 3 == 1 && sdp) dp[us] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows[1][x], gf[us][x], x == 0 ? zero16() : dp[us], 0, 0, 0);
    if (j % 3 == 2 && grad) {
      const int G = x / DT, t = x % DT;
      mfma_acc(dq[ug][t], cols[G][t], __builtin_bit_cast(bf16x8_t, make_uint4(df[ug][G][0], df[ug][G][1], df[ug][G][2], df[ug][G][3])));
    }
  };
  float tm = 0.f;
  const int nm = col - 4 * half;
  auto valu_op = [&](int e, int u, bool mask) {
    if (e == 0) tm = fmaf(s[u][0], scale_log2e, -lse2[u]);
    float p = fast_exp2(tm);
    if (e < 15) tm = fmaf(s[u][e + 1], scale_log2e, -lse2[u]);
    if (e > 0) dp[u][e - 1] = s[u][e - 1] * (dp[u][e - 1] - dl[u]);
    if (mask) p = 8 * (e / 4) + e % 4 <= nm ? p : 0.f;
    s[u][e] = p;
    if (e >= 2 && e % 2 == 0) df[u][(e / 2 - 1) / 4][(e / 2 - 1) % 4] = pack_bf16x2(dp[u][e - 2], dp[u][e - 1]);
    if (e == 15) {
      dp[u][15] = p * (dp[u][15] - dl[u]);
      df[u][1][3] = pack_bf16x2(dp[u][14], dp[u][15]);
    }
  };
#define DQ_PART(SECOND, US, UV, SDP, VAL, MASK, GRAD, QR, QC, BRING)                     \
  {                                                                                      \
    _Pragma("unroll") for (int j = 0; j < NM; ++j) {                                     \
      mfma_op(j, US, 1 - UV, SDP, GRAD);                                                 \
      __builtin_amdgcn_sched_barrier(0);                                                 \
      if (VAL) {                                                                         \
        _Pragma("unroll") for (int e = j * 16 / NM; e < (j + 1) * 16 / NM; ++e) valu_op(e, UV, MASK); \
      }                                                                                  \
      if (!(SECOND) && j >= LAG) load_op(j - LAG, QR, QC);                               \
      if ((SECOND) && j < LAG) load_op(NM - LAG + j, QR, QC);                            \
      if ((BRING) && j % 3 == 1) bring_op(j / 3, nn);                                    \
      __builtin_amdgcn_sched_barrier(0);                                                 \
    }                                                                                    \
  }
  // the operands are here before the first row is asked for: a wait for them behind that would be one for the rows
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      if constexpr (D == 64) asm volatile("" ::"v"(qf[u][x]), "v"(gf[u][x]));
      else asm volatile("" ::"a"(qf[u][x]), "a"(gf[u][x]));
    }
    asm volatile("" ::"v"(lse2[u]), "v"(dl[u]));
  }
  bring(0);
  bring(1);
  arrived();
  group_barrier();
  int cur = 0, i = 0, nxt, nn;
  const int first = wa < bend ? ns - 1 - (wa - kbeg) / BN : ns;  // the step with the wave's diagonal; none if the block ends before the wave
  auto next = [&]() {
    nxt = cur == NB - 1 ? 0 : cur + 1;
    nn = nxt == NB - 1 ? 0 : nxt + 1;
  };
  for (; i < first; ++i) {
    next();
    bring(nn);
    arrived();
    group_barrier();
    cur = nxt;
  }
  if (i < ns) {
    next();
    rows_from(cur);
    cols_from(cur);
#pragma unroll
    for (int j = 0; j < NM; ++j)
      if (j % 3 < 2) load_op(j, 1, 1);
#pragma unroll
    for (int j = 0; j < NM; ++j) mfma_op(j, 0, 1, true, false);
    __builtin_amdgcn_sched_barrier(0);
    DQ_PART(false, 1, 0, false, true, true, false, 0, 1, true)
    fk -= BN;
    DQ_PART(true, 0, 1, true, false, false, true, 0, 1, false)
    arrived();
    group_barrier();
    rows_from(nxt);
    DQ_PART(false, 1, 0, true, true, false, false, 1, 0, false)
    DQ_PART(true, 0, 1, true, true, true, true, 1, 0, false)
    cur = nxt;
    for (++i; i < ns; ++i) {
      next();
      cols_from(cur);
      DQ_PART(false, 1, 0, true, true, false, true, 0, 1, true)
      fk -= BN;
      DQ_PART(true, 0, 1, true, true, false, true, 0, 1, false)
      arrived();
      group_barrier();
      rows_from(nxt);
      DQ_PART(false, 1, 0, true, true, false, true, 1, 0, false)
      DQ_PART(true, 0, 1, true, true, false, true, 1, 0, false)
      cur = nxt;
    }
#pragma unroll
    for (int j = 2; j < NM; j += 3) mfma_op(j, 0, 1, false, true);
    acc_settle();
  }
#undef DQ_PART
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing is on its way into LDS that others may own soon
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int nq = wa + 32 * (1 - u) + col;
    if (nq >= bend) continue;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16_t& a = dq[u][t];
        const float r4[4] = {scale * a[4 * g], scale * a[4 * g + 1], scale * a[4 * g + 2], scale * a[4 * g + 3]};
        st4(dQ, (qh + nq) * D + 32 * t + 8 * g + 4 * half, r4);
      }
  }
}

}  // namespace

// Where a workgroup's fixed part (operands of 256 rows, the masked steps, 64 KB of results) shows, the kernels of 128 rows with two
// or three workgroups on a CU are better.  us, 128 rows / 256 rows:
//   dQ      blocks of 384 35 / 102 at 1024 groups, 22 / 29 at 256; of 640 138 / 187 at 1024, 44 / 51 at 256; of 1024 85 / 84 at 256
//           groups, 51 / 41 at 128, 33 / 28 at 64, 24 / 26 at 32 (128 tiles of 256 rows: half of the chip's CUs); of 2048 39 / 42 at
//           16 groups, 55 / 46 at 32.  D = 128: 81 / 86 (640, 256 groups), 164 / 147 (1024, 256), 37 / 41 (1024, 32), 65 / 67 (2048, 16).
//   dK/dV   blocks of 256 74 / 81 at 1024 groups, 15 / 16 at 64; of 320 110 / 98 and 18 / 18; of 128 37 / 41 and 12 / 11.  D = 128:
//           blocks of 384 223 / 255 at 1024 groups, 25 / 24 at 64; of 512 107 / 105 at 256, 31 / 29 at 64; of 640 454 / 459 and 45 / 35.
//           Few groups need no clause here, although the larger tiles halve the workgroups at D = 64: the longest tile sets the
//           time, and it has twice the keys but reads each query once for them.  At 1 group and at 16: blocks of 320 17 / 16 and 17 /
//           16, of 512 19 / 20 and 20 / 20, of 1024 31 / 30 and 31 / 31, of 2048 53 / 51 and 53 / 52, of 4096 98 / 92 and 140 / 98,
//           of 16k 574 / 386 and 1200 / 948; four query heads per group 56 / 51 and 57 / 52 (512), 2158 / 1412 and 5011 / 3717 (16k).
//           D = 128: of 512 26 / 25 and 27 / 26, of 2048 77 / 68 and 79 / 69, of 16k 1148 / 975 and 2673 / 2187.
bool muse_attn_dq_wide(const MuseDims& d, int Bs) {
  return Bs >= 4 * TR && (long long)((Bs + TR - 1) / TR) * d.B * d.Hq * (d.N / Bs) > 128;
}
bool muse_attn_dkv_wide(const MuseDims& d, int Bs) { return d.D == 64 ? Bs > TR : Bs >= 2 * TR; }

// Rows go from memory to LDS 16 bytes at a time, from 16-byte boundaries: tensors that begin elsewhere (a view one element into
// its storage) are read through registers by the kernels of 128 rows, where any address will do.
bool muse_attn_rows_to_lds(const void* Q, const void* K, const void* V, const void* dO) {
  return ((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)dO) % 16 == 0;
}

// the gradients may leave in bf16 (MuseDims::grads16): all of them come from the kernels of this file
bool muse_attn_bwd_writes16(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V, const void* dO) {
  return d.dtype == MUSE_DTYPE_BF16 && muse_attn_dq_wide(d, Bs) && muse_attn_dkv_wide(d, Bs) && muse_attn_rows_to_lds(Q, K, V, dO);
}

int muse_launch_attn_dq_wide(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                             const float* delta, void* dQ, hipStream_t st) {
  const int tiles = (Bs + TR - 1) / TR, groups = d.B * d.Hq * (d.N / Bs);
  MuseProf prof_("k_flash_bwd_dq", st);
  auto go = [&](auto* kernel, auto* out) {
    hipLaunchKernelGGL(kernel, flash_grid_of(tiles, groups), dim3(256), 0, st, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V,
                       (const bf16_t*)dO, LSE, delta, out, d.N, Bs, d.Hq, d.Hkv, d.B, chunk_groups(Bs, d.D, groups), d.scale, d.scale * 1.4426950408889634f);
  };
  if (d.grads16) d.D == 64 ? go(k_flash_bwd_dq_wide<64, bf16_t>, (bf16_t*)dQ) : go(k_flash_bwd_dq_wide<128, bf16_t>, (bf16_t*)dQ);
  else d.D == 64 ? go(k_flash_bwd_dq_wide<64, float>, (float*)dQ) : go(k_flash_bwd_dq_wide<128, float>, (float*)dQ);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_attn_dkv_wide(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                              const float* delta, void* dK, void* dV, hipStream_t st) {
  const int tr = d.D == 64 ? TR : TR128, tiles = (Bs + tr - 1) / tr, groups = d.B * d.Hkv * (d.N / Bs);
  MuseProf prof_("k_flash_bwd_dkv", st);
  auto go = [&](auto* kernel, auto* k, auto* v) {
    hipLaunchKernelGGL(kernel, flash_grid_of(tiles, groups), dim3(256), 0, st, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V,
                       (const bf16_t*)dO, LSE, delta, k, v, d.N, Bs, d.Hq, d.Hkv, d.B, chunk_groups(Bs, d.D, groups), d.scale, d.scale * 1.4426950408889634f);
  };
  auto as = [&](auto* k, auto* v) {
    using OT = std::remove_pointer_t<decltype(k)>;
    d.D == 64 ? go(k_flash_bwd_dkv_wide<OT>, k, v) : go(k_flash_bwd_dkv128_wide<OT>, k, v);
  };
  if (d.grads16) as((bf16_t*)dK, (bf16_t*)dV);
  else as((float*)dK, (float*)dV);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
