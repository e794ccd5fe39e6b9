// bf16 causal attention, forward (Sec. 3, Eq. 1-2; Sec. 3.3 "Local attention"): keys restricted to the query's own spatial
// block of size Bs (Bs = N gives exact attention), the far-field partial state merged in the epilogue.
//
// S^T = K Q^T on MFMA 32x32x16, a wave owning 32 queries as the columns, so that every softmax quantity lives in one lane
// (two: the halves hold different keys) and the probabilities go from the accumulators straight back as the operand of
// O^T += V^T P^T.  Per score and lane that is D / 8 matrix cycles against some twenty vector cycles, so what counts is that
// the two pipes of a SIMD work at the same time.  Left to themselves the waves of a SIMD take turns (matrix 0.36 + vector
// 0.59 busy at D = 64), so they are set against each other: a workgroup has two waves per SIMD, w and w + 4; a step of 64
// keys is two phases,
//   M  S(i) = K(i) Q^T and O += V(i-1) P(i-1)      V  masks, maximum, exponentials and P(i)
// with a barrier behind each, and waves 4 .. 7 run one phase behind waves 0 .. 3: while one half is in M the other is in V.
// A tile of keys or values lies in LDS once, row-major, and serves both operand forms (lds_tile.h).  The rows go there straight
// from memory: every wave asks for its share of K(i+2) and V(i+1) in M(i), waits for it in V(i), and the barrier behind that V
// phase makes the tile complete, at the latest (the late half's) one phase before the early half first reads K(i+2), in V(i+1).
// Three buffers each: the late half reads K(i) and V(i-1) in its M(i), a phase after the early half's; the barrier behind that
// phase separates the read from the early half's M(i+1), which asks for K(i+3) and V(i+2) into the same buffers.  With two the
// rows would arrive while they are still read.
//
// What it takes now (cycles per step and wave at exact attention over 16k tokens, D = 64): M 930 to 1180 for 512 of matrix
// instructions, V 860 to 1120 for some 130 vector instructions of which 32 are exponentials; the two pipes still slow each
// other down.  What brought it there, us at 8 heads of 16k / 32 heads of 8k with D = 128: one workgroup of four waves with 64 (32) queries each and a
// transposed value tile 480 / 700; two phases and mirrored tiles 420 / 717; rows straight to LDS and operand addresses as xor
// of a base 400 / 580; the maximum looked for only when a probability says so, and one LDS read behind each matrix instruction
// instead of groups of them 355 / 513; wave priority in M 344 / 515.
#include <type_traits>

#include "ff_common.h"
#include "flash_tile.h"
#include "lds_tile.h"

namespace {

constexpr int BN = 64;           // keys per step
constexpr int TR = 256;          // queries of a workgroup's tile
constexpr float kLazyLog2 = 8.f;  // the softmax reference follows the running maximum in steps of more than 2^8

// acc + the sum of the 8 bf16 values of an operand (v_dot2c_f32_bf16 against a pair of ones: two values per
// instruction, where adding the fp32 values takes one each)
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ float sum8(const bf16x8_t& v, float acc) {
  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bf16x2_t p = {v[2 * i], v[2 * i + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(p, ones, acc, false);
  }
  return acc;
}

// The tiles are those of one block: the last one has what is left of it, and a wave that is left without a query steps once and
// brings rows.  With tiles of the whole sequence for blocks that are no multiple of 256, every step masked every score, and a
// wave whose block starts behind its tile's looked for its maximum in steps without a key of its own (us, 8 blocks, whole
// sequence / per block: 64 / 36 at 12 heads with blocks of 749, 184 / 83 with 1408, 531 / 303 at 32 heads with 2176; D = 128,
// 12 heads: 210 / 129 with 1408, 66 / 49 with 640).
// The order of the tiles.  A CU holds one workgroup, a tile of a block is as long as its number, and workgroups are dispatched in
// order, so a short tile handed out late and a long one handed out last both leave CUs idle.  Two ways to spread them:
//   fold    a workgroup takes a long tile and the one that mirrors it; all are equally long.  For even numbers of tiles whose
//           halves come out even on 256 CUs.
//   chunk   else: long tiles first, over as many groups of an XCD as have 8 MB of keys and values (twice its L2; with 4 and
//           16 MB or all groups the same at blocks up to 1k, at 32 heads of 32k with D = 128 1312, 1283 and 1407 against 1274).
// us, group by group / folded / in chunks, groups being heads x blocks: 64 groups of 3 tiles 24 / 34 / 25, 160 of 3 45 / 66 / 40, 96 of
// 4 52 / 41 / 39, 160 of 4 78 / 78 / 61, 96 of 5 57 / 65 / 47, 320 of 7 273 / 277 / 262, 160 of 8 196 / 178 / 165; where folding
// comes out even: 128 of 4 54 / 44 / 46, 64 of 8 85 / 61 / 63, 8 of 64 (exact attention over 16k) 295 / 285 / 294, 128 of 32 1550 /
// 1429 / 1436.
static int fold_tiles(int tpg, int groups) { return tpg % 2 == 0 && (long long)(tpg / 2) * groups % 256 == 0; }

// The end of a phase.  No release or acquire: what the waves exchange are rows that arrive in LDS by themselves and are
// waited for by count, and every LDS read of a phase has fed a matrix instruction before the phase ends.
__device__ __forceinline__ void phase_end() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

using lds_frag = __attribute__((address_space(3))) const bf16x8_t*;
using lds_tr = __attribute__((address_space(3))) s16x4_t*;

template <int D>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) k_flash_fwd(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const float* __restrict__ ff,
    bf16_t* __restrict__ O, float* __restrict__ LSE, int N, int Bs, int Hq, int Hkv, int nbatch, int fold, int tiles, int chunk, float scale_log2e) {
  constexpr int KS = D / 16, DT = D / 32, CPR = D / 8, NCH = BN * CPR / 512, kTile = BN * D, NG = KS / 2, NF = 3;
  __shared__ __attribute__((aligned(256))) bf16_t ks[3][kTile];
  __shared__ __attribute__((aligned(256))) bf16_t vs[3][kTile];
  const FlashTile ft = flash_tile_of((Bs + TR - 1) / TR, N / Bs, Hq, nbatch, tiles, chunk);
  if (!ft.ok) return;
  const int hq = ft.h, b = ft.b, hk = hq / (Hq / Hkv);
  const size_t qh = ((size_t)b * Hq + hq) * N, kh = ((size_t)b * Hkv + hk) * N;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, col = lane % 32, half = lane / 32;
  const bool late = wave >= 4;  // a phase behind
  const int kbeg = ft.blk * Bs, bend = kbeg + Bs;  // the block; its last tile may have fewer than TR rows
  const bf16_t *Kh = K + kh * D, *Vh = V + kh * D;

  // LDS addresses of this lane's operands (tile_row, tile_cols of lds_tile.h) in the first buffer: the other operands of a
  // step differ by a constant, or by an xor with a constant in the chunk bits.
  const uint32_t kat = lds_addr(ks[0] + tile_at<D>(col, half));
  const uint32_t vat = lds_addr(vs[0] + tile_at<D>(4 * half + (lane % 16) / 4, 2 * ((lane / 16) % 2) + (lane % 4) / 2) + 4 * (lane % 2));
  // The chunk of a tile that this thread brings in: LDS takes them in order of the thread, so the swizzle is in the source.
  const int srow = tid / CPR, schunk = (tile_at<D>(srow, tid % CPR) - srow * D) / 8;  // the swizzle is its own inverse

  for (int part = 0; part <= fold; ++part) {
    const int t = part == 0 ? ft.tpg - 1 - ft.t : ft.t;  // long rows first
    const int q0 = kbeg + t * TR;
    const int w0 = q0 + 32 * wave, nq = w0 + col, nqc = min(nq, bend - 1);
    const int kend = min(q0 + TR, bend), nt = (kend - kbeg + BN - 1) / BN;
    bf16x8_t qf[KS];
#pragma unroll
    for (int x = 0; x < KS; ++x) qf[x] = *reinterpret_cast<const bf16x8_t*>(Q + (qh + nqc) * D + 16 * x + 8 * half);

    // K(c) and V(c-1) into their buffers, straight from memory to LDS.  No branch: behind one, every LDS read in flight would
    // be waited for.  Rows past the block's end are its last row again, whose scores are masked or whose tile nobody reads.
    auto bring = [&](int c) {
      using gptr = const __attribute__((address_space(1))) void*;
      using lptr = __attribute__((address_space(3))) void*;
      const int rk = min(kbeg + c * BN, bend - 1), rv = max(min(kbeg + c * BN - BN, bend - 1), kbeg);
      const bf16_t *sk = Kh + (size_t)rk * D, *sv = Vh + (size_t)rv * D;
      bf16_t *dk = ks[c % 3] + wave * 512, *dv = vs[(c + 2) % 3] + wave * 512;
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const int row = srow + BN / NCH * u;
        __builtin_amdgcn_global_load_lds((gptr)(sk + (uint32_t)(min(row, bend - 1 - rk) * D + 8 * schunk)), (lptr)(dk + 4096 * u), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((gptr)(sv + (uint32_t)(min(row, bend - 1 - rv) * D + 8 * schunk)), (lptr)(dv + 4096 * u), 16, 0, 0);
      }
    };
    auto arrived = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

    f32x16_t o[DT], s[2];
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2) o[t2] = zero16();
    bf16x8_t pf[2][2];   // P(i): [key half][16-key group]
    bf16x8_t f[NF][4];   // groups of operands
    float m = MUSE_NEG_INF, l = 0.f;

    // operand u of group g: four of K(i), then as many groups of V(i-1)
    auto load = [&](int g, int u, int i) {
      const int k = 4 * (g % NG) + u;
      if (g < NG) {
        const uint32_t kb = kat + (uint32_t)(i % 3) * (kTile * 2);
        f[g % NF][u] = *(lds_frag)(uintptr_t)((kb ^ (uint32_t)((k % KS) << 5)) + (k / KS) * (32 * D * 2));
      } else {
        const uint32_t at = (vat + (uint32_t)((i + 2) % 3) * (kTile * 2)) ^ (uint32_t)((k % DT) << 6), rows = (k / DT) * (16 * D * 2);
        f[g % NF][u] = tr_join(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)(at + rows)),
                               __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)((at ^ 0x20u) + (rows + 8 * D * 2))));
      }
    };
    // M(i).  An operand is requested two groups of four ahead of its matrix instruction (the first two groups of K during the V
    // phase before), one behind each instruction: four waves read at a time, and a wave that issues its reads in a row stands
    // still until LDS has taken them.  The rows of step i + 2 are requested behind the last read (an LDS read behind such a
    // request would wait for its rows).
    auto matrix_phase = [&](auto qk, auto pv, int i) {
      constexpr int G0 = qk ? 0 : NG, G1 = pv ? 2 * NG : NG;
      __builtin_amdgcn_s_setprio(1);  // a matrix instruction a step late is a gap in its pipe; the other wave has slots enough
      if constexpr (!qk) {
#pragma unroll
        for (int u = 0; u < 8; ++u) load(G0 + u / 4, u % 4, i);
      }
#pragma unroll
      for (int g = G0; g < G1; ++g) {
        if (g == (G0 > G1 - 2 ? G0 : G1 - 2)) bring(i + 2);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = 4 * (g % NG) + u;
          __builtin_amdgcn_sched_barrier(0);
          if (g < NG) {
            if (k % KS == 0) s[k / KS] = zero16();
            s[k / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[g % NF][u], qf[k % KS], s[k / KS], 0, 0, 0);
          } else {
            o[k % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[g % NF][u], pf[k / DT / 2][k / DT % 2], o[k % DT], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (g + 2 < G1) load(g + 2, u, i);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
    };
    // P(i) = exp2(c S(i) - ref) as operands; whether any of them is 2 or more (the bf16 exponent's highest bit, set for an
    // infinity and a NaN too), and the sum of what the matrix cores will see.  The first
    // operands of the next M phase are requested in between.
    auto probs = [&](float ref, float& psum, int next) {
      uint32_t any = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x16_t p;
#pragma unroll
        for (int G = 0; G < 2; ++G) {
#pragma unroll
          for (int e = 8 * G; e < 8 * G + 8; ++e) p[e] = fast_exp2(fmaf(s[h][e], scale_log2e, -ref));
          pf[h][G] = pack8(p, 2 * G, 2 * G + 1);
          const uint4 w = __builtin_bit_cast(uint4, pf[h][G]);
          any |= w.x | w.y | w.z | w.w;
          psum = sum8(pf[h][G], psum);  // the normaliser sums the probabilities as the matrix cores see them
          __builtin_amdgcn_sched_barrier(0);
          load(h, 2 * G, next);
          load(h, 2 * G + 1, next);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      return (any & 0x40004000u) != 0;
    };
    // V(i): P(i) from S(i).  The reference m of the running softmax is 2^7 above the maximum that set it and moves only when a
    // probability reaches 2 (the maximum has grown by 2^8): the maximum of a step is looked for, and the accumulators are
    // rescaled, on those steps only.  O = o / l and LSE = m + log2 l hold for any reference as long as o, l and p use
    // the same one.  m = -inf (no key yet) makes every p an infinity or a NaN.
    auto softmax = [&](int i) {
      const int k0 = kbeg + i * BN;
      if (k0 + BN - 1 > w0) {  // wave-uniform
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int kg = k0 + 32 * h + 8 * (e / 4) + 4 * half + (e % 4);
            if (kg > nq) s[h][e] = MUSE_NEG_INF;
          }
      }
      float psum = 0.f;
      arrived();  // the rows requested in M(i)
      if (__builtin_amdgcn_ballot_w64(probs(m, psum, i + 1)) != 0) {
        float tmax = MUSE_NEG_INF;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, s[h][e]);
        typedef uint32_t u2_t __attribute__((ext_vector_type(2)));  // the other half's maximum, without a trip through LDS
        const u2_t x = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
        const float ts = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1])) * scale_log2e;
        const float mn = ts > m + 1.f ? ts + (kLazyLog2 - 1.f) : m;
        const float ref = mn == MUSE_NEG_INF ? 0.f : mn;
        const float alpha = fast_exp2(m - ref);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[t2][e] *= alpha;
        psum = 0.f;
        (void)probs(ref, psum, i + 1);
      }
      l += psum;
    };
    bring(0);
    bring(1);
    arrived();
    phase_end();
#pragma unroll
    for (int u = 0; u < 8; ++u) load(u / 4, u % 4, 0);
    if (late) phase_end();
    // the wave's own steps end with the tile that its last query is in; after that it only brings rows.  A wave that the block
    // leaves without a query has one step.
    const int nw = w0 < kend ? (min(w0 + 31, kend - 1) - kbeg) / BN + 1 : 1;
    matrix_phase(std::true_type(), std::false_type(), 0);
    phase_end();
    softmax(0);
    phase_end();
    for (int i = 1; i < nw; ++i) {
      matrix_phase(std::true_type(), std::true_type(), i);
      phase_end();
      softmax(i);
      phase_end();
    }
    matrix_phase(std::false_type(), std::true_type(), nw);
    phase_end();
    for (int i = nw + 1; i <= nt; ++i) {
      arrived();
      phase_end();
      bring(i + 2);
      phase_end();
    }
    if (!late) phase_end();  // as many barriers for both halves
    arrived();               // nothing is on its way into buffers that others may own soon
    phase_end();

    l += __shfl_xor(l, 32, 64);
    if (nq >= bend) continue;
    float mnat = m * 0.6931471805599453f;  // natural-log units
    float cl = 1.f;                        // weight of the local part after the merge
    float cf = 0.f, lf = 0.f;
    const float* fa = nullptr;
    if (ff) {
      const float* fm = ff + (size_t)nbatch * Hq * N * D + (qh + nq) * 2;  // [acc | (max,sum)] planes
      const float mf = fm[0];
      lf = fm[1];
      if (lf > 0.f) {
        const float mx = fmaxf(mnat, mf);
        cl = __expf(mnat - mx);
        cf = __expf(mf - mx);
        mnat = mx;
        fa = ff + (qh + nq) * D;
      }
    }
    const float lt = l * cl + lf * cf;
    const float inv = 1.f / lt;
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d = 32 * t2 + 8 * g + 4 * half;
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = o[t2][4 * g + u] * cl;
        if (fa) {
          const float4 f = *reinterpret_cast<const float4*>(fa + d);
          v[0] += cf * f.x; v[1] += cf * f.y; v[2] += cf * f.z; v[3] += cf * f.w;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] *= inv;
        st4(O, (qh + nq) * D + d, v);
      }
    if (half == 0) LSE[qh + nq] = mnat + __logf(lt);
  }
}

}  // namespace

int muse_launch_attn_fwd_mfma(const MuseDims& d, int Bs, const void* Q, const void* K, const void* V,
                              const float* ff, void* O, float* LSE, hipStream_t st) {
  const float sl = d.scale * 1.4426950408889634f;
  const int tpg = (Bs + TR - 1) / TR, groups = d.B * d.Hq * (d.N / Bs);
  const int fold = fold_tiles(tpg, groups), tiles = fold ? tpg / 2 : tpg, chunk = fold ? 1 : chunk_groups(Bs, d.D, groups);
  const dim3 g = flash_grid_of(tiles, groups);
  MuseProf prof_("k_flash_fwd", st);
  auto go = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, g, dim3(512), 0, st, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, ff, (bf16_t*)O, LSE, d.N,
                       Bs, d.Hq, d.Hkv, d.B, fold, tiles, chunk, sl);
  };
  if (d.D == 64) go(k_flash_fwd<64>);
  else go(k_flash_fwd<128>);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
