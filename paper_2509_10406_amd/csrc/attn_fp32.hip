// fp32 causal attention on the fp32 matrix instruction (Sec. 3, Eq. 1-2; Sec. 3.3 "Local attention"): keys restricted to
// the query's own spatial block of size Bs (Bs = N gives exact attention), any Bs.  Forward, dQ per query tile, dK/dV per
// key tile; no atomics.
//
// Bound by v_mfma_f32_16x16x4_f32 (256 flop per cycle and CU).  A wave owns 16 queries (forward, dQ) or 16 keys (dK/dV) as
// the columns of the instruction and a workgroup's four waves share the staged rows, 64 at D = 64 and 32 at D = 128 (two
// tensors of 17 KB either way).  16 columns and not 32: the small problems of this type (one head of 2k tokens is 32
// workgroups) need the waves, and the rate is the same.  With c = lane % 16, h = lane / 16:
//   - scores transposed, X[row][.] . y: the lane reads 16 bytes of row c at dims 16u + 4h and feeds four instructions
//     (k-slot h = dims 16u + 4h + t, the same split on both operands);
//   - accumulator element t is row 4h + t, which is the k-slot order of the second contraction, so probabilities stay in
//     registers; its other operand is read 16 bytes of row 4h + t at dims 64g + 4c, one dim for each of four
//     accumulators, which leaves the lane with the dims 64g + 16h .. + 15 of its column: whole float4 results.
// Rows are padded by four floats: both reads then spread over all banks.
// Measured, 4 heads of 8k tokens, D = 64, blocks of 1024 (vector kernels with four lanes per query before): forward
// 407 -> 63 us, dQ 494 -> 79 us, dK/dV 536 -> 105 us (about a third of the instruction rate; one wave per SIMD there).
#include "fp32_sum.h"

namespace {

template <int D>
struct F32Attn {
  static constexpr int kRows = 4096 / D;  // rows staged per step
  static constexpr int kLd = D + 4;
  static constexpr int kSub = kRows / 16;
  static constexpr int kAcc = D / 16;
};

__device__ __forceinline__ f32x4_t mfma16(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Workgroup -> (tile, head row).  All tiles are in one grid dimension; a device of 256 CUs takes them in rounds of 256,
// and every other round runs backwards so that a CU does not meet the same (long or short) part of a block each time.
struct TileId {
  int tile, row;
};
__device__ __forceinline__ TileId tile_id(int tiles, bool last_first) {
  int id = blockIdx.x;
  const int round = id >> 8;
  if ((round & 1) && ((round + 1) << 8) <= (int)gridDim.x) id = (round << 8) + 255 - (id & 255);
  TileId r;
  r.row = id / tiles;
  r.tile = id - r.row * tiles;
  if (last_first) r.tile = tiles - 1 - r.tile;
  return r;
}

// rows r0 .. of X into registers (clamped addresses), and from there into LDS (rows past the end as zeros)
template <int D>
__device__ __forceinline__ void fetch_rows(const float* __restrict__ X, int r0, int N, float4 (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = threadIdx.x + 256 * i;
    int r = r0 + c / (D / 4);
    r = r < N ? r : N - 1;
    v[i] = *reinterpret_cast<const float4*>(X + (size_t)r * D + 4 * (c % (D / 4)));
  }
}
template <int D>
__device__ __forceinline__ void commit_rows(float* lds, const float4 (&v)[4], int r0, int N, float mul) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = threadIdx.x + 256 * i, row = c / (D / 4);
    const bool ok = r0 + row < N;
    const float4 x = v[i];
    *reinterpret_cast<float4*>(lds + row * F32Attn<D>::kLd + 4 * (c % (D / 4))) =
        ok ? make_float4(mul * x.x, mul * x.y, mul * x.z, mul * x.w) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// the lane's column operand: dims 16u + 4h + t of row `row`, times mul; zeros for a row that is not there
template <int D>
__device__ __forceinline__ void load_col(const float* __restrict__ X, int row, bool live, int h, float mul, float (&y)[D / 4]) {
#pragma unroll
  for (int u = 0; u < D / 16; ++u) {
    const float4 x = live ? *reinterpret_cast<const float4*>(X + (size_t)row * D + 16 * u + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
    y[4 * u] = mul * x.x; y[4 * u + 1] = mul * x.y; y[4 * u + 2] = mul * x.z; y[4 * u + 3] = mul * x.w;
  }
}

// 16 staged rows (from `rows`) times the column operand
template <int D>
__device__ __forceinline__ f32x4_t dot_tile(const float* rows, const float (&y)[D / 4], int c, int h) {
  FoldSum s;
#pragma unroll
  for (int u = 0; u < D / 16; ++u) {
    const float4 a = *reinterpret_cast<const float4*>(rows + c * F32Attn<D>::kLd + 16 * u + 4 * h);
    s.add(0, a.x, y[4 * u]);
    s.add(1, a.y, y[4 * u + 1]);
    s.add(2, a.z, y[4 * u + 2]);
    s.add(3, a.w, y[4 * u + 3]);
    s.fold(u);
  }
  return s.total;
}

// acc += p^T . rows over 16 staged rows.  `masked`: some of the (row, column) pairs are not attended and have p = 0; a
// row that holds an infinity or NaN must not reach their columns through 0 * inf, so it is added pair by pair then.  There
// `attends(row)` says which rows the lane's column has (an attended weight that underflowed counts: 0 * inf).
template <int D, typename F>
__device__ __forceinline__ void add_tile(f32x4_t (&acc)[D / 16], const float* rows, const f32x4_t p, int c, int h, bool masked,
                                         F attends) {
  constexpr int LD = F32Attn<D>::kLd;
  float4 a[4][D / 64];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int g = 0; g < D / 64; ++g) a[t][g] = *reinterpret_cast<const float4*>(rows + (4 * h + t) * LD + 64 * g + 4 * c);
  if (masked) {
    float z = 0.f;  // stays zero exactly if every element is finite
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int g = 0; g < D / 64; ++g) z += 0.f * a[t][g].x + 0.f * a[t][g].y + 0.f * a[t][g].z + 0.f * a[t][g].w;
    if (__any(z != 0.f)) {
      for (int k4 = 0; k4 < 4; ++k4) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float pk = __shfl(p[t], 16 * k4 + c, 64);
          if (!attends(4 * k4 + t)) continue;
          const float* row = rows + (4 * k4 + t) * LD + 16 * h;
#pragma unroll
          for (int e = 0; e < D / 4; ++e)
            acc[4 * (e / 16) + e % 4][(e / 4) % 4] = fmaf(pk, row[64 * (e / 16) + e % 16], acc[4 * (e / 16) + e % 4][(e / 4) % 4]);
        }
      }
      return;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int g = 0; g < D / 64; ++g) {
      acc[4 * g] = mfma16(a[t][g].x, p[t], acc[4 * g]);
      acc[4 * g + 1] = mfma16(a[t][g].y, p[t], acc[4 * g + 1]);
      acc[4 * g + 2] = mfma16(a[t][g].z, p[t], acc[4 * g + 2]);
      acc[4 * g + 3] = mfma16(a[t][g].w, p[t], acc[4 * g + 3]);
    }
}

// the lane's dims 64g + 16h + 4t .. + 3 of its column
template <int D>
__device__ __forceinline__ float4 acc_get(const f32x4_t (&acc)[D / 16], int g, int t) {
  return make_float4(acc[4 * g][t], acc[4 * g + 1][t], acc[4 * g + 2][t], acc[4 * g + 3][t]);
}
template <int D>
__device__ __forceinline__ void store_col(const f32x4_t (&acc)[D / 16], float* __restrict__ dst, int h, float mul) {
#pragma unroll
  for (int g = 0; g < D / 64; ++g)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float4 x = acc_get<D>(acc, g, t);
      *reinterpret_cast<float4*>(dst + 64 * g + 16 * h + 4 * t) = make_float4(mul * x.x, mul * x.y, mul * x.z, mul * x.w);
    }
}

template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_fwd_f32(const float* __restrict__ Q, const float* __restrict__ K,
                                                          const float* __restrict__ V, const float* __restrict__ ff,
                                                          float* __restrict__ O, float* __restrict__ LSE, int N, int Bs,
                                                          int Hq, int Hkv, int B, float scale) {
  using A = F32Attn<D>;
  constexpr int R = A::kRows, LD = A::kLd;
  __shared__ __align__(16) float ks[R * LD];
  __shared__ __align__(16) float vs[R * LD];
  const TileId id = tile_id((N + 63) / 64, true);
  const int hq = id.row % Hq, b = id.row / Hq, hk = hq / (Hq / Hkv);
  const size_t qh = ((size_t)b * Hq + hq) * N, kh = ((size_t)b * Hkv + hk) * N;
  const int q0 = id.tile * 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int c = threadIdx.x % 16, h = (threadIdx.x % 64) / 16;
  const int qa = q0 + 16 * w, qz = min(qa + 15, N - 1), n = qa + c;  // the wave's first and last query, the lane's
  const bool live = n < N;
  const int beg_a = (qa / Bs) * Bs, beg_z = (qz / Bs) * Bs, beg = (n / Bs) * Bs;
  float q[D / 4];
  load_col<D>(Q + qh * D, n, live, h, scale, q);
  f32x4_t acc[A::kAcc];
#pragma unroll
  for (int i = 0; i < A::kAcc; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = MUSE_NEG_INF, l = 0.f;
  const int kbeg = (q0 / Bs) * Bs, kend = min(q0 + 64, N);
  float4 kr[4], vr[4];
  fetch_rows<D>(K + kh * D, kbeg, N, kr);
  fetch_rows<D>(V + kh * D, kbeg, N, vr);
  for (int k0 = kbeg; k0 < kend; k0 += R) {
    __syncthreads();
    commit_rows<D>(ks, kr, k0, N, 1.f);
    commit_rows<D>(vs, vr, k0, N, 1.f);
    __syncthreads();
    fetch_rows<D>(K + kh * D, k0 + R, N, kr);
    fetch_rows<D>(V + kh * D, k0 + R, N, vr);
    f32x4_t s[A::kSub];
    float mx = m;
#pragma unroll
    for (int j = 0; j < A::kSub; ++j) {
      const int kj = k0 + 16 * j;
      s[j] = f32x4_t{MUSE_NEG_INF, MUSE_NEG_INF, MUSE_NEG_INF, MUSE_NEG_INF};
      if (qa < N && kj <= qz && kj + 15 >= beg_a) {
        s[j] = dot_tile<D>(ks + 16 * j * LD, q, c, h);
        if (kj + 15 > qa || kj < beg_z) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int key = kj + 4 * h + t;
            if (key > n || key < beg) s[j][t] = MUSE_NEG_INF;
          }
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) mx = fmaxf(mx, s[j][t]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float ref = mx == MUSE_NEG_INF ? 0.f : mx, al = __expf(m - ref);
    m = mx;
    l *= al;
#pragma unroll
    for (int i = 0; i < A::kAcc; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[i][t] *= al;
#pragma unroll
    for (int j = 0; j < A::kSub; ++j) {
      const int kj = k0 + 16 * j;
      if (qa < N && kj <= qz && kj + 15 >= beg_a) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          s[j][t] = __expf(s[j][t] - ref);
          l += s[j][t];
        }
        add_tile<D>(acc, vs + 16 * j * LD, s[j], c, h, kj + 15 > qa || kj < beg_z, [&](int r) { return kj + r >= beg && kj + r <= n; });
      }
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (!live) return;
  float cf = 0.f;
  const float* f = ff + (qh + n) * D;
  if (ff) {  // merge the far-field partial softmax state (max, sum, acc[D])
    const float* fm = ff + (size_t)B * Hq * N * D + (qh + n) * 2;  // [acc | (max,sum)] planes
    const float mf = fm[0], lf = fm[1];
    if (lf > 0.f) {
      const float mn = fmaxf(m, mf), a = __expf(m - mn);
      cf = __expf(mf - mn);
      l = l * a + lf * cf;
#pragma unroll
      for (int i = 0; i < A::kAcc; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[i][t] *= a;
#pragma unroll
      for (int g = 0; g < D / 64; ++g)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float4 x = *reinterpret_cast<const float4*>(f + 64 * g + 16 * h + 4 * t);
          acc[4 * g][t] = fmaf(cf, x.x, acc[4 * g][t]);
          acc[4 * g + 1][t] = fmaf(cf, x.y, acc[4 * g + 1][t]);
          acc[4 * g + 2][t] = fmaf(cf, x.z, acc[4 * g + 2][t]);
          acc[4 * g + 3][t] = fmaf(cf, x.w, acc[4 * g + 3][t]);
        }
      m = mn;
    }
  }
  store_col<D>(acc, O + (qh + n) * D, h, 1.f / l);
  if (h == 0) LSE[qh + n] = m + __logf(l);
}

template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_dq_f32(const float* __restrict__ Q, const float* __restrict__ K,
                                                             const float* __restrict__ V, const float* __restrict__ dO,
                                                             const float* __restrict__ LSE, const float* __restrict__ delta,
                                                             float* __restrict__ dQ, int N, int Bs, int Hq, int Hkv,
                                                             float scale) {
  using A = F32Attn<D>;
  constexpr int R = A::kRows, LD = A::kLd;
  __shared__ __align__(16) float ks[R * LD];
  __shared__ __align__(16) float vs[R * LD];
  const TileId id = tile_id((N + 63) / 64, true);
  const int hq = id.row % Hq, b = id.row / Hq, hk = hq / (Hq / Hkv);
  const size_t qh = ((size_t)b * Hq + hq) * N, kh = ((size_t)b * Hkv + hk) * N;
  const int q0 = id.tile * 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int c = threadIdx.x % 16, h = (threadIdx.x % 64) / 16;
  const int qa = q0 + 16 * w, qz = min(qa + 15, N - 1), n = qa + c;
  const bool live = n < N;
  const int beg_a = (qa / Bs) * Bs, beg_z = (qz / Bs) * Bs, beg = (n / Bs) * Bs;
  float q[D / 4], g[D / 4];
  load_col<D>(Q + qh * D, n, live, h, scale, q);
  load_col<D>(dO + qh * D, n, live, h, 1.f, g);
  const float lse = live ? LSE[qh + n] : 0.f, dl = live ? delta[qh + n] : 0.f;
  f32x4_t acc[A::kAcc];
#pragma unroll
  for (int i = 0; i < A::kAcc; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int kbeg = (q0 / Bs) * Bs, kend = min(q0 + 64, N);
  float4 kr[4], vr[4];
  fetch_rows<D>(K + kh * D, kbeg, N, kr);
  fetch_rows<D>(V + kh * D, kbeg, N, vr);
  for (int k0 = kbeg; k0 < kend; k0 += R) {
    __syncthreads();
    commit_rows<D>(ks, kr, k0, N, 1.f);
    commit_rows<D>(vs, vr, k0, N, 1.f);
    __syncthreads();
    fetch_rows<D>(K + kh * D, k0 + R, N, kr);
    fetch_rows<D>(V + kh * D, k0 + R, N, vr);
#pragma unroll
    for (int j = 0; j < A::kSub; ++j) {
      const int kj = k0 + 16 * j;
      if (!(qa < N && kj <= qz && kj + 15 >= beg_a)) continue;
      const bool masked = kj + 15 > qa || kj < beg_z;
      const f32x4_t s = dot_tile<D>(ks + 16 * j * LD, q, c, h);
      f32x4_t ds = dot_tile<D>(vs + 16 * j * LD, g, c, h);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int key = kj + 4 * h + t;
        ds[t] = __expf(s[t] - lse) * (ds[t] - dl);
        if (masked && (!live || key > n || key < beg)) ds[t] = 0.f;
      }
      add_tile<D>(acc, ks + 16 * j * LD, ds, c, h, masked, [&](int r) { return kj + r >= beg && kj + r <= n; });
    }
  }
  if (live) store_col<D>(acc, dQ + (qh + n) * D, h, scale);
}

// loop over the query heads of the group and, inside, the queries n >= m of the key's block
template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_dkv_f32(const float* __restrict__ Q, const float* __restrict__ K,
                                                              const float* __restrict__ V, const float* __restrict__ dO,
                                                              const float* __restrict__ LSE, const float* __restrict__ delta,
                                                              float* __restrict__ dK, float* __restrict__ dV, int N, int Bs,
                                                              int Hq, int Hkv, float scale) {
  using A = F32Attn<D>;
  constexpr int R = A::kRows, LD = A::kLd;
  __shared__ __align__(16) float qs[R * LD];
  __shared__ __align__(16) float gs[R * LD];
  __shared__ __align__(16) float ls[R];
  __shared__ __align__(16) float dls[R];
  const TileId id = tile_id((N + 63) / 64, false);
  const int hk = id.row % Hkv, b = id.row / Hkv, G = Hq / Hkv;
  const size_t kh = ((size_t)b * Hkv + hk) * N;
  const int k0 = id.tile * 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int c = threadIdx.x % 16, h = (threadIdx.x % 64) / 16;
  const int ka = k0 + 16 * w, kz = min(ka + 15, N - 1), m = ka + c;
  const bool live = m < N;
  // queries end with the block of the key; a tile may straddle blocks
  const int end_a = (ka / Bs + 1) * Bs, end_z = min((kz / Bs + 1) * Bs, N), end = min((m / Bs + 1) * Bs, N);
  const int qend = min((min(k0 + 63, N - 1) / Bs + 1) * Bs, N);
  float k[D / 4], v[D / 4];
  load_col<D>(K + kh * D, m, live, h, 1.f, k);
  load_col<D>(V + kh * D, m, live, h, 1.f, v);
  f32x4_t ak[A::kAcc], av[A::kAcc];
#pragma unroll
  for (int i = 0; i < A::kAcc; ++i) ak[i] = av[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int gh = 0; gh < G; ++gh) {
    const size_t qh = ((size_t)b * Hq + (size_t)hk * G + gh) * N;
    float4 qr[4], gr[4];
    float lr = 0.f, dr = 0.f;
    const int lrow = threadIdx.x % R;
    if constexpr (D == 64) {  // the next rows are in flight while these are used; at D = 128 the registers are the operands'
      fetch_rows<D>(Q + qh * D, k0, N, qr);
      fetch_rows<D>(dO + qh * D, k0, N, gr);
    }
    lr = LSE[qh + min(k0 + lrow, N - 1)];
    dr = delta[qh + min(k0 + lrow, N - 1)];
    for (int q0 = k0; q0 < qend; q0 += R) {
      __syncthreads();
      if constexpr (D != 64) {
        fetch_rows<D>(Q + qh * D, q0, N, qr);
        fetch_rows<D>(dO + qh * D, q0, N, gr);
      }
      commit_rows<D>(qs, qr, q0, N, scale);
      commit_rows<D>(gs, gr, q0, N, 1.f);
      if (threadIdx.x < R) {
        ls[threadIdx.x] = lr;
        dls[threadIdx.x] = dr;
      }
      __syncthreads();
      if constexpr (D == 64) {
        fetch_rows<D>(Q + qh * D, q0 + R, N, qr);
        fetch_rows<D>(dO + qh * D, q0 + R, N, gr);
      }
      lr = LSE[qh + min(q0 + R + lrow, N - 1)];
      dr = delta[qh + min(q0 + R + lrow, N - 1)];
#pragma unroll
      for (int j = 0; j < A::kSub; ++j) {
        const int qj = q0 + 16 * j;
        if (!(ka < N && qj + 15 >= ka && qj < end_z)) continue;
        const bool masked = qj < kz || qj + 15 >= end_a || qj + 15 >= N;
        f32x4_t p = dot_tile<D>(qs + 16 * j * LD, k, c, h);
        f32x4_t ds = dot_tile<D>(gs + 16 * j * LD, v, c, h);
        const float4 l4 = *reinterpret_cast<const float4*>(ls + 16 * j + 4 * h);
        const float4 d4 = *reinterpret_cast<const float4*>(dls + 16 * j + 4 * h);
        const float la[4] = {l4.x, l4.y, l4.z, l4.w}, da[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int n = qj + 4 * h + t;
          p[t] = __expf(p[t] - la[t]);
          ds[t] = p[t] * (ds[t] - da[t]);
          if (masked && (!live || n < m || n >= end)) p[t] = ds[t] = 0.f;
        }
        const auto attends = [&](int r) { return qj + r >= m && qj + r < end; };
        add_tile<D>(av, gs + 16 * j * LD, p, c, h, masked, attends);
        add_tile<D>(ak, qs + 16 * j * LD, ds, c, h, masked, attends);
      }
    }
  }
  if (!live) return;
  store_col<D>(ak, dK + (kh + m) * D, h, 1.f);
  store_col<D>(av, dV + (kh + m) * D, h, 1.f);
}

}  // namespace

int muse_launch_attn_fwd_f32(const MuseDims& d, int Bs, const float* Q, const float* K, const float* V, const float* ff,
                             float* O, float* LSE, hipStream_t st) {
  const dim3 g((unsigned)(((d.N + 63) / 64) * d.Hq * d.B));
  MuseProf prof_("k_attn_fwd_f32", st);
  if (d.D == 64)
    hipLaunchKernelGGL((k_attn_fwd_f32<64>), g, dim3(256), 0, st, Q, K, V, ff, O, LSE, d.N, Bs, d.Hq, d.Hkv, d.B, d.scale);
  else
    hipLaunchKernelGGL((k_attn_fwd_f32<128>), g, dim3(256), 0, st, Q, K, V, ff, O, LSE, d.N, Bs, d.Hq, d.Hkv, d.B, d.scale);
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}

int muse_launch_attn_bwd_f32(const MuseDims& d, int Bs, const float* Q, const float* K, const float* V, const float* dO,
                             const float* LSE, const float* delta, float* dQ, float* dK, float* dV, hipStream_t st) {
  const unsigned tiles = (unsigned)((d.N + 63) / 64) * d.B;
  const dim3 gq(tiles * d.Hq), gk(tiles * d.Hkv);
  if (d.D == 64) {
    { MuseProf prof_("k_attn_bwd_dq_f32", st); hipLaunchKernelGGL((k_attn_bwd_dq_f32<64>), gq, dim3(256), 0, st, Q, K, V, dO, LSE, delta, dQ, d.N, Bs, d.Hq, d.Hkv, d.scale); }
    { MuseProf prof_("k_attn_bwd_dkv_f32", st); hipLaunchKernelGGL((k_attn_bwd_dkv_f32<64>), gk, dim3(256), 0, st, Q, K, V, dO, LSE, delta, dK, dV, d.N, Bs, d.Hq, d.Hkv, d.scale); }
  } else {
    { MuseProf prof_("k_attn_bwd_dq_f32", st); hipLaunchKernelGGL((k_attn_bwd_dq_f32<128>), gq, dim3(256), 0, st, Q, K, V, dO, LSE, delta, dQ, d.N, Bs, d.Hq, d.Hkv, d.scale); }
    { MuseProf prof_("k_attn_bwd_dkv_f32", st); hipLaunchKernelGGL((k_attn_bwd_dkv_f32<128>), gk, dim3(256), 0, st, Q, K, V, dO, LSE, delta, dK, dV, d.N, Bs, d.Hq, d.Hkv, d.scale); }
  }
  MUSE_LAUNCH_CHECK();
  return MUSE_OK;
}
