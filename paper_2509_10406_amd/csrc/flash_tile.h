// What the bf16 flash kernels share: the numbering of their workgroups.
#pragma once
#include "common.h"

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Numbering of the flash kernels' workgroups.  The tiles of one (batch, head, spatial block) group stream the same keys and
// values (forward, dQ) or queries (dK/dV); workgroups go to the 8 XCDs round-robin by their linear id, so with a grid of
// (8 tiles, ceil(groups / 8)) the workgroup (x, y) is on XCD x % 8 and has number x / 8 in group 8 y + x % 8: a group's
// workgroups run on one XCD, one after the other, and its operand rows stay in that XCD's L2 instead of being fetched by all
// eight.  More than 65535 rows of the grid continue in z.
struct FlashTile {
  int t, blk, tpg, h, b;  // number inside the group, block of the group, tiles per group, head, batch
  bool ok;
};
// chunk > 1: the workgroups of an XCD do not take its groups one by one but `chunk` at a time, all first workgroups before all
// second ones (`tiles` = workgroups per group).
__device__ __forceinline__ FlashTile flash_tile_of(int tpg, int nblk, int H, int nbatch, int tiles = 1, int chunk = 1) {
  FlashTile r;
  r.tpg = tpg;
  const int groups = nbatch * H * nblk, y = blockIdx.z * gridDim.y + blockIdx.y, xcd = blockIdx.x % 8;
  int g = 8 * y + xcd;
  r.t = blockIdx.x / 8;
  if (chunk > 1) {
    const int seq = y * tiles + r.t, first = seq / (tiles * chunk) * chunk, rem = seq - first * tiles;
    const int n = max(min(chunk, (groups + 7) / 8 - first), 1);  // the last chunk is narrower
    r.t = rem / n;
    g = 8 * (first + rem % n) + xcd;
  }
  r.ok = g < groups && r.t < tpg;
  r.blk = g % nblk;
  r.h = (g / nblk) % H;
  r.b = g / nblk / H;
  return r;
}
static inline dim3 flash_grid_of(int tiles, int groups) {
  const int y = (groups + 7) / 8, most = 65535;
  return dim3(8 * tiles, y < most ? y : most, (y + most - 1) / most);
}
// `chunk`: as many groups of an XCD as have 8 MB of keys and values (or queries and their gradients), measured in attn_fwd.hip
static inline int chunk_groups(int Bs, int D, int groups) {
  const int fit = (8 << 20) / (4 * D) / Bs, all = (groups + 7) / 8;
  return fit < 1 ? 1 : fit < all ? fit : all;
}

// The backward kernels' tiles of 128 rows: of a block, or of the whole sequence when the block size is not a multiple of 128.
__device__ __forceinline__ FlashTile flash_tile(int N, int Bs, int H, int nbatch) {
  const bool al = (Bs % 128) == 0;
  return flash_tile_of(al ? Bs / 128 : (N + 127) / 128, al ? N / Bs : 1, H, nbatch);
}
static inline dim3 flash_grid(int N, int Bs, int H, int nbatch) {
  const bool al = (Bs % 128) == 0;
  return flash_grid_of(al ? Bs / 128 : (N + 127) / 128, nbatch * H * (al ? N / Bs : 1));
}
