// What the bf16 flash kernels share: the numbering of their workgroups.
#pragma once
#include "common.h"

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Numbering of the flash kernels' workgroups.  The tiles of 128 rows of one (batch, head, spatial block) group
// stream the same keys and values (forward, dQ) or queries (dK/dV); workgroups go to the 8 XCDs round-robin by
// their linear id, so with a grid of (8 tpg, ceil(groups / 8)) the workgroup (x, y) is on XCD x % 8 and takes
// tile x / 8 of group 8 y + x % 8: a group's tiles run on one XCD, one after the other, and its operand rows
// stay in that XCD's L2 instead of being fetched by all eight.  tpg = tiles per group (a block, or the whole
// sequence when the block size is not a multiple of 128).
struct FlashTile {
  int t, blk, tpg, h, b;  // tile inside the group, block of the group, tiles per group, head, batch
  bool ok;
};
template <int TR = 128>  // rows of a workgroup's tile
__device__ __forceinline__ FlashTile flash_tile(int N, int Bs, int H, int nbatch) {
  FlashTile r;
  const bool al = (Bs % TR) == 0;
  r.tpg = al ? Bs / TR : (N + TR - 1) / TR;
  const int nblk = al ? N / Bs : 1;
  const int g = blockIdx.y * 8 + blockIdx.x % 8;
  r.t = blockIdx.x / 8;
  r.ok = g < nbatch * H * nblk;
  r.blk = g % nblk;
  r.h = (g / nblk) % H;
  r.b = g / nblk / H;
  return r;
}
static inline dim3 flash_grid(int N, int Bs, int H, int nbatch, int TR = 128) {
  const bool al = (Bs % TR) == 0;
  const int tpg = al ? Bs / TR : (N + TR - 1) / TR, nblk = al ? N / Bs : 1;
  return dim3(8 * tpg, (nbatch * H * nblk + 7) / 8, 1);
}
