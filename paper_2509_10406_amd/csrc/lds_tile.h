// Row-major bf16 tiles in LDS whose rows serve both operands of a matrix instruction: 16-byte row reads (lanes along the
// rows, contraction over the head dim) and transposed reads (contraction over the rows, ds_read_b64_tr_b16), so a tile
// is stored once, 16 bytes at a time, and needs no transposed copy.
#pragma once
#include "common.h"

typedef __attribute__((ext_vector_type(4))) short s16x4_t;

template <typename T>
__device__ __forceinline__ uint32_t lds_addr(const T* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const T*)p; }

// Four k-slots of a transposed operand straight from a row-major tile: the 16 lanes of a group name rows r0 .. r0+3
// (lane s: row r0 + s / 4, columns c0 + 4 (s % 4) ..) and each receives its own column c0 + s of the four.
__device__ __forceinline__ s16x4_t lds_tr4(const bf16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)p);
}
__device__ __forceinline__ bf16x8_t tr_join(s16x4_t a, s16x4_t b) {
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Element offset of the 16-byte chunk `chunk` of row `row` in an unpadded tile.  The chunks of a row change places by an
// xor of row bits such that both kinds of read spread over all banks: of any 16 consecutive rows the same chunk lies in
// 16 different bank groups (row reads), and of any 4 consecutive rows (aligned) four adjacent chunks do (transposed reads).
template <int D>
__device__ __forceinline__ int tile_at(int row, int chunk) {
  static_assert(D == 64 || D == 128, "head dims the kernels are built for");
  const int f = D == 64 ? (((row >> 1) & 1) << 2) | ((row >> 2) & 3) : ((row & 3) << 2) | ((row >> 2) & 3);
  return row * D + ((chunk ^ f) << 3);
}
template <int D>
__device__ __forceinline__ bf16x8_t tile_row(const bf16_t* tile, int row, int chunk) {
  return *reinterpret_cast<const bf16x8_t*>(tile + tile_at<D>(row, chunk));
}
// the lane's 4 rows x 4 columns share of a transposed read; col is a multiple of 4
template <int D>
__device__ __forceinline__ s16x4_t tile_tr4(const bf16_t* tile, int row, int col) {
  return lds_tr4(tile + tile_at<D>(row, col >> 3) + (col & 4));
}
// transposed operand of a 32x32x16 instruction: columns 32 t .. of the 16 rows from r0, k-slots in accumulator order
template <int D>
__device__ __forceinline__ bf16x8_t tile_cols(const bf16_t* tile, int r0, int t, int lane) {
  const int row = r0 + 4 * (lane / 32) + (lane % 16) / 4, col = 32 * t + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
  return tr_join(tile_tr4<D>(tile, row, col), tile_tr4<D>(tile, row + 8, col));
}

// 16 bytes of every lane from base + off to LDS at at + 16 lane.  Written out, because behind the builtin the compiler lets every
// LDS read wait for the rows; they are waited for by count (the caller's s_waitcnt vmcnt).  m0 is reserved and cannot be named as
// clobbered; nothing else in the kernels that use this does (tests/test_attn_bwd_code.py and tests/test_farfield_code.py look
// through the machine code for that).
__device__ __forceinline__ void rows_to_lds(uint32_t at, uint32_t off, const bf16_t* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(at), "v"(off), "s"(base) : "memory");
}
// the same with 4 bytes of every lane, to at + 4 lane
__device__ __forceinline__ void words_to_lds(uint32_t at, uint32_t off, const float* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(at), "v"(off), "s"(base) : "memory");
}
