// Tiles of 16-bit rows in LDS that serve as both operands of the 32x32x16
// MFMA (gfx950): the row operand (a lane reads 16 bytes of its own row) and the
// transposed operand (a lane needs a column across rows), from one row-major
// copy.  A row is a run of 16-byte chunks; its pitch is 16 or 48 banks modulo
// the 64 LDS banks, and chunk c of row r is stored at chunk c ^ ((r / 4) % 4):
// both reads are then free of bank conflicts.
#pragma once

#include "sfa_device.h"

namespace sfa {
namespace {

// Byte offset of 16-bit column `col` of row r in a tile of row pitch RB.
template <int RB>
__device__ __forceinline__ int img_pos(int r, int col) {
  return r * RB + 16 * ((col >> 3) ^ ((r >> 2) & 3)) + 2 * (col & 7);
}

// Per-lane byte offsets into a tile image of row pitch RB (a multiple
// of 16).
//   Row operand (B of 32x32x16): lane (l32, hh) reads row l32, columns
//   8 (c0 + 2 kb + hh) .. + 7 for a chunk c0 that is a multiple of 4:
//   row[kb & 1] + 16 (c0 + 4 (kb / 2)).
//   Transposed operand (A of 32x32x16, the image's rows as its k index in
//   the order of the MFMA output layout): lane (l32, hh) needs columns
//   8 c0 + l32 of rows 16 kk + 4 hh + (0..3) and 16 kk + 4 hh + 8 + (0..3).
//   A transposing read hands lane i of a 16-lane group element i % 4 of
//   the 8 bytes addressed by lane 4 e + i / 4 of the group, as its element
//   e; so lane j of group g addresses row 4 hh + j / 4 (+ 8), columns
//   8 c0 + 16 (g % 2) + 4 (j % 4) + (0..3): tr[0] / tr[1] + (16 kk) RB + 16 c0.
template <int RB>
struct LaneOff {
  int row[2], tr[2];
  __device__ __forceinline__ explicit LaneOff(int lane) {
    const int l32 = lane & 31, hh = lane >> 5, g = lane >> 4, j = lane & 15;
    row[0] = l32 * RB + 16 * (hh ^ ((l32 >> 2) & 3));
    row[1] = row[0] ^ 32;
    tr[0] = (4 * hh + (j >> 2)) * RB + 8 * (j & 1) + 16 * ((2 * (g & 1) + ((j >> 1) & 1)) ^ hh);
    tr[1] = (tr[0] ^ 32) + 8 * RB;
  }
};

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ i16x4 lds_read_tr(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p));
}

// Transposed operand of 32 columns from chunk c0 on, rows from 16 kk on.
template <int RB>
__device__ __forceinline__ bf16x8 tr_operand(const unsigned char* img, const LaneOff<RB>& o, int kk,
                                             int c0) {
  const int off = 16 * kk * RB + 16 * c0;
  const i16x4 a = lds_read_tr(img + o.tr[0] + off);
  const i16x4 b = lds_read_tr(img + o.tr[1] + off);
  const u32x2 x = __builtin_bit_cast(u32x2, a), y = __builtin_bit_cast(u32x2, b);
  const u32x4 w = {x.x, x.y, y.x, y.y};
  return __builtin_bit_cast(bf16x8, w);
}

// Row operand: chunk c0 + 2 kb + hh of the lane's row.
template <int RB>
__device__ __forceinline__ bf16x8 row_operand(const unsigned char* img, const LaneOff<RB>& o, int kb,
                                              int c0) {
  return *(const bf16x8*)(img + o.row[kb & 1] + 16 * (c0 + 4 * (kb >> 1)));
}

// The same split for two values at once, packed: word 0 holds the high
// pieces of (x0, x1), word 1 the low pieces; the rounding to nearest-even is
// the hardware conversion (v_cvt_pk_bf16_f32), identical to split2 for
// finite values.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split2_pair(float x0, float x1, uint32_t& hw, uint32_t& lw) {
  const f32x2 v = {x0, x1};
  hw = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  const f32x2 r = {x0 - __uint_as_float(hw << 16), x1 - __uint_as_float(hw & 0xffff0000u)};
  lw = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
}

}  // namespace
}  // namespace sfa
