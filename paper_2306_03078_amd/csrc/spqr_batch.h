// What the matrix-core products of all batch sizes share: the part of a tile a lane holds when 16 lanes hold the same
// tile column of 16 strips, and its dequantisation into operands of v_mfma_f32_16x16x32_f16.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spqr_tile.h"

namespace spqr {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kUnitTiles = 16;               // tile columns of a unit of the split: one step of 4 for each of 4 wavefronts
// Rows a lane multiplies: its tile's 8 or 16; a tile of 32 rows is taken as two of 16 (128 accumulators a lane spill), so
// that the strips of the kernel are 8 or 16 rows in every format.
constexpr int lane_rows(int tile_rows) { return tile_rows == 32 ? 16 : tile_rows; }

// What a lane holds of its tile: the codes of its LR rows (one of TR / LR parts of the tile) and the tile's statistics.
template <int W, int TR, int TC, int AXIS, int LR = lane_rows(TR)> struct BatchTile {
  using T = TileRegs<W, TR, TC, AXIS>;
  static constexpr int DW = 4 * T::KW * LR / TR;              // dwords of codes: whole 16-byte words, or one and a half
  uint32_t c[DW];
  uint32_t s[T::SD];
};

// `blk` and L (the block and its tiles) are uniform, `l` is the lane's tile in it, `off` the lane's strip's byte offset,
// `part` (tiles of more than LR rows) which rows.
template <int W, int TR, int TC, int AXIS, int LR>
__device__ __forceinline__ void load_batch_tile(BatchTile<W, TR, TC, AXIS, LR>& t, const uint8_t* blk, int L, uint32_t off,
                                                uint32_t l, int part) {
  using B = BatchTile<W, TR, TC, AXIS, LR>;
  using T = typename B::T;
  const uint32_t off16 = off + 16u * l, off4 = off + 4u * l;
  const uint8_t* sb = blk + 16 * T::KW * L;
#pragma unroll
  for (int k = 0; k < T::SWF; ++k) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(sb + 16 * k * L + off16);
    t.s[4 * k] = v.x; t.s[4 * k + 1] = v.y; t.s[4 * k + 2] = v.z; t.s[4 * k + 3] = v.w;
  }
  const uint8_t* rb = sb + 16 * T::SWF * L;
#pragma unroll
  for (int k = 0; k < T::SR; ++k) t.s[4 * T::SWF + k] = *reinterpret_cast<const uint32_t*>(rb + 4 * k * L + off4);
  if constexpr (B::DW % 4 == 0) {
    const uint32_t offc = TR == LR ? off16 : off16 + (uint32_t)part * (4u * B::DW) * (uint32_t)L;
#pragma unroll
    for (int k = 0; k < B::DW / 4; ++k) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(blk + 16 * k * L + offc);
      t.c[4 * k] = v.x; t.c[4 * k + 1] = v.y; t.c[4 * k + 2] = v.z; t.c[4 * k + 3] = v.w;
    }
  } else {                                   // six dwords: a word and the lower half of the next, or an upper half and a word
    static_assert(B::DW == 6, "a quarter of a 3-bit tile");
    const uint32_t offc = off16 + (uint32_t)(part + (part >> 1)) * 16u * (uint32_t)L;
    const u32x4 v = *reinterpret_cast<const u32x4*>(blk + offc), w = *reinterpret_cast<const u32x4*>(blk + 16 * L + offc);
    const bool odd = part & 1;
    t.c[0] = odd ? v.z : v.x; t.c[1] = odd ? v.w : v.y; t.c[2] = odd ? w.x : v.z;
    t.c[3] = odd ? w.y : v.w; t.c[4] = odd ? w.z : w.x; t.c[5] = odd ? w.w : w.y;
  }
}

// Two binary32 numbers to a binary16 pair, to nearest even.  The fused multiply-add with a binary16 result that the compiler
// would take for (_Float16)fmaf(..) twice runs at half rate: 17 clocks a pair against 14 with one conversion of both.
__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
  uint32_t d;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(d) : "v"(lo), "v"(hi));
  return d;
}

// Dequantisation of a lane's rows, 8 columns at a time: w = s_hat * (q - z_hat) in one binary32 FMA, rounded once to
// binary16, where s_hat = s_s*(s_q - z_s) and z_hat = s_z*(z_q - z_z).  The codes of the statistics come as 1 + code/8.
// Groups along the tile's rows: the weight's code comes as 1 + q/2^W, and
//   w = fa*(1 + q/2^W) + fb with fa = 2^W*s_hat, fb = -s_hat*(2^W + z_hat), per group:
//   fa = c1*(1 + s_q/8) + c2,   -(2^W + z_hat)/2^W = e1*(1 + z_q/8) + e2,   fb = fa * that.
// Groups along the tile's columns: the code is used where it lies, as the subnormal q * 2^(bit - 24), and the power of two
// goes into the column's factor (exactly): w = fa*(q * 2^(bit - 24)) + fb with fa = s_hat * 2^(24 - bit), fb = -s_hat*z_hat.
// No shift for most codes, and no offset that would have to cancel inside the FMA: the offset 2^(7 - bit) that the batch-1
// kernel's extraction leaves is up to 128 times a weight of s_hat, and with it 8 to 11 % of the weights were not the
// nearest binary16.  So measured over 16384 weights per format none is not, with 1 + q/2^W 0.2 to 0.4 %; same time.
template <int W, int TR, int TC, int AXIS, int LR_ = lane_rows(TR)> struct Dequant {
  using B = BatchTile<W, TR, TC, AXIS, LR_>;
  using T = typename B::T;
  static constexpr int LR = LR_, NSUB = TR / LR;              // rows of a lane; strips of the kernel per strip of tiles
  static constexpr int PPR = TC / 2, KG = TC / 8;             // code pairs per row; blocks of 8 columns
  static constexpr int NG = AXIS == 1 ? TC : LR;              // first-level groups of a lane
  // The bit a code lies at (its class, see CodeClass) is a function of the pair's column, for 3-bit codes in rows of 8
  // pairs of the column and the parity of the row.
  static constexpr bool INPLACE = AXIS == 1;
  static constexpr int NK = INPLACE && W == 3 && PPR == 8 ? 2 : 1;
  static constexpr int NF = AXIS == 1 ? 8 : NG;               // groups whose constants are alive at a time
  static constexpr float SCALE = (float)(1 << W);
  PairConsts kc, k3;
  ClassConsts kk;
  int part;                                                   // which rows of a tile of more than LR
  float c1, c2, e1, e2;                                       // of the current tile
  float fa[NK][NF], fb[NF];

  __device__ __forceinline__ Dequant(int part_) : part(part_) {
    kc = make_pair_consts<W>();
    k3 = make_pair_consts<3>();
    kk = make_class_consts<W>();
  }
  // A lane without a tile of its own (live = false) gets zero weights.
  __device__ __forceinline__ void begin(const B& t, bool live) {
    const uint32_t a2 = t.s[T::SD - 2], b2 = t.s[T::SD - 1];
    const float s_s = h2f((uint16_t)(a2 & 0xFFFF)), z_s = h2f((uint16_t)(a2 >> 16));
    const float s_z = h2f((uint16_t)(b2 & 0xFFFF)), z_z = h2f((uint16_t)(b2 >> 16));
    constexpr float UP = INPLACE ? 0x1p24f : SCALE, OFFSET = INPLACE ? 0.f : SCALE;
    c1 = live ? UP * 8.f * s_s : 0.f;
    c2 = live ? UP * (-s_s * z_s - 8.f * s_s) : 0.f;
    e1 = -8.f * s_z / UP;
    e2 = -(OFFSET - s_z * z_z - 8.f * s_z) / UP;
    if constexpr (AXIS == 0) {
#pragma unroll
      for (int p = 0; p < NG / 2; ++p) group_pair(t, p, 2 * p);
    }
  }
  // The constants of columns 8j .. 8j+7 (groups along the columns; groups along the rows have theirs from begin()).
  __device__ __forceinline__ void columns(const B& t, int j) {
    if constexpr (AXIS == 1) {
#pragma unroll
      for (int d = 0; d < 4; ++d) group_pair(t, 4 * j + d, 2 * d);
    }
  }
  // Row r, columns 8j + 2d and 8j + 2d + 1: a quarter of an operand.
  __device__ __forceinline__ uint32_t pair(const B& t, int r, int j, int d) const {
    const int q = r * PPR + 4 * j + d;
    const half2_t q2 = as_half2(INPLACE ? pair_code_bits<W>(t.c, q, kk) : pair_f16<W>(t.c, q, kc));
    const int g0 = AXIS == 1 ? 2 * d : r, g1 = AXIS == 1 ? 2 * d + 1 : r;
    return pack_f16(fmaf((float)q2.x, fa[r % NK][g0], fb[g0]), fmaf((float)q2.y, fa[r % NK][g1], fb[g1]));
  }
  // Row r, columns 8j .. 8j+7 as an operand.
  __device__ __forceinline__ half8_t operand(const B& t, int r, int j) const {
    const uint32_t o[4] = {pair(t, r, j, 0), pair(t, r, j, 1), pair(t, r, j, 2), pair(t, r, j, 3)};
    return __builtin_bit_cast(half8_t, o);
  }

 private:
  __device__ __forceinline__ void group_pair(const B& t, int p, int at) {    // groups 2p and 2p + 1 of the lane
    uint32_t sp = pair_f16<3>(t.s, p, k3), zp = pair_f16<3>(t.s, T::B2 / 2 + p, k3);
    if constexpr (AXIS == 0) {                 // the groups of the lane's part of the rows
#pragma unroll
      for (int h = 1; h < NSUB; ++h) {
        sp = part == h ? pair_f16<3>(t.s, h * NG / 2 + p, k3) : sp;
        zp = part == h ? pair_f16<3>(t.s, T::B2 / 2 + h * NG / 2 + p, k3) : zp;
      }
    }
    const half2_t sq = as_half2(sp), zq = as_half2(zp);
    const float f0 = fmaf((float)sq.x, c1, c2), f1 = fmaf((float)sq.y, c1, c2);
    fb[at] = f0 * fmaf((float)zq.x, e1, e2);
    fb[at + 1] = f1 * fmaf((float)zq.y, e1, e2);
#pragma unroll
    for (int h = 0; h < NK; ++h) {             // NK == 2: even and odd rows; exact
      const float down = INPLACE ? 1.f / (float)(1 << class_bit<W>(CodeClass<W, true>::of_pair(h * PPR + p))) : 1.f;
      fa[h][at] = f0 * down;
      fa[h][at + 1] = f1 * down;
    }
  }
};

}  // namespace spqr
