// lg_f32.h — building blocks of the float32 kernels: 64-row float32 tiles in LDS and the float32 matrix
// instruction they feed (v_mfma_f32_16x16x4_f32: IEEE float32 products and sums, twice the rate of plain vector
// multiply-adds and one LDS operand per 32 cycles instead of one per multiply-add).
//
// Instruction layout (lane = 16 h + n, h = 0..3, n = 0..15):
//   A operand (16 x 4): lane holds row n, contraction slot h      B operand (4 x 16): lane holds column n, slot h
//   C/D (16 x 16): register r (0..3) of a lane is row 4 h + r, column n
// Which index a slot stands for is free as long as both operands agree:
//   contraction over dims       slot h of step (c, t) = dim 16 c + 4 h + t: a lane reads one float4 of its row per
//                               four instructions
//   contraction over tile rows  slot h of step r = row 4 h + r: register r of an accumulator whose rows are the
//                               tile's rows IS the B operand, no exchange between lanes
//
// A tile is 64 (dk/dv at head dim 128: 32) rows x D floats, row-major, its 16-byte chunks XOR-swizzled: chunk c of row r sits at c ^ (r & 15).
// Row reads (16 rows x one chunk each) and column reads (4 rows 4 apart x 16 consecutive floats) then both touch
// all 64 banks once.
#ifndef LG_F32_H_
#define LG_F32_H_

#include "lg_mask.h"
#include "lg_swz.h"

template <int D, int ROWS_ = 64>
struct LgF32Tile {
  static constexpr int ROWS = ROWS_;
  static constexpr int CPR = D / 4;
  static constexpr int ROW_BYTES = D * 4;
  static constexpr int BYTES = ROWS * ROW_BYTES;
  __device__ __forceinline__ static int pi(int r) { return r & 15; }
};

__device__ __forceinline__ f32x4_t lg_mfma16(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D>
struct LgF32Reader {
  using T = LgF32Tile<D>;
  int rbase, cbase;
  __device__ __forceinline__ void init(int n, int h) {
    rbase = n * T::ROW_BYTES + ((h ^ n) << 4);
    cbase = 4 * h * T::ROW_BYTES + (h << 6) + ((n >> 2) << 4) + (n & 3) * 4;
  }
  // row 16 rb + n, dims 16 c + 4 h .. + 3; tile = byte offset of the tile (a multiple of 1024)
  __device__ __forceinline__ float4 row4(const unsigned char* smem, int tile, int rb, int c) const {
    return *reinterpret_cast<const float4*>(smem + (((rbase + tile) ^ (c << 6)) + rb * 16 * T::ROW_BYTES));
  }
  // row 16 rb + 4 h + r, dim 16 db + n
  __device__ __forceinline__ float col(const unsigned char* smem, int tile, int rb, int r, int db) const {
    return *reinterpret_cast<const float*>(smem + (((cbase + tile) ^ ((db << 6) | (r << 4))) +
                                                   (rb * 16 + r) * T::ROW_BYTES));
  }
};

// The live keys of a lane's query row: bit 4 x + r is key k0 + 16 x + 4 h + r, as the accumulators of two 16-key blocks
// hold them.  (Element by element, with the pattern's divisions and a branch each:
// 1 head of 64, 128 tokens, forward 6.7 us, so 6.2; 2 x 8 heads, 1024 tokens, window 128 14.6, 14.0, backward 45.2, 44.5.)
struct LgF32Row {
  int i, w;  // the row, the first key of its window
  __device__ __forceinline__ void init(const LgMask& m, int row) {
    i = min(row, m.N - 1);
    w = (lg_div_b(m, i) - m.wb + 1) * m.b;
  }
  __device__ __forceinline__ uint32_t bits(const LgMask& m, int k0, int h) const {
    const uint32_t all = lg_row_key_bits(m, i, w, k0, m.stride > 0 ? lg_strided_bits(m, k0) : 0u) >> (4 * h);
    return (all & 0xfu) | ((all >> 12) & 0xf0u);
  }
};

// Sum over the four lanes that hold one column (lanes n, n + 16, n + 32, n + 48); every one receives it.
__device__ __forceinline__ float lg_col_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + lg_other_half(x);
}
__device__ __forceinline__ float lg_col_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, lg_other_half(x));
}

#endif  // LG_F32_H_
