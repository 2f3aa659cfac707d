// Device helpers shared by the sq_gemm kernels (gfx950).
#pragma once
#include "sq_device.h"

namespace sq {
namespace gemm {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Byte offset of 16-byte chunk c of a row inside an operand tile.
__device__ __forceinline__ int off4(int row, int c) { return (row << 6) + (((c ^ (row >> 2)) & 3) << 4); }   // 4 chunks / row
__device__ __forceinline__ int off8(int row, int c) { return (row << 7) + (((c ^ (row >> 1)) & 7) << 4); }   // 8 chunks / row

// 16 zero bytes in device memory: the source of operand chunks that lie past the end of K.
__device__ __attribute__((aligned(16))) const unsigned int kZeroChunk[4] = {0u, 0u, 0u, 0u};

// Half s (0/1) of a packed chunk (16 of its 32 INT4 codes) -> the INT8 operand of matrix instruction s.
__device__ __forceinline__ v4i widen(const v4u p, int s) {
  const unsigned a = p[2 * s], b = p[2 * s + 1];
  return v4i{static_cast<int>((a << 4) & 0xF0F0F0F0u), static_cast<int>(a & 0xF0F0F0F0u),
             static_cast<int>((b << 4) & 0xF0F0F0F0u), static_cast<int>(b & 0xF0F0F0F0u)};
}

// fp32 -> bf16, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t bf16_rne(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }

// Maps the linear workgroup id to a tile so that (a) the workgroups resident on one XCD at a time
// (ids congruent mod 8 go to the same XCD) cover a compact 4 x 8 patch of tiles and share operand
// tiles in that XCD's L2, and (b) every XCD walks its own contiguous range of the tile order.
__device__ __forceinline__ void tile_of_block(int id, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int per_xcd = (total + 7) / 8;
  const int lin = (id & 7) * per_xcd + (id >> 3);  // position in the tile order
  if (lin >= total) {  // the grid is rounded up to a multiple of 8: the overhang does nothing
    tm = -1;
    tn = -1;
    return;
  }
  constexpr int BAND = 4;  // tile rows walked together
  const int band = lin / (BAND * tiles_n);
  const int within = lin - band * (BAND * tiles_n);
  const int rows_here = min(BAND, tiles_m - band * BAND);
  tn = within / rows_here;
  tm = band * BAND + within - tn * rows_here;
}

}  // namespace gemm
}  // namespace sq
