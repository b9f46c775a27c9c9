// What the 32x32x16 attention kernels use beside tile_common.h: the MFMA
// wrapper and the LDS tile layout that its operands read without bank
// conflicts.
//
// MFMA register layout (v_mfma_f32_32x32x16_bf16, wave64):
//   A[i][k] : lane l holds row i = l%32 and 8 k-values in "k-slots"
//   B[k][j] : lane l holds col j = l%32 and 8 k-values in the same k-slots
//   C[i][j] : lane l holds col j = l%32, rows i = 8*(v/4) + 4*(l/32) + v%4,
//             v = 0..15
// Chained products: for a 16-wide k-block kb, slot e of lane-half g = l/32
// holds k = 16*kb + 8*(e/4) + 4*g + e%4, which is exactly where rows 16*kb.. of
// a C tile live (v = 8*(kb%2) + e).  A natural-layout operand (k contiguous in
// memory) uses the plain map k = 16*kk + 8*g + e.
#pragma once

#include "tile_common.h"

namespace sppo {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mfma32(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// A bf16 tile [rows][D], unpadded, the 16-byte chunk c of row r at physical
// chunk c ^ f(r): natural reads (16 consecutive rows at one chunk) hit 16
// different slots of the 256-byte bank window (D = 64: two rows a window, f
// bijective per row parity), and the 4 rows x 4 chunks of 32 lanes of a
// transposed read four different 64-byte quarters.
template <int D>
struct Tile32 {
  static constexpr int P = D;         // row pitch, elements
  static constexpr int CG = D / 8;    // 16-byte chunks per row
  static constexpr int RPI = 512 / D; // rows per LDS-DMA wave instruction
  static __device__ __forceinline__ int f(int r) {
    if constexpr (D == 128) {
      return ((r & 3) << 2) | ((r >> 2) & 3);
    } else {
      return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
    }
  }
  // Natural operand read of k-step kk for rows rb + l%32 (rb % 32 == 0):
  // element offset (add rb * P).
  static __device__ __forceinline__ int nat(int lane, int kk) {
    const int l32 = lane & 31, g = lane >> 5;
    return l32 * P + 8 * ((2 * kk + g) ^ f(l32));
  }
  // Transposed read of rows k0 + {0..7} (hi = 0) or k0 + {8..15} (hi = 1),
  // columns 32 db..32 db+31 (add k0 * P, k0 % 16 == 0).  Source lane
  // s = 16q + 4e + a supplies the 8 bytes at row 4(q/2) + e, columns
  // 16(q%2) + 4a of the 16x32 block; ds_read_b64_tr_b16 hands output lane
  // 16q + 4a' + b element b of source lanes 16q + 4e + a', e = 0..3.
  static __device__ __forceinline__ int tr(int lane, int db, int hi) {
    const int q = lane >> 4, e = (lane >> 2) & 3, a = lane & 3;
    const int row = 4 * (q >> 1) + e + 8 * hi;
    const int c = 4 * db + 2 * (q & 1) + (a >> 1);
    return row * P + 8 * (c ^ f(row)) + 4 * (a & 1);
  }
  // Byte offset, relative to the first row of a tile in global memory, of
  // the chunk lane `lane` fetches in LDS-DMA instruction u of the tile.
  static __device__ __forceinline__ int dma(int lane, int u, int64_t row_stride) {
    const int row = RPI * u + lane / CG, p = lane % CG;
    return (int)((row * row_stride + 8 * (p ^ f(row))) * (int64_t)sizeof(uint16_t));
  }
};

}  // namespace sppo
