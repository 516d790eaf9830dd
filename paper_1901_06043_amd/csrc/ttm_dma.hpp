// Index maps of the LDS chunk images used by the FP64 mode-product kernel
// (ttm_dma.hip).  Host and device code: the kernel uses them to place and
// read elements; a host build can replay the same maps.
//
// Z_(n) = M Y_(n) is computed in tiles of 128 output rows k by 128 columns c
// of the unfolding, over chunks of 16 reduction indices j.  Per chunk each
// operand is held in LDS as an image of 128 "rows" (k for M, c for Y) by 16
// j, in 16-byte units (E = 16 / sizeof(T) elements per unit), in one of two
// forms:
//   row form: 16 j per row (128 bytes of doubles, 64 of floats); unit u (j =
//     E u .. E u + E - 1) of row r stored at unit position u ^ ((r >> 1) & 7)
//     (doubles) or u ^ ((r >> 2) & 3) (floats);
//   column form: per j, the 128 rows' elements (128 sizeof(T) bytes); unit u
//     (rows E u .. E u + E - 1) of column j stored at u ^ sw(j).
// The reduction index of MFMA step s (of 4) in lane group q is
// j(s, q) = 2 q + (s & 1) + 8 (s >> 1), the same for both operands: in the
// row form a lane then reads two consecutive values for two steps (doubles:
// the 16-byte unit q, then q | 4; floats: half a unit), and in the column form the swizzle sw(j) = ((j >> 1) & 1) << 3
// (doubles) or ((j >> 1) & 3) << 2 (floats) depends on q only, so that the
// four lane groups read distinct banks and a step moves by a fixed offset.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace tk {
namespace tdma {

constexpr int kRows = 128;  // rows of an image (output rows or columns of a tile)
constexpr int kJC = 16;     // reduction indices per chunk

template <int FORM, int ES>
struct TImg {
  static constexpr int E = 16 / ES;
  static constexpr int RB = kJC * ES;             // row form: bytes per row
  static constexpr int BYTES = kRows * kJC * ES;  // 16 KB (doubles) or 8 KB (floats)
  static constexpr int CB = kRows * ES;           // column form: bytes per j

  __host__ __device__ static constexpr int sw(int j) { return ES == 8 ? (((j >> 1) & 1) << 3) : (((j >> 1) & 3) << 2); }

  // Reduction index of MFMA step s in lane group q.
  __host__ __device__ static constexpr int jstep(int s, int q) { return 2 * q + (s & 1) + 8 * (s >> 1); }

  // Row form: the swizzle of row r's units.
  __host__ __device__ static constexpr int rsw(int r) { return ES == 8 ? ((r >> 1) & 7) : ((r >> 2) & 3); }

  // Byte offset of element (row r, reduction index j).
  __host__ __device__ static int at(int r, int j) {
    if (FORM == 0) return r * RB + (((j / E) ^ rsw(r)) << 4) + (j % E) * ES;
    return j * CB + (((r / E) ^ sw(j)) << 4) + (r % E) * ES;
  }

  // The first element (row r, index j) of the unit that lane `lane` of
  // instruction jj (covering bytes [1024 jj, 1024 jj + 1024)) loads.
  __host__ __device__ static void unit_of(int jj, int lane, int& r, int& j) {
    const int P = jj * 1024 + lane * 16;
    if (FORM == 0) {
      r = P / RB;
      j = (((P % RB) >> 4) ^ rsw(r)) * E;
    } else {
      j = P / CB;
      r = ((((P % CB) >> 4) ^ sw(j))) * E;
    }
  }
};

}  // namespace tdma
}  // namespace tk
