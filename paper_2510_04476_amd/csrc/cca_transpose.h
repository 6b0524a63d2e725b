// The transposes of the projection weights, as a workgroup's work: launched alone (cca_gemm.hip) or with the prologue's set-up
// (cca_prologue.hip).
#pragma once

#include "cca_internal.h"

namespace cca {

struct TransposeTile {
  alignas(16) bf16_t at[64][72];  // [source column][source row], rows of 144 bytes
};

// Workgroups [0, n1) serve the first matrix, the rest the second.  256 threads, 64 x 64 tiles; both sizes are multiples of 8
// (checked by the launcher) and a thread moves 16 bytes per memory access (the tile is transposed element by element on its
// way into LDS).
__device__ __forceinline__ void transpose_block(const TransposePair &p, int block, TransposeTile &tile) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const bool second = block >= p.n1;
  const bf16_t *src = second ? p.src2 : p.src1;
  bf16_t *dst = second ? p.dst2 : p.dst1;
  const int rows = second ? p.rows2 : p.rows1, cols = second ? p.cols2 : p.cols1;
  const int id = second ? block - p.n1 : block, tiles_c = (cols + 63) / 64;
  const int c0 = (id % tiles_c) * 64, r0 = (id / tiles_c) * 64;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ch = threadIdx.x + i * 256, r = ch >> 3, c = (ch & 7) * 8;  // chunk of 8 columns of source row r0 + r
    u4 v = {0, 0, 0, 0};
    if (r0 + r < rows && c0 + c < cols) v = *reinterpret_cast<const u4 *>(src + (long long)(r0 + r) * cols + c0 + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile.at[c + 2 * e][r] = (bf16_t)(v[e] & 0xffffu);
      tile.at[c + 2 * e + 1][r] = (bf16_t)(v[e] >> 16);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ch = threadIdx.x + i * 256, c = ch >> 3, r = (ch & 7) * 8;  // 8 source rows of source column c0 + c
    if (c0 + c < cols && r0 + r < rows)
      *reinterpret_cast<u4 *>(dst + (long long)(c0 + c) * rows + r0 + r) = *reinterpret_cast<const u4 *>(&tile.at[c][r]);
  }
}

}  // namespace cca
