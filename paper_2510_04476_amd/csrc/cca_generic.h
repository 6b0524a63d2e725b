// Pieces shared by the shape-generic kernels (cca_generic.hip, cca_generic_bwd.hip): products of fp32 values on the matrix
// cores with v_mfma_f32_32x32x2_f32, operands straight from memory (any storage type, converted on the way).
//
// One such MFMA adds, for a 32 x 32 tile D[row][col], two terms of the contraction: lane (l32, half) supplies term `half`
// of row l32 (first operand) and of column l32 (second).  Which two terms meet is free, so the contraction is walked 8 at a
// time and lane half h takes terms 4 h + i of MFMA i: four adjacent values, one 16-byte load where the operand is stored
// along the contraction.  The result sits as D[8 (r / 4) + 4 half + r % 4][l32] in register r - which is also that order, so
// a tile of results is the second operand of the next product as it stands.
#pragma once

#include "cca_internal.h"

namespace cca {

typedef float gen_f32x16 __attribute__((ext_vector_type(16)));
typedef float gen_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t gen_u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ gen_f32x4 load4(const float *p) { return *reinterpret_cast<const gen_f32x4 *>(p); }
__device__ __forceinline__ gen_f32x4 load4(const bf16_t *p) {
  const gen_u32x2 w = *reinterpret_cast<const gen_u32x2 *>(p);
  return gen_f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                   __uint_as_float(w.y & 0xffff0000u)};
}
__device__ __forceinline__ gen_f32x16 zero16() {
  gen_f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
__device__ __forceinline__ int tile_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// acc += rows . cols over `dh` channels (a multiple of 4): row l32 of the tile at `rows` (this lane's row), column l32 in LDS
// at `cols`, zero from dh up to DHM.
template <int DHM, typename T, typename F>
__device__ __forceinline__ gen_f32x16 dot_tile(const T *rows, const float *cols, int dh, int half, F &&map) {
  gen_f32x16 acc = zero16();
#pragma unroll 4
  for (int c = 0; c < DHM; c += 8) {
    const int ch = c + 4 * half;
    gen_f32x4 a = load4(rows + (ch < dh ? ch : 0));
    const gen_f32x4 b = load4(cols + ch);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ch < dh ? map(a[i]) : 0.f, b[i], acc, 0, 0, 0);
  }
  return acc;
}

// acc[dt][.] (rows: channels 32 dt + ..., column: this lane's) += sum over the 32 rows x of X[x][channel] w[x][column], w in
// the register order of a tile.  `row(x)`: pointer to row x (always readable).  `mixed`: some weights are zero because the
// pair is masked, and a masked row must not count even where it holds an infinity or NaN (0 * inf): then, and only if such
// a value is there, the sum runs on the vector ALU and skips zero weights.
template <int DT, typename T, typename Row>
__device__ __forceinline__ void add_outer(gen_f32x16 (&acc)[DT], const float (&w)[16], Row &&row, int dh, int lane, bool mixed) {
  const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const int ch = 32 * dt + l32;
    float x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = load_f(static_cast<const T *>(row(tile_row(r, half))) + (ch < dh ? ch : 0));
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      x[r] = ch < dh ? x[r] : 0.f;
      bad |= !(fabsf(x[r]) < INFINITY);
    }
    if (mixed && __any(bad)) {
#pragma unroll 1
      for (int k = 0; k < 32; ++k) {
        float wk = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float o = __shfl(w[r], l32 + 32 * ((k >> 2) & 1));
          wk = r == (k >> 3) * 4 + (k & 3) ? o : wk;
        }
        const T *p = row(k);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int c = 32 * dt + tile_row(r, half);
          const float v = load_f(p + (c < dh ? c : 0));
          acc[dt][r] = wk != 0.f && c < dh ? fmaf(v, wk, acc[dt][r]) : acc[dt][r];
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[r], w[r], acc[dt], 0, 0, 0);
    }
  }
}

// 32 rows of `dh` channels -> LDS [32][DHM + 4] floats (rows padded by 16 bytes: conflict-free 16-byte reads down a column
// of rows), times `map`; rows past `last` repeat it, channels from dh on are zero.
template <int DHM, typename T, typename F>
__device__ __forceinline__ void stage_rows32(float *dst, const T *base, long long stride, int first, int last, int dh, F &&map) {
  for (int i = threadIdx.x; i < 32 * DHM; i += blockDim.x) {
    const int r = i / DHM, c = i % DHM;
    const float v = load_f(base + (long long)(first + r < last ? first + r : last) * stride + (c < dh ? c : 0));
    dst[r * (DHM + 4) + c] = c < dh ? map(v) : 0.f;
  }
}

}  // namespace cca
