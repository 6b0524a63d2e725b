// Pieces shared by the shape-generic kernels (cca_generic.hip, cca_generic_bwd.hip): products of fp32 values on the matrix
// cores with v_mfma_f32_32x32x2_f32, operands straight from memory (any storage type, converted on the way).
//
// One such MFMA adds, for a 32 x 32 tile D[row][col], two terms of the contraction: lane (l32, half) supplies term `half`
// of row l32 (first operand) and of column l32 (second).  Which two terms meet is free, so the contraction is walked 8 at a
// time and lane half h takes terms 4 h + i of MFMA i: four adjacent values, one 16-byte load where the operand is stored
// along the contraction.  The result sits as D[8 (r / 4) + 4 half + r % 4][l32] in register r - which is also that order, so
// a tile of results is the second operand of the next product as it stands.
#pragma once

#include <type_traits>

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
// Four values as they lie in memory, and their conversion
__device__ __forceinline__ gen_f32x4 raw4(const float *p) { return *reinterpret_cast<const gen_f32x4 *>(p); }
__device__ __forceinline__ gen_u32x2 raw4(const bf16_t *p) { return *reinterpret_cast<const gen_u32x2 *>(p); }
template <typename T>
struct Raw4 {
  T v[4];
};
__device__ __forceinline__ gen_f32x4 raw_to_f32(gen_f32x4 r) { return r; }
__device__ __forceinline__ gen_f32x4 raw_to_f32(gen_u32x2 w) {
  return gen_f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u)};
}
template <typename T>
__device__ __forceinline__ gen_f32x4 raw_to_f32(const Raw4<T> &r) {
  return gen_f32x4{load_f(r.v), load_f(r.v + 1), load_f(r.v + 2), load_f(r.v + 3)};
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
__device__ __forceinline__ gen_f32x16 dot_tile32(const T *rows, const float *cols, int dh, int half, F &&map) {
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
__device__ __forceinline__ void add_outer32(gen_f32x16 (&acc)[DT], const float (&w)[16], Row &&row, int dh, int lane, bool mixed) {
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

// ---- 16 x 16 tiles (attention): v_mfma_f32_16x16x4_f32 -------------------------------------------------------------------
// Lane (l16, g), g = lane / 16, supplies term g of row l16 and of column l16; the result sits as D[4 g + r][l16] in register
// r, which is again the order of a second operand when MFMA i takes the terms 4 g + i.  Half the rows of the 32 x 32 form: twice
// the workgroups and half the accumulators for the same rate.

// rows . cols over `dh` channels (a multiple of 4): row l16 of the tile at `rows` (this lane's row), column l16 in LDS
// at `cols`, zero from dh up to DHM.
template <int DHM, typename T, typename F>
__device__ __forceinline__ gen_f32x4 dot_tile16(const T *rows, const float *cols, int dh, int g, F &&map) {
  gen_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int CHUNK = DHM <= 64 ? 32 : 64;  // channels in flight
#pragma unroll 1
  for (int c0 = 0; c0 < DHM; c0 += CHUNK)
#pragma unroll
    for (int c = 0; c < CHUNK; c += 16) {
      const int ch = c0 + c + 4 * g;
      gen_f32x4 a = load4(rows + (ch < dh ? ch : 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = ch < dh ? map(a[i]) : 0.f;
      const gen_f32x4 b = load4(cols + ch);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], acc, 0, 0, 0);
    }
  return acc;
}

// add_outer32 for 16 rows: acc[dt][.] (rows: channels 16 dt + ..., column: this lane's)
template <int DT, typename T, typename Row>
__device__ __forceinline__ void add_outer16(gen_f32x4 (&acc)[DT], const gen_f32x4 &w, Row &&row, int dh, int lane, bool mixed) {
  const int l16 = lane & 15, g = lane >> 4;
  const T *p[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) p[i] = static_cast<const T *>(row(4 * g + i));
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const int ch = 16 * dt + l16;
    float x[4];
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = load_f(p[i] + (ch < dh ? ch : 0));
      x[i] = ch < dh ? x[i] : 0.f;
      bad |= !(fabsf(x[i]) < INFINITY);
    }
    if (mixed && __any(bad)) {
#pragma unroll 1
      for (int k = 0; k < 16; ++k) {
        float wk = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float o = __shfl(w[i], l16 + 16 * (k >> 2));
          wk = i == (k & 3) ? o : wk;
        }
        const T *pk = static_cast<const T *>(row(k));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = 16 * dt + 4 * g + r;
          const float v = load_f(pk + (c < dh ? c : 0));
          acc[dt][r] = wk != 0.f && c < dh ? fmaf(v, wk, acc[dt][r]) : acc[dt][r];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], w[i], acc[dt], 0, 0, 0);
    }
  }
}

// ROWS rows of `dh` channels -> LDS [ROWS][DHM + 4] floats (rows padded by 16 bytes), times `map`; rows past `last` repeat it,
// channels from dh on are zero.
template <int DHM, int ROWS, typename T, typename F>
__device__ __forceinline__ void stage_rows(float *dst, const T *base, long long stride, int first, int last, int dh, F &&map) {
  for (int i = threadIdx.x; i < ROWS * DHM; i += blockDim.x) {
    const int r = i / DHM, c = i % DHM;
    const float v = load_f(base + (long long)(first + r < last ? first + r : last) * stride + (c < dh ? c : 0));
    dst[r * (DHM + 4) + c] = c < dh ? map(v) : 0.f;
  }
}

// Threads of an attention workgroup: the 16-row form's at most (beyond d_h = 64 the accumulators want more than the 128 registers that 1024 leave), and
// output tiles whose partial sums are added in one go
constexpr int G32_NT = 512, G32_WAVES = G32_NT / 64;  // the 32-row form
template <int DHM>
constexpr int G16_NT = DHM <= 64 ? 1024 : 512;
constexpr int G16_TILES = 2;
typedef float G16Partial[G16_TILES][4][64];

// Sums of the wavefronts' accumulators, each times f(wavefront) where that is not 0, in wavefront order: out(channel, sum) once
// per element of the tile, for column l16 of the calling lane.
template <int WAVES, int DT, typename W, typename F>
__device__ __forceinline__ void sum_wavefronts16(const gen_f32x4 (&acc)[DT], G16Partial *so, W &&weight, F &&out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d0 = 0; d0 < DT; d0 += G16_TILES) {
    __syncthreads();
#pragma unroll
    for (int x = 0; x < G16_TILES; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) so[wave][x][r][lane] = acc[d0 + x][r];
    __syncthreads();
    static_assert(WAVES >= G16_TILES * 4, "a wavefront per register of the tiles");
    if (wave < G16_TILES * 4) {
      const int x = wave >> 2, r = wave & 3;
      float sum = 0.f;
#pragma unroll
      for (int y = 0; y < WAVES; ++y) {
        const float f = weight(y);
        sum += f == 0.f ? 0.f : so[y][x][r][lane] * f;
      }
      out(16 * (d0 + x) + 4 * (lane >> 4) + r, sum);
    }
  }
}

// ---- prologue and its adjoint: one head x 32 tokens of a sequence per workgroup of four wavefronts ------------------------
constexpr int GP_NT = 256, GP_WAVES = GP_NT / 64, GP_TOK = 32;
constexpr int GP_RED = GP_WAVES * 16 * 64;       // floats of gp_sum's buffer
constexpr size_t GP_MAX_LDS = 160 * 1024;
constexpr long long GP_GRID = 1ll << 23;         // workgroups of a launch, which takes fewer than 2^32 threads in one dimension
// Launches `go(first block, blocks)` over B sequences of T tokens, `tok` of them to a workgroup
template <typename F>
inline hipError_t gp_launches(int B, int T, int tok, F &&go) {
  const long long blocks = (long long)((T + tok - 1) / tok) * B;
  for (long long x = 0; x < blocks; x += GP_GRID) {
    go((unsigned)x, (unsigned)(blocks - x < GP_GRID ? blocks - x : GP_GRID));
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// cos, sin of the RoPE angles of `rows` tokens from t0 on, (token, pair) to sa[2 (token * d_h / 2 + pair)].  fp64: t * theta loses
// ~1e-3 rad in fp32 at t ~ 16k.  A thread takes one pair and a run of tokens, whose angles follow from the first by rotation in fp64
// (the error grows by 1e-16 a token).
__device__ __forceinline__ void rope_angles(float *sa, float base, int dh, int t0, int rows) {
  const int half = dh / 2, runs = GP_NT / half > 0 ? GP_NT / half : 1, len = (rows + runs - 1) / runs;
  for (int id = threadIdx.x; id < half * runs; id += GP_NT) {
    const int p = id % half, x0 = id / half * len;
    const double theta = pow((double)base, -2.0 * (double)p / (double)dh);
    double sn, cs, s1 = 0.0, c1 = 1.0;
    sincos((double)(t0 + x0) * theta, &sn, &cs);
    if (len > 1) sincos(theta, &s1, &c1);
    for (int x = x0; x < x0 + len && x < rows; ++x) {
      sa[2 * (x * half + p)] = (float)cs;
      sa[2 * (x * half + p) + 1] = (float)sn;
      const double c2 = cs * c1 - sn * s1;
      sn = sn * c1 + cs * s1;
      cs = c2;
    }
  }
}

// go(std::integral_constant<int, n>) for n = 1 ... 4: a tap count the compiler knows, so that an index costs no division
template <typename F>
__device__ __forceinline__ void gp_taps(int n, F &&go) {
  if (n == 1) go(std::integral_constant<int, 1>{});
  else if (n == 2) go(std::integral_constant<int, 2>{});
  else if (n == 3) go(std::integral_constant<int, 3>{});
  else go(std::integral_constant<int, 4>{});
}

// The wavefronts' shares added in order: out(row, column, sum) once per element of the 32 x 32 tile
template <typename F>
__device__ __forceinline__ void gp_sum(const gen_f32x16 &acc, float *red, F &&out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[r];
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 16 / GP_WAVES; ++x) {
    const int r = wave * (16 / GP_WAVES) + x;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < GP_WAVES; ++w) sum += red[(w * 16 + r) * 64 + lane];
    out(tile_row(r, lane >> 5), lane & 31, sum);
  }
}

// sum_n A[row][n] B[n][column] over the terms n = c * TAPS + j, c < dh (a multiple of 4), j < TAPS, for ceil(rows / 32) tiles of 32 rows one
// after the other, the terms dealt to the wavefronts in blocks of 8: lane (l32, half) supplies row r as a4(r, n), terms n ... n + 3 (n a
// multiple of 4) as they lie in memory, and column l32 as b(c, j); out(row, column, sum).  What bounds it is the latency of a's loads,
// so those of a tile's first AHEAD blocks per wavefront are requested before the sums of the tile before it are added.
template <int TAPS, int AHEAD, typename FA, typename FB, typename F>
__device__ __forceinline__ void gp_product(int dh, int rows, float *red, FA &&a4, FB &&b, F &&out) {
  constexpr int STEP = GP_WAVES * 8;
  const int terms = dh * TAPS, half = (threadIdx.x >> 5) & 1, l32 = threadIdx.x & 31, first = (threadIdx.x >> 6) * 8;
  decltype(a4(0, 0)) x[AHEAD];
  auto request = [&](int r0, int b0) __attribute__((always_inline)) {
    const int r = r0 + l32 < rows ? r0 + l32 : rows - 1;  // past the last: results not kept
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (b0 + u * STEP >= terms) break;
      const int n = b0 + u * STEP + 4 * half;
      x[u] = a4(r, n < terms ? n : 0);
    }
  };
  request(0, first);
  for (int r0 = 0; r0 < rows; r0 += 32) {
    gen_f32x16 acc = zero16();
    for (int b0 = first; b0 < terms; b0 += AHEAD * STEP) {
      if (b0 != first) request(r0, b0);
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (b0 + u * STEP >= terms) break;
        const int n0 = b0 + u * STEP + 4 * half;
        const bool in = n0 < terms;  // a multiple of 4: the four terms of a lane are in or out together
        const int n = in ? n0 : 0;
        const gen_f32x4 v = raw_to_f32(x[u]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float y = TAPS == 3 ? b((n + i) / 3, (n + i) % 3) : b(n / TAPS + i / TAPS, i % TAPS);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? v[i] : 0.f, in ? y : 0.f, acc, 0, 0, 0);
        }
      }
    }
    if (r0 + 32 < rows) request(r0 + 32, first);
    gp_sum(acc, red, [&](int r, int column, float sum) {
      if (r0 + r < rows) out(r0 + r, column, sum);
    });
  }
}

}  // namespace cca
