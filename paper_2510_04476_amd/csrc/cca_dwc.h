// Gradient of the folded filters (a partial sum per chunk of tokens): device code shared by the launch of its own
// (cca_prologue_bwd.hip) and by the one beside the adjoint of the prologue (cca_prologue.hip).
#pragma once

#include "cca_internal.h"

namespace cca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// ---------------------------------------------------------------------------
// 3. folded-filter gradient, partial sums per chunk of tokens.
//    Unit = (head, chunk of `chunk` tokens of one sequence[, slice of the output channels at d_h = 256]);
//    wavefront w owns OX output-channel tiles starting at OX*(w&1) and IX input-channel tiles starting at
//    IX*(w>>1), for all D taps (OX = d_h / 64 and IX = 1 up to d_h = 128).
// ---------------------------------------------------------------------------
// MFMA operand fragment of the TRANSPOSE of a row-major LDS tile: lane (c = lane & 31, half) receives
// tile[r0 + 4*half + {0..3}][c0 + c] and tile[r0 + 8 + 4*half + {0..3}][c0 + c].  `base` already holds the
// per-lane part  (4*half + ((lane & 15) >> 2)) * ROW + (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2.
template <int ROW>
__device__ __forceinline__ bf16x8 tr_frag(const unsigned char *base, int r0, int c0) {
  const unsigned char *p = base + r0 * ROW + c0 * 2;
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)p);
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(p + 8 * ROW));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

constexpr int DW_BT = 64;  // tokens per LDS tile

// Output slices per head and threads per workgroup: at d_h <= 128 one workgroup of d_h * 4 threads owns all of a head's
// d_h x D x d_h sums; at d_h = 256 they would not fit its registers, so 512 threads own a slice of 128 (D <= 2) or 64
// (D = 3) output channels and each such workgroup re-reads the token rows of all 256 input channels.
constexpr int dwc_slices(int DH, int D) { return DH <= 128 ? 1 : (D <= 2 ? 2 : 4); }
constexpr int dwc_threads(int DH) { return DH <= 128 ? DH * 4 : 512; }

struct DwcArgs {
  const bf16_t *d3, *lat;
  float *part;
  int T, Hq, Hk, e_q, e_kv, n_lat, chunk, chunks_per_seq, units;  // units = chunks of all sequences x heads
};
constexpr size_t dwc_lds(int DH, int D) {  // two stages of a gradient tile and a token tile
  return 2 * ((size_t)DW_BT * (DH / dwc_slices(DH, D) * 2 + 64) + (size_t)(DW_BT + D - 1) * (DH * 2 + 64));
}

// One unit by dwc_threads(DH) threads, `tid` of them the caller.  SHARED: several units to a workgroup, which pass the same barriers;
// a unit past the last works on the last one's tokens and stores nothing.
template <int DH, int D, bool SHARED = false>
__device__ __forceinline__ void dwc_body(const DwcArgs &w, int unit_, int slice, int tid, unsigned char *smem) {
  constexpr int OS = dwc_slices(DH, D), DHO = DH / OS, DW_NT = dwc_threads(DH), NW = DW_NT / 64;
  // LDS rows of the gradient tile (this slice's output channels) and of the token tile (all input channels); the
  // 64-byte pad keeps the transposing reads conflict-free
  constexpr int ROWY = DHO * 2 + 64, ROWU = DH * 2 + 64, CPWY = DHO / 8, CPWU = DH / 8;
  constexpr int OX = DHO / 64, IX = (DH / 32) / (NW / 2);  // output / input channel tiles per wavefront
  static_assert(OX >= 1 && IX >= 1 && OX * 2 * 32 == DHO && IX * (NW / 2) * 32 == DH, "wavefront tiling");
  constexpr int UROWS = DW_BT + D - 1;
  constexpr int DY_TILE = DW_BT * ROWY, U_TILE = UROWS * ROWU;
  static_assert(2 * (DY_TILE + U_TILE) == dwc_lds(DH, D), "LDS");
  unsigned char *const sDy = smem, *const sU = smem + 2 * DY_TILE;

  const int lane = tid & 63, wave = tid >> 6, T = w.T, NH = w.Hq + w.Hk, n_lat = w.n_lat;
  const bool stores = unit_ < w.units;
  const int unit = stores ? unit_ : w.units - 1;
  const int l32 = lane & 31, half = lane >> 5;
  const int head = unit % NH, cid = unit / NH;  // cid = b * chunks_per_seq + chunk index
  const int o_base = slice * DHO;               // first output channel of this slice
  const int b = cid / w.chunks_per_seq, t_begin = (cid % w.chunks_per_seq) * w.chunk;
  const int t_end = min(T, t_begin + w.chunk);
  const int ch0 = head < w.Hq ? head * DH : w.e_q + (head - w.Hq) * DH;
  const int ld3 = w.e_q + w.e_kv;
  const bf16_t *const d3b = w.d3 + (long long)b * T * ld3 + ch0 + o_base;
  const bf16_t *const ub = w.lat + (long long)b * T * n_lat + ch0;

  constexpr int DY_CHUNKS = DW_BT * CPWY, U_CHUNKS = UROWS * CPWU;  // 16-byte chunks per tile
  constexpr int DY_PER = DY_CHUNKS / DW_NT, U_PER = (U_CHUNKS + DW_NT - 1) / DW_NT;
  static_assert(DY_CHUNKS % DW_NT == 0, "gradient tile must divide over the threads");
  u32x4 rdy[DY_PER], ru[U_PER];
  auto load_tile = [&](int t0) {
#pragma unroll
    for (int i = 0; i < DY_PER; ++i) {
      const int id = tid + i * DW_NT, r = id / CPWY, c = id % CPWY;
      const int t = t0 + r;
      u32x4 val = {0, 0, 0, 0};
      if (t < t_end) val = *reinterpret_cast<const u32x4 *>(d3b + (long long)t * ld3 + c * 8);
      rdy[i] = val;
    }
#pragma unroll
    for (int i = 0; i < U_PER; ++i) {
      const int id = tid + i * DW_NT, r = id / CPWU, c = id % CPWU;
      const int t = t0 - (D - 1) + r;  // row r of the tile holds token t0 - (D-1) + r
      u32x4 val = {0, 0, 0, 0};
      if (id < U_CHUNKS && t >= 0 && t < t_end) val = *reinterpret_cast<const u32x4 *>(ub + (long long)t * n_lat + c * 8);
      ru[i] = val;
    }
  };
  auto store_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < DY_PER; ++i) {
      const int id = tid + i * DW_NT, r = id / CPWY, c = id % CPWY;
      *reinterpret_cast<u32x4 *>(sDy + buf * DY_TILE + r * ROWY + c * 16) = rdy[i];
    }
#pragma unroll
    for (int i = 0; i < U_PER; ++i) {
      const int id = tid + i * DW_NT, r = id / CPWU, c = id % CPWU;
      if (id < U_CHUNKS) *reinterpret_cast<u32x4 *>(sU + buf * U_TILE + r * ROWU + c * 16) = ru[i];
    }
  };

  const uint32_t tr_row = (uint32_t)(4 * half + ((lane & 15) >> 2)), tr_col = (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2;
  const uint32_t tr_off_y = tr_row * ROWY + tr_col, tr_off_u = tr_row * ROWU + tr_col;
  const int o_tile0 = OX * (wave & 1), i_tile0 = IX * (wave >> 1);

  f32x16 acc[OX][IX][D];
#pragma unroll
  for (int x = 0; x < OX; ++x)
#pragma unroll
    for (int y = 0; y < IX; ++y)
#pragma unroll
      for (int d = 0; d < D; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[x][y][d][r] = 0.f;

  const int ntiles = ((SHARED ? min(w.chunk, T) : t_end - t_begin) + DW_BT - 1) / DW_BT;  // (past t_end the tiles are zeros)
  load_tile(t_begin);
  store_tile(0);
  if (ntiles > 1) load_tile(t_begin + DW_BT);
  __syncthreads();
  for (int it = 0; it < ntiles; ++it) {
    const int buf = it & 1;
    if (it + 1 < ntiles) store_tile(buf ^ 1);
    if (it + 2 < ntiles) load_tile(t_begin + (it + 2) * DW_BT);
    const unsigned char *dyp = sDy + buf * DY_TILE + tr_off_y, *up = sU + buf * U_TILE + tr_off_u;
#pragma unroll
    for (int kk = 0; kk < DW_BT / 16; ++kk) {
      bf16x8 fo[OX], fu[IX][D];
#pragma unroll
      for (int x = 0; x < OX; ++x) fo[x] = tr_frag<ROWY>(dyp, kk * 16, (o_tile0 + x) * 32);
#pragma unroll
      for (int y = 0; y < IX; ++y)
#pragma unroll
        for (int d = 0; d < D; ++d) fu[y][d] = tr_frag<ROWU>(up, kk * 16 + d, (i_tile0 + y) * 32);  // token t - (D-1-d)
#pragma unroll
      for (int x = 0; x < OX; ++x)
#pragma unroll
        for (int y = 0; y < IX; ++y)
#pragma unroll
          for (int d = 0; d < D; ++d)
            acc[x][y][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo[x], fu[y][d], acc[x][y][d], 0, 0, 0);
    }
    __syncthreads();
  }
  // acc[x][y][d][r]: o = o_base + (o_tile0 + x)*32 + 8*(r/4) + 4*half + r%4,  i = (i_tile0 + y)*32 + l32
  if (!stores) return;
  float *out = w.part + (long long)unit * DH * D * DH;  // [o][d][i] of (cid, head)
#pragma unroll
  for (int x = 0; x < OX; ++x)
#pragma unroll
    for (int y = 0; y < IX; ++y)
#pragma unroll
      for (int d = 0; d < D; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int o = o_base + (o_tile0 + x) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
          out[(o * D + d) * DH + (i_tile0 + y) * 32 + l32] = acc[x][y][d][r];
        }
}

}  // namespace cca
