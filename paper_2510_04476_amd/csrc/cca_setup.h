// Set-up of the fused prologue and of its adjoint: device code shared by the launch of its own (cca_prologue.hip) and by a launch
// that does it beside other work (cca_attention_bwd.hip).
//   folded filters Wc [h][o][d][i] (adjoint: [h][i][d][o]; d_h = 256: in the slab order of prologue_stream_kernel), bf16
//   ropeA [t_hi][i]            float2 (cos, sin) of t_hi * 128 * theta_i
//   ropeB [i / 4][t_lo][i % 4] float2 (cos, sin) of t_lo * theta_i
#pragma once

#include "cca_internal.h"

namespace cca {

// d_h = 256: the filter as prologue_stream_kernel moves it, in slabs of all 256 rows x 32 contracted channels of one tap,
// each slab exactly as it lies in LDS (two rows share a 128-byte line; 16-byte chunk c of row r at line r / 2, position
// (4 (r mod 2) + c) ^ ((r / 4) mod 4): 16 consecutive rows of one chunk column fall in 16 different bank groups).
constexpr int SLAB_K = 32, SLAB_BYTES = 256 * SLAB_K * 2;
__device__ __forceinline__ long long slab_elem(int h, int D, int r, int d, int k) {
  const int c = (k & 31) >> 3;
  return ((long long)(h * D + d) * (256 / SLAB_K) + (k >> 5)) * (SLAB_BYTES / 2) + ((r >> 1) * 8 + ((((r & 1) << 2) | c) ^ ((r >> 2) & 3))) * 8 + (k & 7);
}

// One block of 256 threads of the set-up's `s.n_blocks`
__device__ __forceinline__ void setup_block(const PrologueSetup &s, int block) {
  const int DH = s.dh, D = s.D;
  if (block < s.n_fold) {
    const long long id = (long long)block * 256 + threadIdx.x;  // (h, o, i)
    if (id >= (long long)s.heads * DH * DH) return;
    const int i = (int)(id % DH), o = (int)((id / DH) % DH), h = (int)(id / (DH * DH));
    const int ch = h * DH + i;  // packed q|k channel: q heads first, then k heads
    // D = k_seq + k_ch - 1 <= 3 on this path; absent taps read the last one and are dropped, so that all loads are in flight together
    const bf16_t *const p0 = s.w0 ? s.w0 + (long long)ch * s.k_seq : s.w1, *const p1 = s.w1 + id * s.k_ch;
    bf16_t f0[3], f1[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) f0[j] = p0[min(j, s.k_seq - 1)], f1[j] = p1[min(j, s.k_ch - 1)];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if (d >= D) break;
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j <= d; ++j)
        if (j < s.k_ch && d - j < s.k_seq) acc = fmaf(bf16_to_f32(f1[j]), s.w0 ? bf16_to_f32(f0[d - j]) : 1.f, acc);
      // the adjoint convolution contracts over the output channel: filter stored [h][i][d][o]
      const int r = s.transposed ? i : o, k = s.transposed ? o : i;
      s.wc[DH == 256 ? slab_elem(h, D, r, d, k) : (((long long)h * DH + r) * D + d) * DH + k] = f32_to_bf16(acc);
    }
    return;
  }
  const int id = (block - s.n_fold) * 256 + threadIdx.x;
  const int nA = s.n_thi * (DH / 2), nB = (DH / 2) * 128;
  if (id >= nA + nB) return;
  const bool hi = id < nA;
  const int i = hi ? id % (DH / 2) : (id - nA) / 128, t = hi ? id / (DH / 2) * 128 : (id - nA) % 128;
  const double theta = pow((double)s.rope_base, -2.0 * (double)i / (double)DH);
  double sn, cs;
  sincos((double)t * theta, &sn, &cs);
  float2 *const to = hi ? s.ropeA + id : s.ropeB + ((i >> 2) * 128 + t) * 4 + (i & 3);
  *to = make_float2((float)cs, (float)sn);
}

}  // namespace cca
