// Shape-generic backward kernels (adjoints of the steps of Sec. 2.2, which the
// paper states forward only): fp32 or bf16 storage, fp32 arithmetic (the
// contractions on the fp32 matrix cores).  They serve the fp32 configuration and
// every bf16 shape the bf16 MFMA backward kernels do not cover.  Every sum runs in a fixed order (no
// atomics), so results are reproducible bit for bit.
#include "cca_generic.h"

namespace cca {

// ---------------------------------------------------------------------------
// Attention backward.  With P = softmax(scale Q K^T) row-wise and
// Delta_t = <dO_t, O_t>:  dS = P * (dO V^T - Delta),  dQ = scale dS K,
// dK = scale dS^T Q,  dV = P^T dO;  dK, dV summed over the query heads of a group.
// ---------------------------------------------------------------------------
// Delta: 8 lanes per row, 4 channels each at a time
template <typename T>
__global__ __launch_bounds__(256) void delta_generic_kernel(const T *__restrict__ dO, const T *__restrict__ O,
                                                           const T *__restrict__ OLO, float *__restrict__ delta,
                                                           long long n_rows, int Tn, int Hq, int dh) {
  for (long long row0 = (long long)blockIdx.x * 32; row0 < n_rows; row0 += (long long)gridDim.x * 32) {
    const long long row = row0 + (threadIdx.x >> 3);  // (b*T + t)*Hq + h
    const long long off = (row < n_rows ? row : n_rows - 1) * dh;
    float acc = 0.f;
#pragma unroll 2
    for (int i = 4 * (threadIdx.x & 7); i < dh; i += 32) {
      const gen_f32x4 d = load4(dO + off + i);
      gen_f32x4 v = load4(O + off + i);
      if (OLO) v += load4(OLO + off + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = fmaf(d[e], v[e], acc);
    }
#pragma unroll
    for (int x = 1; x < 8; x *= 2) acc += __shfl_xor(acc, x);
    if (row < n_rows && (threadIdx.x & 7) == 0) {
      const long long bt = row / Hq;
      const int h = (int)(row % Hq);
      delta[((bt / Tn) * Hq + h) * Tn + (bt % Tn)] = acc;
    }
  }
}

// log2-unit score against the forward MFMA kernel's own rounding of q (q * scale * log2(e) rounded to bf16):
// used when that kernel produced lse, so that the recomputed probabilities are exactly its probabilities
__device__ __forceinline__ float q_log2_rounded(float q, float c) { return bf16_to_f32(f32_to_bf16(q * c)); }
constexpr float kLog2e = 1.44269504088896340736f;

// Sums of the wavefronts' accumulators, in wavefront order: out(channel, column l32, sum) once per element of the tile
template <int DT, typename F>
__device__ __forceinline__ void sum_wavefronts32(const gen_f32x16 (&acc)[DT], float (*so)[16][64], int wave, int lane, F &&out) {
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) so[wave][r][lane] = acc[dt][r];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 16 / G32_WAVES; ++x) {
      const int r = wave * (16 / G32_WAVES) + x;
      float sum = 0.f;
#pragma unroll
      for (int y = 0; y < G32_WAVES; ++y) sum += so[y][r][lane];
      out(32 * dt + tile_row(r, lane >> 5), sum);
    }
  }
}

// Workgroup = 32 query rows of one head, the key tiles dealt to its 8 wavefronts; S^T and dP^T with one query per lane, dS^T
// is the second operand of dQ^T += K^T dS^T as it stands.  T = 1000, 2 heads of 32, fp32: 26 us; one wavefront per row on
// the vector ALU took 117.
template <typename T, int DHM>
__global__ __launch_bounds__(G32_NT) void attn_bwd_dq_generic_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                   const T *__restrict__ v, const T *__restrict__ dO,
                                                                   const float *__restrict__ lse,
                                                                   const float *__restrict__ delta, T *__restrict__ dq, int Tn,
                                                                   int Hq, int Hk, int dh, float scale, int causal,
                                                                   int q_rounded) {
  constexpr int DT = DHM / 32;
  __shared__ __attribute__((aligned(16))) float sq[32 * (DHM + 4)], sd[32 * (DHM + 4)];
  __shared__ float so[G32_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int qb = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z, g = h / (Hq / Hk);
  const int q0 = qb * 32, t = q0 + l32, tc = min(t, Tn - 1);
  const T *const kb = k + ((long long)b * Tn * Hk + g) * dh, *const vb = v + ((long long)b * Tn * Hk + g) * dh;
  const long long ks = (long long)Hk * dh, qs = (long long)Hq * dh, q_off = ((long long)b * Tn * Hq + h) * dh;
  stage_rows<DHM, 32>(sq, q + q_off, qs, q0, Tn - 1, dh,
                    [=](float x) { return q_rounded ? q_log2_rounded(x, scale * kLog2e) : x * scale; });
  stage_rows<DHM, 32>(sd, dO + q_off, qs, q0, Tn - 1, dh, [](float x) { return x; });
  const float L = lse[((long long)b * Hq + h) * Tn + tc] * (q_rounded ? kLog2e : 1.f);
  const float Dl = delta[((long long)b * Hq + h) * Tn + tc];
  __syncthreads();
  gen_f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16();
  const int end = causal ? min(q0 + 32, Tn) : Tn;
  auto same = [](float x) { return x; };
  for (int k0 = wave * 32; k0 < end; k0 += G32_WAVES * 32) {
    const long long krow = min(k0 + l32, Tn - 1) * ks;
    const gen_f32x16 s = dot_tile32<DHM>(kb + krow, sq + l32 * (DHM + 4), dh, half, same);
    const gen_f32x16 dp = dot_tile32<DHM>(vb + krow, sd + l32 * (DHM + 4), dh, half, same);
    const bool mixed = k0 + 32 > Tn || (causal && k0 + 31 > q0);
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + tile_row(r, half);
      const float x = (q_rounded ? exp2f(s[r] - L) : expf(s[r] - L)) * (dp[r] - Dl);
      w[r] = key < Tn && (!causal || key <= t) ? x : 0.f;
    }
    add_outer32<DT, T>(acc, w, [=](int x) { return kb + min(k0 + x, Tn - 1) * ks; }, dh, lane, mixed);
  }
  sum_wavefronts32(acc, so, wave, lane, [&](int ch, float sum) {
    if (t < Tn && ch < dh) store_f(dq + q_off + t * qs + ch, sum * scale);
  });
}

// Workgroup = 32 keys of one KV head, the (query head of the group, query tile) pairs that see them dealt to its 8
// wavefronts; S and dP with one key per lane.  WHICH: 1 = dK, 2 = dV, 3 = both in one pass, up to d_h = 128.  T = 1000, 2 heads of
// 32, fp32: 41.5 us; one wavefront per key, dK and dV apart, on the vector ALU took 305 + 189.
// At d_h 65 ... 128 the two sets of accumulators do not quite fit (79 registers spilled, none with one set), and one pass is
// still the faster: attention backward, fp32, d_h = 128, 1000 tokens, 8 / 1 heads 1130 us against 1323 in two, 4096, 4 / 4
// 1652 against 1729 (bf16, d_h = 96, 4096 causal the other way, 1879 and 1764).  The d_h = 256 instantiations here and in
// cca_generic.hip spill 79 to 93 registers of one set: 4096 tokens, 4 / 2 heads, backward 4.1 ms, on the vector ALU 154.
template <typename T, int DHM, int WHICH>
__global__ __launch_bounds__(G32_NT) void attn_bwd_dkv_generic_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                    const T *__restrict__ v, const T *__restrict__ dO,
                                                                    const float *__restrict__ lse,
                                                                    const float *__restrict__ delta, T *__restrict__ dk,
                                                                    T *__restrict__ dv, int Tn, int Hq, int Hk, int dh,
                                                                    float scale, int causal, int q_rounded) {
  constexpr int DT = DHM / 32;
  __shared__ __attribute__((aligned(16))) float sk[32 * (DHM + 4)], sv[32 * (DHM + 4)];
  __shared__ float so[G32_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int k0 = blockIdx.x * 32, g = blockIdx.y, b = blockIdx.z, R = Hq / Hk, key = k0 + l32;
  const long long ks = (long long)Hk * dh, qs = (long long)Hq * dh, k_off = ((long long)b * Tn * Hk + g) * dh;
  stage_rows<DHM, 32>(sk, k + k_off, ks, k0, Tn - 1, dh, [=](float x) { return x * (q_rounded ? 1.f : scale); });
  stage_rows<DHM, 32>(sv, v + k_off, ks, k0, Tn - 1, dh, [](float x) { return x; });
  __syncthreads();
  gen_f32x16 ak[WHICH & 1 ? DT : 1], av[WHICH & 2 ? DT : 1];
#pragma unroll
  for (int dt = 0; dt < (WHICH & 1 ? DT : 1); ++dt) ak[dt] = zero16();
#pragma unroll
  for (int dt = 0; dt < (WHICH & 2 ? DT : 1); ++dt) av[dt] = zero16();
  const int first = causal ? k0 / 32 : 0, tiles = (Tn + 31) / 32 - first;
  for (int idx = wave; idx < R * tiles; idx += G32_WAVES) {
    const int h = g * R + idx / tiles, t0 = (first + idx % tiles) * 32;
    const T *const qb = q + ((long long)b * Tn * Hq + h) * dh, *const db = dO + ((long long)b * Tn * Hq + h) * dh;
    const long long qrow = min(t0 + l32, Tn - 1) * qs, st = ((long long)b * Hq + h) * Tn;
    const gen_f32x16 s = dot_tile32<DHM>(qb + qrow, sk + l32 * (DHM + 4), dh, half,
                                       [=](float x) { return q_rounded ? q_log2_rounded(x, scale * kLog2e) : x; });
    gen_f32x16 dp;
    if constexpr (WHICH & 1) dp = dot_tile32<DHM>(db + qrow, sv + l32 * (DHM + 4), dh, half, [](float x) { return x; });
    const bool mixed = t0 + 32 > Tn || (causal && t0 < k0 + 31);
    float p[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int t = t0 + tile_row(r, half), tc = min(t, Tn - 1);
      const float L = lse[st + tc];
      const bool in = t < Tn && (!causal || key <= t);
      p[r] = in ? (q_rounded ? exp2f(s[r] - L * kLog2e) : expf(s[r] - L)) : 0.f;
      if constexpr (WHICH & 1) ds[r] = in ? p[r] * (dp[r] - delta[st + tc]) * scale : 0.f;
    }
    if constexpr (WHICH & 2) add_outer32<DT, T>(av, p, [=](int x) { return db + min(t0 + x, Tn - 1) * qs; }, dh, lane, mixed);
    if constexpr (WHICH & 1) add_outer32<DT, T>(ak, ds, [=](int x) { return qb + min(t0 + x, Tn - 1) * qs; }, dh, lane, mixed);
  }
  if constexpr (WHICH & 1)
    sum_wavefronts32(ak, so, wave, lane, [&](int ch, float sum) {
      if (key < Tn && ch < dh) store_f(dk + k_off + key * ks + ch, sum);
    });
  if constexpr (WHICH & 2)
    sum_wavefronts32(av, so, wave, lane, [&](int ch, float sum) {
      if (key < Tn && ch < dh) store_f(dv + k_off + key * ks + ch, sum);
    });
}

template <typename T>
struct AttnBwdArgs {
  const T *q, *k, *v, *dO;
  const float *lse, *delta;
  T *dq, *dk, *dv;
  int Tn, Hq, Hk, dh;
  float scale;
  int causal, q_rounded;
};

// 16 query rows of one head, the key steps dealt to the 16 wavefronts; S^T and dP^T with one query per lane, dS^T
// is the second operand of dQ^T += K^T dS^T as it stands.
template <typename T, int DHM>
__device__ __forceinline__ void attn_bwd_dq_rows(const AttnBwdArgs<T> &a, int q0, int h, int b, float *sq, float *sd, G16Partial *so) {
  constexpr int DT = DHM / 16, WAVES = G16_NT<DHM> / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
  const int Tn = a.Tn, dh = a.dh, g = h / (a.Hq / a.Hk), t = q0 + l16, tc = min(t, Tn - 1);
  const T *const kb = a.k + ((long long)b * Tn * a.Hk + g) * dh, *const vb = a.v + ((long long)b * Tn * a.Hk + g) * dh;
  const long long ks = (long long)a.Hk * dh, qs = (long long)a.Hq * dh, q_off = ((long long)b * Tn * a.Hq + h) * dh;
  const bool q_rounded = a.q_rounded;
  const float scale = a.scale;
  stage_rows<DHM, 16>(sq, a.q + q_off, qs, q0, Tn - 1, dh,
                    [=](float x) { return q_rounded ? q_log2_rounded(x, scale * kLog2e) : x * scale; });
  stage_rows<DHM, 16>(sd, a.dO + q_off, qs, q0, Tn - 1, dh, [](float x) { return x; });
  const float L = a.lse[((long long)b * a.Hq + h) * Tn + tc] * (q_rounded ? kLog2e : 1.f);
  const float Dl = a.delta[((long long)b * a.Hq + h) * Tn + tc];
  __syncthreads();
  gen_f32x4 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
  const int end = a.causal ? min(q0 + 16, Tn) : Tn;
  auto same = [](float x) { return x; };
  for (int k0 = wave * 16; k0 < end; k0 += WAVES * 16) {
    const long long krow = min(k0 + l16, Tn - 1) * ks;
    const gen_f32x4 s = dot_tile16<DHM>(kb + krow, sq + l16 * (DHM + 4), dh, grp, same);
    const gen_f32x4 dp = dot_tile16<DHM>(vb + krow, sd + l16 * (DHM + 4), dh, grp, same);
    gen_f32x4 w;
    const bool mixed = k0 + 16 > Tn || (a.causal && k0 + 15 > q0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = k0 + 4 * grp + r;
      const float x = (q_rounded ? exp2f(s[r] - L) : expf(s[r] - L)) * (dp[r] - Dl);
      w[r] = key < Tn && (!a.causal || key <= t) ? x : 0.f;
    }
    add_outer16<DT, T>(acc, w, [=](int x) { return kb + min(k0 + x, Tn - 1) * ks; }, dh, lane, mixed);
  }
  sum_wavefronts16<WAVES>(acc, so, [](int) { return 1.f; }, [&](int ch, float sum) {
    if (t < Tn && ch < dh) store_f(a.dq + q_off + t * qs + ch, sum * scale);
  });
}

// 16 keys of one KV head, the (query head of the group, query tile) pairs that see them dealt to the 16
// wavefronts; S and dP with one key per lane.
template <typename T, int DHM>
__device__ __forceinline__ void attn_bwd_dkv_rows(const AttnBwdArgs<T> &a, int k0, int g, int b, float *sk, float *sv, G16Partial *so) {
  constexpr int DT = DHM / 16, WAVES = G16_NT<DHM> / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
  const int Tn = a.Tn, dh = a.dh, Hq = a.Hq, Hk = a.Hk, R = Hq / Hk, key = k0 + l16;
  const long long ks = (long long)Hk * dh, qs = (long long)Hq * dh, k_off = ((long long)b * Tn * Hk + g) * dh;
  const bool q_rounded = a.q_rounded;
  const float scale = a.scale;
  stage_rows<DHM, 16>(sk, a.k + k_off, ks, k0, Tn - 1, dh, [=](float x) { return x * (q_rounded ? 1.f : scale); });
  stage_rows<DHM, 16>(sv, a.v + k_off, ks, k0, Tn - 1, dh, [](float x) { return x; });
  __syncthreads();
  gen_f32x4 ak[DT], av[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) ak[dt] = av[dt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
  const int first = a.causal ? k0 / 16 : 0, tiles = (Tn + 15) / 16 - first;
  for (int idx = wave; idx < R * tiles; idx += WAVES) {
    const int h = g * R + idx / tiles, t0 = (first + idx % tiles) * 16;
    const T *const qb = a.q + ((long long)b * Tn * Hq + h) * dh, *const db = a.dO + ((long long)b * Tn * Hq + h) * dh;
    const long long qrow = min(t0 + l16, Tn - 1) * qs, st = ((long long)b * Hq + h) * Tn;
    float L[4], Dl[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int tc = min(t0 + 4 * grp + r, Tn - 1);
      L[r] = a.lse[st + tc];
      Dl[r] = a.delta[st + tc];
    }
    const gen_f32x4 s = dot_tile16<DHM>(qb + qrow, sk + l16 * (DHM + 4), dh, grp,
                                        [=](float x) { return q_rounded ? q_log2_rounded(x, scale * kLog2e) : x; });
    const gen_f32x4 dp = dot_tile16<DHM>(db + qrow, sv + l16 * (DHM + 4), dh, grp, [](float x) { return x; });
    gen_f32x4 p, ds;
    const bool mixed = t0 + 16 > Tn || (a.causal && t0 < k0 + 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 4 * grp + r;
      const bool in = t < Tn && (!a.causal || key <= t);
      p[r] = in ? (q_rounded ? exp2f(s[r] - L[r] * kLog2e) : expf(s[r] - L[r])) : 0.f;
      ds[r] = in ? p[r] * (dp[r] - Dl[r]) * scale : 0.f;
    }
    add_outer16<DT, T>(av, p, [=](int x) { return db + min(t0 + x, Tn - 1) * qs; }, dh, lane, mixed);
    add_outer16<DT, T>(ak, ds, [=](int x) { return qb + min(t0 + x, Tn - 1) * qs; }, dh, lane, mixed);
  }
  auto one = [](int) { return 1.f; };
  sum_wavefronts16<WAVES>(ak, so, one, [&](int ch, float sum) {
      if (key < Tn && ch < dh) store_f(a.dk + k_off + key * ks + ch, sum);
    });
  sum_wavefronts16<WAVES>(av, so, one, [&](int ch, float sum) {
      if (key < Tn && ch < dh) store_f(a.dv + k_off + key * ks + ch, sum);
    });
}

// Both in one launch, the key blocks (the longer chains) first: grid (blocks of 16 rows, KV heads + query heads, B).
// With Delta, T = 1000, 2 heads of 32, fp32: 24.5 us, where the 32-row kernels one after the other took 75.1; 200 tokens, 4 / 2 heads of 64:
// 67.9 -> 22.3.
template <typename T, int DHM>
__global__ __launch_bounds__(G16_NT<DHM>) void attn_bwd_generic16_kernel(AttnBwdArgs<T> a) {
  __shared__ __attribute__((aligned(16))) float s0[16 * (DHM + 4)], s1[16 * (DHM + 4)];
  __shared__ G16Partial so[G16_NT<DHM> / 64];
  const int y = blockIdx.y, b = blockIdx.z, keys = a.Hk;
  if (y >= keys) {
    attn_bwd_dq_rows<T, DHM>(a, ((int)gridDim.x - 1 - (int)blockIdx.x) * 16, y - keys, b, s0, s1, so);
  } else {
    attn_bwd_dkv_rows<T, DHM>(a, blockIdx.x * 16, y, b, s0, s1, so);
  }
}

template <typename T>
static hipError_t attention_bwd_generic_t(const Dims &d, const void *q, const void *k, const void *v, const void *o,
                                          const void *o_lo, const float *lse, const void *d_o, void *d_q, void *d_k, void *d_v,
                                          float *delta, hipStream_t s) {
  const long long n_rows = d.rows() * d.Hq;
  const long long delta_blocks = (n_rows + 31) / 32;
  delta_generic_kernel<T><<<(unsigned)(delta_blocks < 65536 ? delta_blocks : 65536), 256, 0, s>>>((const T *)d_o, (const T *)o, (const T *)o_lo, delta, n_rows,
                                                                        d.T, d.Hq, d.dh);
  const int causal = (d.flags & CCA_CAUSAL) ? 1 : 0;
  const int q_rounded = attention_mfma_supported(d) ? 1 : 0;  // lse then comes from the MFMA forward kernel
  if (generic_attention_bwd_16((long long)d.B * d.Hk, d.R, d.T, d.dh, causal, d.bf16)) {
    const AttnBwdArgs<T> a{(const T *)q, (const T *)k, (const T *)v, (const T *)d_o, lse, delta, (T *)d_q, (T *)d_k, (T *)d_v,
                           d.T, d.Hq, d.Hk, d.dh, d.scale, causal, q_rounded};
    const dim3 grid((d.T + 15) / 16, d.Hk + d.Hq, d.B);
    if (d.dh <= 32) attn_bwd_generic16_kernel<T, 32><<<grid, G16_NT<32>, 0, s>>>(a);
    else if (d.dh <= 64) attn_bwd_generic16_kernel<T, 64><<<grid, G16_NT<64>, 0, s>>>(a);
    else if (d.dh <= 128) attn_bwd_generic16_kernel<T, 128><<<grid, G16_NT<128>, 0, s>>>(a);
    else attn_bwd_generic16_kernel<T, 256><<<grid, G16_NT<256>, 0, s>>>(a);
    return hipGetLastError();
  }
  const dim3 gq((d.T + 31) / 32, d.Hq, d.B), gk((d.T + 31) / 32, d.Hk, d.B);
#define DQ(DH)                                                                                                          \
  attn_bwd_dq_generic_kernel<T, DH><<<gq, G32_NT, 0, s>>>((const T *)q, (const T *)k, (const T *)v, (const T *)d_o, lse, \
                                                         delta, (T *)d_q, d.T, d.Hq, d.Hk, d.dh, d.scale, causal, q_rounded)
#define DKV(DH, W)                                                                                                      \
  attn_bwd_dkv_generic_kernel<T, DH, W><<<gk, G32_NT, 0, s>>>((const T *)q, (const T *)k, (const T *)v, (const T *)d_o,  \
                                                             lse, delta, (T *)d_k, (T *)d_v, d.T, d.Hq, d.Hk, d.dh,     \
                                                             d.scale, causal, q_rounded)
#define LAUNCH(DH)          \
  do {                      \
    DQ(DH);                 \
    if constexpr (DH <= 128) { \
      DKV(DH, 3);           \
    } else {                \
      DKV(DH, 1);           \
      DKV(DH, 2);           \
    }                       \
  } while (0)
  if (d.dh <= 32) LAUNCH(32);
  else if (d.dh <= 64) LAUNCH(64);
  else if (d.dh <= 128) LAUNCH(128);
  else LAUNCH(256);
#undef LAUNCH
#undef DKV
#undef DQ
  return hipGetLastError();
}

hipError_t attention_bwd_generic(const Dims &d, const void *q, const void *k, const void *v, const void *o,
                                 const void *o_lo, const float *lse, const void *d_o, void *d_q, void *d_k, void *d_v, float *delta,
                                 hipStream_t s) {
  return d.bf16 ? attention_bwd_generic_t<bf16_t>(d, q, k, v, o, o_lo, lse, d_o, d_q, d_k, d_v, delta, s)
                : attention_bwd_generic_t<float>(d, q, k, v, o, nullptr, lse, d_o, d_q, d_k, d_v, delta, s);
}

// ---------------------------------------------------------------------------
// Prologue backward.  Notation: y5 = q / k as they enter attention, d3 = gradient
// of the vectors entering the norm step (= gradient of the conv2 output, since
// qk-mean adds to it), d1 = gradient of the conv1_seq output.  d3, d1 are fp32
// scratch of shape (B*T, e_q + e_kv), q channels first.
// ---------------------------------------------------------------------------
struct ProBwdArgs {
  int T, Hq, Hk, dh, R, e_q, e_kv, n_lat, v_half, k_seq, k_ch;
  long long rows;
  uint32_t flags;
  float rope_base;
};

// RoPE^T, norm / temperature backward:  y = x * mul with mul = sqrt(d_h) beta / |x|:  dx = mul * (dy - y <y,dy> / (d_h beta^2)),
// then (CONV_CH) conv2_seq+ch transposed: d1[t,h,i] = sum_j sum_o w1[h,o,i,j] d3[t + (k_ch-1-j), h, o] within the sequence.
// Workgroup = one q or k head x 32 tokens of a sequence, whose d3 rows (and the k_ch - 1 after them, formed again by the next
// workgroup) stay in LDS for the convolution, a product on the fp32 matrix cores with its terms (j, o) dealt to the four
// wavefronts (gp_product).  With the gradients below, us, a workgroup per token and unsplit sums -> this: fp32, 1000 tokens, 2 / 2 heads of 32
// 81.9 -> 20.7; 4096, 4 / 2 x 128 710 -> 164; 64 tokens, 2 / 2 x 256 69.0 -> 64.7; bf16, 64, 2 / 2 x 200 60.1 -> 53.3.
template <typename T, bool NARROW>
__global__ __launch_bounds__(GP_NT) void pro_bwd_point_generic_kernel(ProBwdArgs a, const T *__restrict__ q, const T *__restrict__ k,
                                                                     const float *__restrict__ rnorm,
                                                                     const float *__restrict__ temp, const T *__restrict__ dq,
                                                                     const T *__restrict__ dk, const T *__restrict__ w1,
                                                                     float *__restrict__ d3, float *__restrict__ d1,
                                                                     float *__restrict__ rowdot, unsigned block0) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int dh = a.dh, kc = (a.flags & CCA_CONV_CH) ? a.k_ch : 1, rows = GP_TOK + kc - 1, ldy = dh + 1;
  float *const sx = sm, *const sa = sx + rows * ldy, *const red = sa + 2 * rows * (dh / 2);  // d3 | cos, sin | sums of the wavefronts
  const int tid = threadIdx.x, head = blockIdx.y;
  const unsigned tiles = (a.T + GP_TOK - 1) / GP_TOK, block = block0 + blockIdx.x;
  const long long row0 = (long long)(block / tiles) * a.T;  // the sequence's first row
  const int t0 = block % tiles * GP_TOK;
  const bool is_q = head < a.Hq;
  const int g = head - a.Hq, ch0 = is_q ? head * dh : a.e_q + g * dh, ld = a.e_q + a.e_kv;
  if (a.flags & CCA_ROPE) rope_angles(sa, a.rope_base, dh, t0, rows);
  const float beta2 = (!is_q && (a.flags & CCA_KEY_TEMP) && (a.flags & CCA_QK_NORM)) ? expf(2.f * temp[g]) : 1.f;
  const T *const y5 = is_q ? q + head * dh : k + g * dh, *const dy5 = is_q ? dq + head * dh : dk + g * dh;
  const long long ldq = is_q ? a.e_q : a.e_kv;
  for (int x = tid >> 3; x < rows; x += GP_NT / 8) {  // 8 lanes to a token
    const int t = t0 + x, l8 = tid & 7;
    const bool in = t < a.T;
    const long long row = row0 + (in ? t : a.T - 1);
    float dot = 0.f;
#pragma unroll 8
    for (int o = l8; o < dh; o += 8) dot = fmaf(load_f(y5 + row * ldq + o), load_f(dy5 + row * ldq + o), dot);
#pragma unroll
    for (int e = 1; e < 8; e *= 2) dot += __shfl_xor(dot, e);
    if (!is_q && rowdot && in && x < GP_TOK && l8 == 0) rowdot[row * a.Hk + g] = dot;
    const bool norm = a.flags & CCA_QK_NORM;
    const float c = norm ? dot / ((float)dh * beta2) : 0.f, mul = norm ? rnorm[row * (a.Hq + a.Hk) + head] : 1.f;
#pragma unroll 8
    for (int o = l8; o < dh; o += 8)
      sx[x * ldy + o] = in ? (load_f(dy5 + row * ldq + o) - load_f(y5 + row * ldq + o) * c) * mul : 0.f;
  }
  __syncthreads();
  if (a.flags & CCA_ROPE) {
    // forward: (a, b) -> (a c - b s, b c + a s); adjoint rotates back
    const int half = dh / 2;
    for (int x = tid >> 3; x < rows; x += GP_NT / 8)
      for (int p = tid & 7; p < half; p += 8) {
        const bool il = a.flags & CCA_ROPE_INTERLEAVED;
        float *const f = sx + x * ldy + (il ? 2 * p : p), *const e = f + (il ? 1 : half);
        const float cs = sa[2 * (x * half + p)], sn = sa[2 * (x * half + p) + 1], u = *f, v = *e;
        *f = u * cs + v * sn;
        *e = v * cs - u * sn;
      }
    __syncthreads();
  }
  if (const int x = tid >> 3; t0 + x < a.T)
    for (int o = tid & 7; o < dh; o += 8) d3[(row0 + t0 + x) * ld + ch0 + o] = sx[x * ldy + o];
  if (!(a.flags & CCA_CONV_CH)) return;
  const T *const wh = w1 + (long long)head * dh * dh * kc;
  gp_taps(kc, [&](auto taps_c) __attribute__((always_inline)) {  // terms: output channel o of the forward convolution, tap j
    constexpr int TAPS = decltype(taps_c)::value;
    const int l32 = tid & 31;
    gp_product<TAPS, NARROW ? 2 : 8>(
        dh, dh, red,
        [&](int i, int n) {
          Raw4<T> w;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int o = TAPS == 3 ? (n + e) / 3 : n / TAPS + e / TAPS, j = TAPS == 3 ? (n + e) % 3 : e % TAPS;
            w.v[e] = wh[(o * dh + i) * TAPS + j];
          }
          return w;
        },
        [&](int o, int j) { return sx[(l32 + TAPS - 1 - j) * ldy + o]; },
        [&](int i, int tok, float sum) {
          if (t0 + tok < a.T) d1[(row0 + t0 + tok) * ld + ch0 + i] = sum;
        });
  });
}

// conv1_seq transposed + qk-mean adjoint + value-shift adjoint: element `id` of d_lat
template <typename T>
__device__ __forceinline__ void dlat_element(const ProBwdArgs &a, const T *__restrict__ w0, const float *__restrict__ d3,
                                             const float *__restrict__ d1, const T *__restrict__ dv, T *__restrict__ d_lat, long long id) {
  if (id >= a.rows * a.n_lat) return;
  const long long row = id / a.n_lat;
  const int c = (int)(id % a.n_lat);
  const int t = (int)(row % a.T);
  const int ld = a.e_q + a.e_kv, dh = a.dh;
  float val;
  if (c < ld) {
    if (a.flags & CCA_CONV_SEQ) {
      val = 0.f;
      for (int jj = 0; jj < a.k_seq; ++jj) {
        const int fwd = a.k_seq - 1 - jj;
        if (t + fwd < a.T) val = fmaf(load_f(w0 + (long long)c * a.k_seq + jj), d1[(row + fwd) * ld + c], val);
      }
    } else {
      val = d1[row * ld + c];
    }
    if (a.flags & CCA_QK_MEAN) {
      // m_q[h] = (q0[h] + k0[g]) / 2 enters q3[h] and, averaged over the group, k3[g]
      if (c < a.e_q) {
        const int h = c / dh, i = c % dh, g = h / a.R;
        val += 0.5f * d3[row * ld + c] + (0.5f / (float)a.R) * d3[row * ld + a.e_q + g * dh + i];
      } else {
        const int g = (c - a.e_q) / dh, i = (c - a.e_q) % dh;
        float sq = 0.f;
        for (int r = 0; r < a.R; ++r) sq += d3[row * ld + (g * a.R + r) * dh + i];
        val += 0.5f * sq + 0.5f * d3[row * ld + c];
      }
    }
  } else {
    const int cc = c - ld;
    const bool shifted = (a.flags & CCA_V_SHIFT) && cc >= a.v_half;
    if (!shifted) val = load_f(dv + row * a.e_kv + cc);
    else val = (t + 1 < a.T) ? load_f(dv + (row + 1) * a.e_kv + cc) : 0.f;
  }
  store_f(d_lat + id, val);
}

template <typename T>
__global__ __launch_bounds__(256) void pro_bwd_dlat_generic_kernel(ProBwdArgs a, const T *__restrict__ w0,
                                                                  const float *__restrict__ d3,
                                                                  const float *__restrict__ d1,
                                                                  const T *__restrict__ dv, T *__restrict__ d_lat) {
  dlat_element(a, w0, d3, d1, dv, d_lat, (long long)blockIdx.x * 256 + threadIdx.x);
}

// The parameters' gradients, sums over all rows:
//   dw1[h,o,i,j] = sum_rows d3[row,h,o] * u1[row - (k_ch-1-j), h, i], u1 = the conv1_seq output, recomputed from the pre-conv
//   latent (zero before the sequence start).  Unit = (head, tap j, 32 outputs o, 32 inputs i), the rows dealt to its 8
//   wavefronts 8 at a time;
//   dw0[c,jj] = sum_rows d1[row,c] * lat[row - (k_seq-1-jj), c].  Unit = 32 channels x 16 groups of rows, all taps at once;
//   d_temp[g] = sum_rows rowdot[row,g].  Unit = one column.
// One launch; each unit of the first two kinds is split over the rows (grad_splits) into workgroups whose sums go to `part` and
// are added in order by grad_reduce_kernel: a unit's chain of row blocks is what a launch of few units waits for.
// T = 1000, 4 heads of 32: dw1 37 us, dw0 21.5 and d_temp 4.5 in unsplit launches of their own.  Behind these units the launch's other
// workgroups form d_lat, which needs the same d3 and d1 and nothing of theirs (apart 7.8 + 4.3 us, together 7.9);
// generic_gradients_share.
struct GradPlan {
  int n1, s1, n0, s0, nt;     // units and splits of dw1 and dw0, d_temp's columns
  long long e1, e0;           // elements of dw1, dw0
};
constexpr int GR_NT = 512, GR_WAVES = GR_NT / 64;

static GradPlan grad_plan(const Dims &d, bool want1, bool want0, bool want_temp) {
  GradPlan p{};
  const int nt = (d.dh + 31) / 32, NH = d.Hq + d.Hk;
  p.n1 = want1 ? nt * nt * NH * d.k_ch : 0;
  p.n0 = want0 ? (d.e_q + d.e_kv + 31) / 32 : 0;
  p.s1 = want1 ? grad_splits(p.n1, d.rows()) : 1;
  p.s0 = want0 ? grad_splits(p.n0, d.rows()) : 1;
  p.nt = want_temp ? d.Hk : 0;
  p.e1 = (long long)NH * d.dh * d.dh * d.k_ch;
  p.e0 = (long long)(d.e_q + d.e_kv) * d.k_seq;
  return p;
}

template <typename T>
__device__ __forceinline__ void grad_w1_unit(const ProBwdArgs &a, const T *__restrict__ lat, const T *__restrict__ w0,
                                             const float *__restrict__ d3, T *__restrict__ dw1, float *__restrict__ part, int unit,
                                             long long r_begin, long long r_end, float (*so)[16][64]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int dh = a.dh, kc = a.k_ch, nt = (dh + 31) / 32, ks = (a.flags & CCA_CONV_SEQ) ? a.k_seq : 1;
  const int o0 = unit % (nt * nt) / nt * 32, i0 = unit % nt * 32, j = unit / (nt * nt) % kc, h = unit / (nt * nt * kc);
  const int ch0 = h < a.Hq ? h * dh : a.e_q + (h - a.Hq) * dh, ld = a.e_q + a.e_kv, back = kc - 1 - j;
  const int oc = ch0 + min(o0 + l32, dh - 1), ic = ch0 + min(i0 + l32, dh - 1);  // past the head: results not stored
  float f[4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
    f[jj] = (a.flags & CCA_CONV_SEQ) ? load_f(w0 + (long long)ic * a.k_seq + min(jj, a.k_seq - 1)) : 1.f;
  gen_f32x16 acc = zero16();
  constexpr int AHEAD = 2;  // blocks of 8 rows in flight
  for (long long b0 = r_begin + wave * 8; b0 < r_end; b0 += AHEAD * GR_WAVES * 8) {
    float x[AHEAD][4], y[AHEAD][4];
#pragma unroll
    for (int e8 = 0; e8 < AHEAD * 4; ++e8) {
      const int u = e8 / 4, e = e8 % 4;
      const long long r = b0 + u * GR_WAVES * 8 + 4 * half + e, row = r < r_end ? r : r_end - 1;
      const int t = (int)(row % a.T);
      x[u][e] = d3[row * ld + oc];
      float v = 0.f;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int dist = back + ks - 1 - jj;  // tokens back from the row
        const bool in = jj < ks && t >= dist;
        const float l = load_f(lat + (in ? row - dist : row) * a.n_lat + ic);
        v = in ? fmaf(f[jj], l, v) : v;
      }
      const bool live = r < r_end && t >= back;
      x[u][e] = live ? x[u][e] : 0.f;
      y[u][e] = live ? v : 0.f;
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u][e], y[u][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) so[wave][r][lane] = acc[r];
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 16 / GR_WAVES; ++x) {
    const int r = wave * (16 / GR_WAVES) + x, o = o0 + tile_row(r, half);
    float sum = 0.f;
#pragma unroll
    for (int y = 0; y < GR_WAVES; ++y) sum += so[y][r][lane];
    if (o < dh && i0 + l32 < dh) {
      const long long at = (((long long)h * dh + o) * dh + i0 + l32) * kc + j;
      if (part) part[at] = sum;
      else store_f(dw1 + at, sum);
    }
  }
}

template <typename T>
__device__ __forceinline__ void grad_w0_unit(const ProBwdArgs &a, const T *__restrict__ lat, const float *__restrict__ d1,
                                             T *__restrict__ dw0, float *__restrict__ part, int unit, long long r_begin,
                                             long long r_end, float (*red)[4][33]) {
  constexpr int GROUPS = GR_NT / 32;
  const int ld = a.e_q + a.e_kv, cl = threadIdx.x & 31, grp = threadIdx.x >> 5, ks = a.k_seq;
  const int c = unit * 32 + cl, cc = min(c, ld - 1);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (long long row = r_begin + grp; row < r_end; row += GROUPS) {
    const int t = (int)(row % a.T);
    const float g = d1[row * ld + cc];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int back = ks - 1 - jj;
      const bool in = jj < ks && t >= back;
      const float l = load_f(lat + (in ? row - back : row) * a.n_lat + cc);
      acc[jj] = in ? fmaf(g, l, acc[jj]) : acc[jj];
    }
  }
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) red[grp][jj][cl] = acc[jj];
  __syncthreads();
  if (grp < ks && c < ld) {  // group jj adds tap jj
    float sum = 0.f;
#pragma unroll
    for (int x = 0; x < GROUPS; ++x) sum += red[x][grp][cl];
    const long long at = (long long)c * ks + grp;
    if (part) part[at] = sum;
    else store_f(dw0 + at, sum);
  }
}

template <typename T>
__global__ __launch_bounds__(GR_NT) void pro_bwd_grads_generic_kernel(ProBwdArgs a, GradPlan p, const T *__restrict__ lat,
                                                                     const T *__restrict__ w0, const float *__restrict__ d3,
                                                                     const float *__restrict__ d1,
                                                                     const float *__restrict__ rowdot, T *__restrict__ dw1,
                                                                     T *__restrict__ dw0, float *__restrict__ dtemp,
                                                                     float *__restrict__ part, const T *__restrict__ dv,
                                                                     T *__restrict__ d_lat) {
  __shared__ union {
    float w1[GR_WAVES][16][64], w0[GR_NT / 32][4][33], sum[GR_NT];
  } sh;
  int id = blockIdx.x;
  auto rows_of = [&](int split, int splits, long long &r0, long long &r1) {
    const long long per = (a.rows + splits - 1) / splits;
    r0 = (long long)split * per < a.rows ? (long long)split * per : a.rows;
    r1 = r0 + per < a.rows ? r0 + per : a.rows;
  };
  long long r0, r1;
  if (id < p.n1 * p.s1) {
    rows_of(id / p.n1, p.s1, r0, r1);
    grad_w1_unit(a, lat, w0, d3, dw1, p.s1 > 1 ? part + id / p.n1 * p.e1 : nullptr, id % p.n1, r0, r1, sh.w1);
    return;
  }
  id -= p.n1 * p.s1;
  if (id < p.n0 * p.s0) {
    rows_of(id / p.n0, p.s0, r0, r1);
    float *const to = part + (p.s1 > 1 ? p.s1 * p.e1 : 0) + id / p.n0 * p.e0;
    grad_w0_unit(a, lat, d1, dw0, p.s0 > 1 ? to : nullptr, id % p.n0, r0, r1, sh.w0);
    return;
  }
  id -= p.n0 * p.s0;
  if (id >= p.nt) {
    dlat_element(a, w0, d3, d1, dv, d_lat, (long long)(id - p.nt) * GR_NT + threadIdx.x);
    return;
  }
  const int col = id, tid = threadIdx.x;
  float acc = 0.f;
#pragma unroll 4
  for (long long r = tid; r < a.rows; r += GR_NT) acc += rowdot[r * a.Hk + col];
  sh.sum[tid] = acc;
  __syncthreads();
  for (int s = GR_NT / 2; s > 0; s >>= 1) {
    if (tid < s) sh.sum[tid] += sh.sum[tid + s];
    __syncthreads();
  }
  if (tid == 0) dtemp[col] = sh.sum[0];
}

template <typename T>
__global__ __launch_bounds__(256) void grad_reduce_kernel(GradPlan p, const float *__restrict__ part, T *__restrict__ dw1,
                                                         T *__restrict__ dw0) {
  const long long n1 = p.s1 > 1 ? p.e1 : 0;
  long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  const bool first = id < n1;
  if (!first) {
    id -= n1;
    part += n1 * p.s1;
    if (p.s0 == 1 || id >= p.e0) return;
  }
  const long long step = first ? p.e1 : p.e0;
  float sum = 0.f;
#pragma unroll 8
  for (int s = 0; s < (first ? p.s1 : p.s0); ++s) sum += part[s * step + id];
  store_f((first ? dw1 : dw0) + id, sum);
}

// d3 | d1 | rowdot | the partial sums of the filter gradients
struct ProBwdScratch {
  size_t d1, rowdot, part, total;
};
static ProBwdScratch pro_bwd_scratch(const Dims &d) {
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  const size_t plane = up((size_t)d.rows() * (d.e_q + d.e_kv) * sizeof(float));
  const GradPlan p = grad_plan(d, d.flags & CCA_CONV_CH, d.flags & CCA_CONV_SEQ, false);
  ProBwdScratch s;
  s.d1 = plane;
  s.rowdot = 2 * plane;
  s.part = s.rowdot + up((size_t)d.rows() * d.Hk * sizeof(float));
  s.total = s.part + sizeof(float) * (size_t)((p.s1 > 1 ? p.s1 * p.e1 : 0) + (p.s0 > 1 ? p.s0 * p.e0 : 0));
  return s;
}
size_t prologue_bwd_generic_scratch_bytes(const Dims &d) { return pro_bwd_scratch(d).total; }

template <typename T>
static hipError_t prologue_bwd_generic_t(const Dims &d, const cca_weights &w, const void *lat, const void *q,
                                         const void *k, const float *rnorm, const void *d_q, const void *d_k,
                                         const void *d_v, void *d_lat, const cca_grads *gr, void *scratch,
                                         hipStream_t s) {
  ProBwdArgs a{d.T, d.Hq, d.Hk, d.dh, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, d.rows(), d.flags,
               d.rope_base};
  const ProBwdScratch L = pro_bwd_scratch(d);
  char *const sc = static_cast<char *>(scratch);
  float *const d3 = reinterpret_cast<float *>(sc), *const rowdot = reinterpret_cast<float *>(sc + L.rowdot);
  float *const d1 = (d.flags & CCA_CONV_CH) ? reinterpret_cast<float *>(sc + L.d1) : d3;
  float *const part = reinterpret_cast<float *>(sc + L.part);
  const bool want_temp = (d.flags & CCA_KEY_TEMP) && gr && gr->temp;
  const bool want1 = (d.flags & CCA_CONV_CH) && gr && gr->w_conv_ch, want0 = (d.flags & CCA_CONV_SEQ) && gr && gr->w_conv_seq;
  const int kc = (d.flags & CCA_CONV_CH) ? d.k_ch : 1, n_tok = GP_TOK + kc - 1;
  const size_t smem = sizeof(float) * ((size_t)n_tok * (d.dh + 1) + (size_t)n_tok * d.dh + GP_RED);
  auto point = [&](auto narrow_c) {
    constexpr bool NARROW = decltype(narrow_c)::value;
    if (hipError_t e = raise_lds_limit<pro_bwd_point_generic_kernel<T, NARROW>>(GP_MAX_LDS); e != hipSuccess) return e;
    return gp_launches(d.B, d.T, GP_TOK, [&](unsigned first, unsigned blocks) {
      pro_bwd_point_generic_kernel<T, NARROW><<<dim3(blocks, d.Hq + d.Hk), GP_NT, smem, s>>>(
          a, (const T *)q, (const T *)k, rnorm, w.temp, (const T *)d_q, (const T *)d_k, (const T *)w.w_conv_ch, d3, d1,
          want_temp ? rowdot : nullptr, first);
    });
  };
  hipError_t e = d.dh <= 32 ? point(std::true_type{}) : point(std::false_type{});
  if (e != hipSuccess) return e;
  const GradPlan p = grad_plan(d, want1, want0, want_temp);
  const long long units = (long long)p.n1 * p.s1 + (long long)p.n0 * p.s0 + p.nt;
  const long long n = d.rows() * d.n_lat, blocks = (n + GR_NT - 1) / GR_NT;
  const size_t w0_bytes = (size_t)(d.Hq + d.Hk) * d.dh * d.k_seq * sizeof(T);  // (read for d_lat)
  const bool share = generic_gradients_share(units + blocks) && !(want0 && overlap(gr->w_conv_seq, w0_bytes, w.w_conv_seq, w0_bytes));
  if (!share || !units)
    pro_bwd_dlat_generic_kernel<T><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a, (const T *)w.w_conv_seq, d3, d1,
                                                                              (const T *)d_v, (T *)d_lat);
  if (units)
    pro_bwd_grads_generic_kernel<T><<<(unsigned)(units + (share ? blocks : 0)), GR_NT, 0, s>>>(
        a, p, (const T *)lat, (const T *)w.w_conv_seq, d3, d1, rowdot, want1 ? (T *)gr->w_conv_ch : nullptr,
        want0 ? (T *)gr->w_conv_seq : nullptr, want_temp ? gr->temp : nullptr, part, (const T *)d_v, (T *)d_lat);
  const long long sums = (p.s1 > 1 ? p.e1 : 0) + (p.s0 > 1 ? p.e0 : 0);
  if (sums)
    grad_reduce_kernel<T><<<(unsigned)((sums + 255) / 256), 256, 0, s>>>(p, part, want1 ? (T *)gr->w_conv_ch : nullptr,
                                                                        want0 ? (T *)gr->w_conv_seq : nullptr);
  return hipGetLastError();
}

hipError_t prologue_bwd_generic(const Dims &d, const cca_weights &w, const void *lat, const void *q, const void *k,
                                const float *rnorm, const void *d_q, const void *d_k, const void *d_v, void *d_lat,
                                const cca_grads *gr, void *scratch, hipStream_t s) {
  return d.bf16 ? prologue_bwd_generic_t<bf16_t>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s)
                : prologue_bwd_generic_t<float>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s);
}

}  // namespace cca
