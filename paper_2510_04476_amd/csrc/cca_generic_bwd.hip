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
template <typename T>
__global__ __launch_bounds__(256) void delta_generic_kernel(const T *__restrict__ dO, const T *__restrict__ O,
                                                           const T *__restrict__ OLO, float *__restrict__ delta,
                                                           long long n_rows, int Tn, int Hq, int dh) {
  const long long row = (long long)blockIdx.x * 256 + threadIdx.x;  // (b*T + t)*Hq + h
  if (row >= n_rows) return;
  float acc = 0.f;
  for (int i = 0; i < dh; ++i)
    acc = fmaf(load_f(dO + row * dh + i), load_f(O + row * dh + i) + (OLO ? load_f(OLO + row * dh + i) : 0.f), acc);
  const long long bt = row / Hq;
  const int h = (int)(row % Hq);
  delta[((bt / Tn) * Hq + h) * Tn + (bt % Tn)] = acc;
}

// log2-unit score against the forward MFMA kernel's own rounding of q (q * scale * log2(e) rounded to bf16):
// used when that kernel produced lse, so that the recomputed probabilities are exactly its probabilities
__device__ __forceinline__ float q_log2_rounded(float q, float c) { return bf16_to_f32(f32_to_bf16(q * c)); }
constexpr float kLog2e = 1.44269504088896340736f;

constexpr int GB_NT = 512, GB_WAVES = GB_NT / 64;

// Sums of the wavefronts' accumulators, in wavefront order: out(channel, column l32, sum) once per element of the tile
template <int DT, typename F>
__device__ __forceinline__ void sum_wavefronts(const gen_f32x16 (&acc)[DT], float (*so)[16][64], int wave, int lane, F &&out) {
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) so[wave][r][lane] = acc[dt][r];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 16 / GB_WAVES; ++x) {
      const int r = wave * (16 / GB_WAVES) + x;
      float sum = 0.f;
#pragma unroll
      for (int y = 0; y < GB_WAVES; ++y) sum += so[y][r][lane];
      out(32 * dt + tile_row(r, lane >> 5), sum);
    }
  }
}

// Workgroup = 32 query rows of one head, the key tiles dealt to its 8 wavefronts; S^T and dP^T with one query per lane, dS^T
// is the second operand of dQ^T += K^T dS^T as it stands.  T = 1000, 2 heads of 32, fp32: 26 us; one wavefront per row on
// the vector ALU took 117.
template <typename T, int DHM>
__global__ __launch_bounds__(GB_NT) void attn_bwd_dq_generic_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                   const T *__restrict__ v, const T *__restrict__ dO,
                                                                   const float *__restrict__ lse,
                                                                   const float *__restrict__ delta, T *__restrict__ dq, int Tn,
                                                                   int Hq, int Hk, int dh, float scale, int causal,
                                                                   int q_rounded) {
  constexpr int DT = DHM / 32;
  __shared__ __attribute__((aligned(16))) float sq[32 * (DHM + 4)], sd[32 * (DHM + 4)];
  __shared__ float so[GB_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int qb = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z, g = h / (Hq / Hk);
  const int q0 = qb * 32, t = q0 + l32, tc = min(t, Tn - 1);
  const T *const kb = k + ((long long)b * Tn * Hk + g) * dh, *const vb = v + ((long long)b * Tn * Hk + g) * dh;
  const long long ks = (long long)Hk * dh, qs = (long long)Hq * dh, q_off = ((long long)b * Tn * Hq + h) * dh;
  stage_rows32<DHM>(sq, q + q_off, qs, q0, Tn - 1, dh,
                    [=](float x) { return q_rounded ? q_log2_rounded(x, scale * kLog2e) : x * scale; });
  stage_rows32<DHM>(sd, dO + q_off, qs, q0, Tn - 1, dh, [](float x) { return x; });
  const float L = lse[((long long)b * Hq + h) * Tn + tc] * (q_rounded ? kLog2e : 1.f);
  const float Dl = delta[((long long)b * Hq + h) * Tn + tc];
  __syncthreads();
  gen_f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16();
  const int end = causal ? min(q0 + 32, Tn) : Tn;
  auto same = [](float x) { return x; };
  for (int k0 = wave * 32; k0 < end; k0 += GB_WAVES * 32) {
    const long long krow = min(k0 + l32, Tn - 1) * ks;
    const gen_f32x16 s = dot_tile<DHM>(kb + krow, sq + l32 * (DHM + 4), dh, half, same);
    const gen_f32x16 dp = dot_tile<DHM>(vb + krow, sd + l32 * (DHM + 4), dh, half, same);
    const bool mixed = k0 + 32 > Tn || (causal && k0 + 31 > q0);
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + tile_row(r, half);
      const float x = (q_rounded ? exp2f(s[r] - L) : expf(s[r] - L)) * (dp[r] - Dl);
      w[r] = key < Tn && (!causal || key <= t) ? x : 0.f;
    }
    add_outer<DT, T>(acc, w, [=](int x) { return kb + min(k0 + x, Tn - 1) * ks; }, dh, lane, mixed);
  }
  sum_wavefronts(acc, so, wave, lane, [&](int ch, float sum) {
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
__global__ __launch_bounds__(GB_NT) void attn_bwd_dkv_generic_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                    const T *__restrict__ v, const T *__restrict__ dO,
                                                                    const float *__restrict__ lse,
                                                                    const float *__restrict__ delta, T *__restrict__ dk,
                                                                    T *__restrict__ dv, int Tn, int Hq, int Hk, int dh,
                                                                    float scale, int causal, int q_rounded) {
  constexpr int DT = DHM / 32;
  __shared__ __attribute__((aligned(16))) float sk[32 * (DHM + 4)], sv[32 * (DHM + 4)];
  __shared__ float so[GB_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int k0 = blockIdx.x * 32, g = blockIdx.y, b = blockIdx.z, R = Hq / Hk, key = k0 + l32;
  const long long ks = (long long)Hk * dh, qs = (long long)Hq * dh, k_off = ((long long)b * Tn * Hk + g) * dh;
  stage_rows32<DHM>(sk, k + k_off, ks, k0, Tn - 1, dh, [=](float x) { return x * (q_rounded ? 1.f : scale); });
  stage_rows32<DHM>(sv, v + k_off, ks, k0, Tn - 1, dh, [](float x) { return x; });
  __syncthreads();
  gen_f32x16 ak[WHICH & 1 ? DT : 1], av[WHICH & 2 ? DT : 1];
#pragma unroll
  for (int dt = 0; dt < (WHICH & 1 ? DT : 1); ++dt) ak[dt] = zero16();
#pragma unroll
  for (int dt = 0; dt < (WHICH & 2 ? DT : 1); ++dt) av[dt] = zero16();
  const int first = causal ? k0 / 32 : 0, tiles = (Tn + 31) / 32 - first;
  for (int idx = wave; idx < R * tiles; idx += GB_WAVES) {
    const int h = g * R + idx / tiles, t0 = (first + idx % tiles) * 32;
    const T *const qb = q + ((long long)b * Tn * Hq + h) * dh, *const db = dO + ((long long)b * Tn * Hq + h) * dh;
    const long long qrow = min(t0 + l32, Tn - 1) * qs, st = ((long long)b * Hq + h) * Tn;
    const gen_f32x16 s = dot_tile<DHM>(qb + qrow, sk + l32 * (DHM + 4), dh, half,
                                       [=](float x) { return q_rounded ? q_log2_rounded(x, scale * kLog2e) : x; });
    gen_f32x16 dp;
    if constexpr (WHICH & 1) dp = dot_tile<DHM>(db + qrow, sv + l32 * (DHM + 4), dh, half, [](float x) { return x; });
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
    if constexpr (WHICH & 2) add_outer<DT, T>(av, p, [=](int x) { return db + min(t0 + x, Tn - 1) * qs; }, dh, lane, mixed);
    if constexpr (WHICH & 1) add_outer<DT, T>(ak, ds, [=](int x) { return qb + min(t0 + x, Tn - 1) * qs; }, dh, lane, mixed);
  }
  if constexpr (WHICH & 1)
    sum_wavefronts(ak, so, wave, lane, [&](int ch, float sum) {
      if (key < Tn && ch < dh) store_f(dk + k_off + key * ks + ch, sum);
    });
  if constexpr (WHICH & 2)
    sum_wavefronts(av, so, wave, lane, [&](int ch, float sum) {
      if (key < Tn && ch < dh) store_f(dv + k_off + key * ks + ch, sum);
    });
}

template <typename T>
static hipError_t attention_bwd_generic_t(const Dims &d, const void *q, const void *k, const void *v, const void *o,
                                          const void *o_lo, const float *lse, const void *d_o, void *d_q, void *d_k, void *d_v,
                                          float *delta, hipStream_t s) {
  const long long n_rows = d.rows() * d.Hq;
  delta_generic_kernel<T><<<(unsigned)((n_rows + 255) / 256), 256, 0, s>>>((const T *)d_o, (const T *)o, (const T *)o_lo, delta, n_rows,
                                                                          d.T, d.Hq, d.dh);
  const int causal = (d.flags & CCA_CAUSAL) ? 1 : 0;
  const int q_rounded = attention_mfma_supported(d) ? 1 : 0;  // lse then comes from the MFMA forward kernel
  const dim3 gq((d.T + 31) / 32, d.Hq, d.B), gk((d.T + 31) / 32, d.Hk, d.B);
#define DQ(DH)                                                                                                          \
  attn_bwd_dq_generic_kernel<T, DH><<<gq, GB_NT, 0, s>>>((const T *)q, (const T *)k, (const T *)v, (const T *)d_o, lse, \
                                                         delta, (T *)d_q, d.T, d.Hq, d.Hk, d.dh, d.scale, causal, q_rounded)
#define DKV(DH, W)                                                                                                      \
  attn_bwd_dkv_generic_kernel<T, DH, W><<<gk, GB_NT, 0, s>>>((const T *)q, (const T *)k, (const T *)v, (const T *)d_o,  \
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

// RoPE^T, norm / temperature backward.  One workgroup per (token, q or k head).
//   y = x * mul with mul = sqrt(d_h) beta / |x|:  dx = mul * (dy - y <y,dy> / (d_h beta^2)).
template <typename T>
__global__ void pro_bwd_point_generic_kernel(ProBwdArgs a, const T *__restrict__ q, const T *__restrict__ k,
                                             const float *__restrict__ rnorm, const float *__restrict__ temp,
                                             const T *__restrict__ dq, const T *__restrict__ dk,
                                             float *__restrict__ d3, float *__restrict__ rowdot) {
  extern __shared__ float sm[];  // tmp[dh] | red[blockDim]
  const long long row = blockIdx.x;
  const int t = (int)(row % a.T);
  const int head = blockIdx.y, dh = a.dh, tid = threadIdx.x;
  const bool is_q = head < a.Hq;
  const int g = head - a.Hq;
  const T *y5 = is_q ? q + (row * a.Hq + head) * dh : k + (row * a.Hk + g) * dh;
  const T *dy5 = is_q ? dq + (row * a.Hq + head) * dh : dk + (row * a.Hk + g) * dh;
  float *tmp = sm, *red = sm + dh;
  float part = 0.f;
  for (int o = tid; o < dh; o += blockDim.x) part = fmaf(load_f(y5 + o), load_f(dy5 + o), part);
  red[tid] = part;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  const float dot = red[0];
  float mul = 1.f, c = 0.f;
  if (a.flags & CCA_QK_NORM) {
    mul = rnorm[row * (a.Hq + a.Hk) + head];
    const float beta2 = (!is_q && (a.flags & CCA_KEY_TEMP)) ? expf(2.f * temp[g]) : 1.f;
    c = dot / ((float)dh * beta2);
  }
  if (!is_q && rowdot && tid == 0) rowdot[row * a.Hk + g] = dot;
  for (int o = tid; o < dh; o += blockDim.x) tmp[o] = load_f(dy5 + o) - load_f(y5 + o) * c;
  __syncthreads();
  const int ch0 = is_q ? head * dh : a.e_q + g * dh;
  for (int o = tid; o < dh; o += blockDim.x) {
    float val = tmp[o];
    if (a.flags & CCA_ROPE) {
      const int half = dh / 2;
      int pair, partner;
      bool first;
      if (a.flags & CCA_ROPE_INTERLEAVED) {
        pair = o / 2; first = (o % 2) == 0; partner = first ? o + 1 : o - 1;
      } else {
        pair = o % half; first = o < half; partner = first ? o + half : o - half;
      }
      const double theta = pow((double)a.rope_base, -2.0 * (double)pair / (double)dh);
      double sn, cs;
      sincos((double)t * theta, &sn, &cs);
      // forward: (a, b) -> (a c - b s, b c + a s); adjoint rotates back
      val = first ? (val * (float)cs + tmp[partner] * (float)sn) : (val * (float)cs - tmp[partner] * (float)sn);
    }
    d3[row * (a.e_q + a.e_kv) + ch0 + o] = val * mul;
  }
}

// out[col] = sum over rows of src[row*ncol + col]; one workgroup per column, fixed summation order
__global__ __launch_bounds__(256) void column_sum_kernel(const float *__restrict__ src, long long rows, int ncol,
                                                        float *__restrict__ out) {
  __shared__ float red[256];
  const int col = blockIdx.x, tid = threadIdx.x;
  float acc = 0.f;
  for (long long r = tid; r < rows; r += 256) acc += src[r * ncol + col];
  red[tid] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) out[col] = red[0];
}

// conv2_seq+ch transposed: d1[t,h,i] = sum_j sum_o w1[h,o,i,j] d3[t + (k_ch-1-j), h, o] within the sequence
template <typename T>
__global__ void pro_bwd_convch_generic_kernel(ProBwdArgs a, const T *__restrict__ w1, const float *__restrict__ d3,
                                              float *__restrict__ d1) {
  extern __shared__ float sm[];  // d3 rows of the k_ch taps: [kc][dh]
  const long long row = blockIdx.x;
  const int t = (int)(row % a.T);
  const int head = blockIdx.y, dh = a.dh, kc = a.k_ch, tid = threadIdx.x;
  const int ch0 = head < a.Hq ? head * dh : a.e_q + (head - a.Hq) * dh;
  const int ld = a.e_q + a.e_kv;
  for (int idx = tid; idx < kc * dh; idx += blockDim.x) {
    const int j = idx / dh, o = idx % dh;
    const int fwd = kc - 1 - j;
    sm[idx] = (t + fwd < a.T) ? d3[(row + fwd) * ld + ch0 + o] : 0.f;
  }
  __syncthreads();
  for (int i = tid; i < dh; i += blockDim.x) {
    float acc = 0.f;
    for (int o = 0; o < dh; ++o) {
      const T *wp = w1 + (((long long)head * dh + o) * dh + i) * kc;
      for (int j = 0; j < kc; ++j) acc = fmaf(load_f(wp + j), sm[j * dh + o], acc);
    }
    d1[row * ld + ch0 + i] = acc;
  }
}

// conv1_seq transposed + qk-mean adjoint + value-shift adjoint: one thread per element of d_lat
template <typename T>
__global__ __launch_bounds__(256) void pro_bwd_dlat_generic_kernel(ProBwdArgs a, const T *__restrict__ w0,
                                                                  const float *__restrict__ d3,
                                                                  const float *__restrict__ d1,
                                                                  const T *__restrict__ dv, T *__restrict__ d_lat) {
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
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

// dw1[h,o,i,j] = sum_rows d3[row,h,o] * u1[row - (k_ch-1-j), h, i], u1 = the conv1_seq output, recomputed from the pre-conv
// latent (zero before the sequence start).  Workgroup = (head, tap j, 32 outputs o, 32 inputs i), the rows dealt to its 8
// wavefronts 8 at a time.  T = 1000, 4 heads of 32, k_ch = 2, fp32: 37 us; one thread per filter element took 535.
template <typename T>
__global__ __launch_bounds__(GB_NT) void pro_bwd_dw1_generic_kernel(ProBwdArgs a, const T *__restrict__ lat,
                                                                   const T *__restrict__ w0, const float *__restrict__ d3,
                                                                   T *__restrict__ dw1) {
  __shared__ float so[GB_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int dh = a.dh, kc = a.k_ch, nt = (dh + 31) / 32, ks = (a.flags & CCA_CONV_SEQ) ? a.k_seq : 1;
  const int h = blockIdx.y, j = blockIdx.z, o0 = blockIdx.x / nt * 32, i0 = blockIdx.x % nt * 32;
  const int ch0 = h < a.Hq ? h * dh : a.e_q + (h - a.Hq) * dh, ld = a.e_q + a.e_kv, back = kc - 1 - j;
  const int oc = ch0 + min(o0 + l32, dh - 1), ic = ch0 + min(i0 + l32, dh - 1);  // past the head: results not stored
  float f[4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
    f[jj] = (a.flags & CCA_CONV_SEQ) ? load_f(w0 + (long long)ic * a.k_seq + min(jj, a.k_seq - 1)) : 1.f;
  gen_f32x16 acc[1] = {zero16()};
#pragma unroll 2
  for (long long r0 = wave * 8 + 4 * half; r0 - 4 * half < a.rows; r0 += GB_WAVES * 8) {
    float x[4], y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const long long row = r0 + e < a.rows ? r0 + e : a.rows - 1;
      const int t = (int)(row % a.T);
      x[e] = d3[row * ld + oc];
      float u = 0.f;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int dist = back + ks - 1 - jj;  // tokens back from the row
        const bool in = jj < ks && t >= dist;
        const float l = load_f(lat + (in ? row - dist : row) * a.n_lat + ic);
        u = in ? fmaf(f[jj], l, u) : u;
      }
      const bool live = r0 + e < a.rows && t >= back;
      x[e] = live ? x[e] : 0.f;
      y[e] = live ? u : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], acc[0], 0, 0, 0);
  }
  sum_wavefronts(acc, so, wave, lane, [&](int o, float sum) {
    if (o0 + o < dh && i0 + l32 < dh) store_f(dw1 + (((long long)h * dh + o0 + o) * dh + i0 + l32) * kc + j, sum);
  });
}

// dw0[c,jj] = sum_rows d1[row,c] * lat[row - (k_seq-1-jj), c].  Workgroup = 32 channels x 32 groups of rows, all taps at
// once; the groups' sums are added through LDS in order.  T = 1000, 128 channels, 2 taps: 21.5 us; one thread per element
// took 288.
template <typename T>
__global__ __launch_bounds__(1024) void pro_bwd_dw0_generic_kernel(ProBwdArgs a, const T *__restrict__ lat,
                                                                  const float *__restrict__ d1, T *__restrict__ dw0) {
  __shared__ float red[32][4][33];
  const int ld = a.e_q + a.e_kv, cl = threadIdx.x & 31, grp = threadIdx.x >> 5, ks = a.k_seq;
  const int c = blockIdx.x * 32 + cl, cc = min(c, ld - 1);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (long long row = grp; row < a.rows; row += 32) {
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
    for (int x = 0; x < 32; ++x) sum += red[x][grp][cl];
    store_f(dw0 + (long long)c * ks + grp, sum);
  }
}

size_t prologue_bwd_generic_scratch_bytes(const Dims &d) {
  const size_t plane = (size_t)d.rows() * (d.e_q + d.e_kv) * sizeof(float);
  return 2 * ((plane + 255) / 256 * 256) + (size_t)d.rows() * d.Hk * sizeof(float);
}

template <typename T>
static hipError_t prologue_bwd_generic_t(const Dims &d, const cca_weights &w, const void *lat, const void *q,
                                         const void *k, const float *rnorm, const void *d_q, const void *d_k,
                                         const void *d_v, void *d_lat, const cca_grads *gr, void *scratch,
                                         hipStream_t s) {
  ProBwdArgs a{d.T, d.Hq, d.Hk, d.dh, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, d.rows(), d.flags,
               d.rope_base};
  const size_t plane = ((size_t)d.rows() * (d.e_q + d.e_kv) * sizeof(float) + 255) / 256 * 256;
  float *d3 = reinterpret_cast<float *>(scratch);
  float *d1 = reinterpret_cast<float *>(static_cast<char *>(scratch) + plane);
  float *rowdot = reinterpret_cast<float *>(static_cast<char *>(scratch) + 2 * plane);
  const bool want_temp = (d.flags & CCA_KEY_TEMP) && gr && gr->temp;
  int threads = 64;
  while (threads < d.dh && threads < 256) threads *= 2;
  const int NH = d.Hq + d.Hk;
  dim3 grid_rh((unsigned)d.rows(), NH);
  pro_bwd_point_generic_kernel<T><<<grid_rh, threads, sizeof(float) * (d.dh + threads), s>>>(
      a, (const T *)q, (const T *)k, rnorm, w.temp, (const T *)d_q, (const T *)d_k, d3, want_temp ? rowdot : nullptr);
  if (want_temp) column_sum_kernel<<<d.Hk, 256, 0, s>>>(rowdot, d.rows(), d.Hk, gr->temp);
  if (d.flags & CCA_CONV_CH)
    pro_bwd_convch_generic_kernel<T><<<grid_rh, threads, sizeof(float) * d.k_ch * d.dh, s>>>(
        a, (const T *)w.w_conv_ch, d3, d1);
  else
    d1 = d3;
  const long long n = d.rows() * d.n_lat;
  pro_bwd_dlat_generic_kernel<T><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a, (const T *)w.w_conv_seq, d3, d1,
                                                                            (const T *)d_v, (T *)d_lat);
  if ((d.flags & CCA_CONV_CH) && gr && gr->w_conv_ch) {
    const int nt = (d.dh + 31) / 32;
    pro_bwd_dw1_generic_kernel<T><<<dim3(nt * nt, NH, d.k_ch), GB_NT, 0, s>>>(a, (const T *)lat, (const T *)w.w_conv_seq, d3,
                                                                             (T *)gr->w_conv_ch);
  }
  if ((d.flags & CCA_CONV_SEQ) && gr && gr->w_conv_seq)
    pro_bwd_dw0_generic_kernel<T><<<(d.e_q + d.e_kv + 31) / 32, 1024, 0, s>>>(a, (const T *)lat, d1, (T *)gr->w_conv_seq);
  return hipGetLastError();
}

hipError_t prologue_bwd_generic(const Dims &d, const cca_weights &w, const void *lat, const void *q, const void *k,
                                const float *rnorm, const void *d_q, const void *d_k, const void *d_v, void *d_lat,
                                const cca_grads *gr, void *scratch, hipStream_t s) {
  return d.bf16 ? prologue_bwd_generic_t<bf16_t>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s)
                : prologue_bwd_generic_t<float>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s);
}

}  // namespace cca
