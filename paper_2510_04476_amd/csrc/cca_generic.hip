// Shape-generic kernels for every stage of the CCA block: fp32 or bf16 storage,
// fp32 arithmetic (the contractions on the fp32 matrix cores).  They serve the fp32
// configuration and every bf16 shape the bf16 MFMA kernels do not cover.
#include "cca_generic.h"

namespace cca {

// ---------------------------------------------------------------------------
// GEMM: C (M,N) = op(A) op(B), op(A)[m][k] = TA ? A[k*lda + m] : A[m*lda + k], op(B)[k][n] = TB ? B[n*ldb + k] : B[k*ldb + n].
// Workgroup = one 32 x 32 tile of C, the contraction dealt to its 8 wavefronts 8 terms at a time and their sums added
// through LDS in order: these products are mostly small (the fp32 configuration, odd bf16 shapes), so a walk along all of K by
// one wavefront is what they would wait for.  K is a multiple of 4 where an operand is stored along it; lda, ldb likewise.
// us, 64 x 64 tiles through LDS on the vector ALU -> this, fp32: 1000 x 192 over K = 256 31 -> 5.2, 256 x 192 over K = 1000
// tokens 132 -> 12.1, 4096 x 1536 over 2048 580 -> 341, 16384 x 1536 over 2048 2087 -> 1356 (there the operand loads, 32 rows
// apart, bound it); bf16, 16384 x 4056 over 2056 5250 -> 3800.
// ---------------------------------------------------------------------------
constexpr int GG_NT = 512, GG_WAVES = GG_NT / 64;
constexpr long long GG_GRID = 1ll << 22;  // tiles of a launch, which takes fewer than 2^32 threads in one dimension

template <typename T, bool TA, bool TB>
__global__ __launch_bounds__(GG_NT) void gemm_generic_kernel(const T *__restrict__ A, long long lda, const T *__restrict__ Bm,
                                                            long long ldb, T *__restrict__ C, long long ldc, long long M, int N,
                                                            long long K, unsigned tile0) {
  __shared__ float red[GG_WAVES][32][33];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const unsigned tiles_n = (N + 31) / 32, tile = tile0 + blockIdx.x;
  const long long m0 = (long long)(tile / tiles_n) * 32;
  const int n0 = tile % tiles_n * 32;
  const long long m = m0 + l32 < M ? m0 + l32 : M - 1;  // rows and columns past the edge feed outputs that are not stored
  const int n = n0 + l32 < N ? n0 + l32 : N - 1;
  gen_f32x16 acc = zero16();
  const long long last = K - 1;
#pragma unroll 4
  for (long long k0 = wave * 8 + 4 * half; k0 - 4 * half < K; k0 += GG_WAVES * 8) {
    float a[4], b[4];
    // terms past K: some readable value, dropped below
    if constexpr (TA) {
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = load_f(A + (k0 + i < last ? k0 + i : last) * lda + m);
    } else {
      const gen_f32x4 v = load4(A + m * lda + (k0 < K ? k0 : 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = v[i];
    }
    if constexpr (TB) {
      const gen_f32x4 v = load4(Bm + n * ldb + (k0 < K ? k0 : 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = v[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = load_f(Bm + (k0 + i < last ? k0 + i : last) * ldb + n);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = k0 + i < K;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? a[i] : 0.f, in ? b[i] : 0.f, acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][tile_row(r, half)][l32] = acc[r];
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 32 * 32 / GG_NT; ++x) {
    const int r = (tid >> 5) + x * (GG_NT / 32), c = tid & 31;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < GG_WAVES; ++w) sum += red[w][r][c];
    if (m0 + r < M && n0 + c < N) store_f(C + (m0 + r) * ldc + n0 + c, sum);
  }
}

template <typename T>
static hipError_t gemm_generic_t(const void *A, long long lda, bool ta, const void *Bm, long long ldb, bool tb, void *C,
                                 long long ldc, long long M, int N, long long K, hipStream_t s) {
  const long long tiles = (M + 31) / 32 * ((N + 31) / 32);
  if (tiles > UINT32_MAX) return hipErrorInvalidValue;  // (2^42 outputs)
  for (long long t = 0; t < tiles; t += GG_GRID) {  // one launch below 2^32 outputs; a second grid dimension cost 0.2 of 2.8 us
    const unsigned grid = (unsigned)(tiles - t < GG_GRID ? tiles - t : GG_GRID);
#define GO(TA, TB)                                                                                                          \
  gemm_generic_kernel<T, TA, TB><<<grid, GG_NT, 0, s>>>((const T *)A, lda, (const T *)Bm, ldb, (T *)C, ldc, M, N, K, (unsigned)t)
    if (ta && tb) GO(true, true);
    else if (ta) GO(true, false);
    else if (tb) GO(false, true);
    else GO(false, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
#undef GO
  return hipSuccess;
}

hipError_t gemm_generic_ex(bool bf16, const void *A, long long lda, bool ta, const void *Bm, long long ldb, bool tb,
                           void *C, long long ldc, long long M, int N, long long K, hipStream_t s) {
  return bf16 ? gemm_generic_t<bf16_t>(A, lda, ta, Bm, ldb, tb, C, ldc, M, N, K, s)
              : gemm_generic_t<float>(A, lda, ta, Bm, ldb, tb, C, ldc, M, N, K, s);
}

hipError_t gemm_generic(bool bf16, const void *A, const void *Bm, void *C, long long M, int N, int K,
                        hipStream_t s) {
  return gemm_generic_ex(bf16, A, K, false, Bm, N, false, C, N, M, N, K, s);
}

// ---------------------------------------------------------------------------
// Prologue: one workgroup per (token, head).  Heads 0..Hq-1 are query heads,
// Hq..Hq+Hk-1 key heads, Hq+Hk..Hq+2Hk-1 value heads.
// ---------------------------------------------------------------------------
struct PrologueArgs {
  int T, Hq, Hk, dh, R, e_q, e_kv, n_lat, v_half, k_seq, k_ch;
  uint32_t flags;
  float rope_base, norm_eps;
};

template <typename T>
__global__ void prologue_generic_kernel(PrologueArgs a, const T *__restrict__ lat, const T *__restrict__ w0,
                                        const T *__restrict__ w1, const float *__restrict__ temp,
                                        T *__restrict__ q, T *__restrict__ k, T *__restrict__ v,
                                        float *__restrict__ rnorm) {
  extern __shared__ float sm[];  // y0[k_ch][dh] | red[blockDim] | yrot[dh]
  const long long row = blockIdx.x;  // b*T + t
  const int t = (int)(row % a.T);
  const int head = blockIdx.y;
  const int dh = a.dh;
  const int tid = threadIdx.x;

  if (head >= a.Hq + a.Hk) {  // value head: copy, second stream delayed by one token
    const int g = head - a.Hq - a.Hk;
    for (int i = tid; i < dh; i += blockDim.x) {
      const int c = g * dh + i;  // channel within e_kv
      float val;
      if (c < a.v_half || !(a.flags & CCA_V_SHIFT))
        val = load_f(lat + row * a.n_lat + a.e_q + a.e_kv + c);
      else
        val = (t == 0) ? 0.f : load_f(lat + (row - 1) * a.n_lat + a.e_q + a.e_kv + c);
      store_f(v + row * a.e_kv + c, val);
    }
    return;
  }

  const bool is_q = head < a.Hq;
  const int ch0 = is_q ? head * dh : a.e_q + (head - a.Hq) * dh;  // first packed q|k channel of this head
  const int kc = (a.flags & CCA_CONV_CH) ? a.k_ch : 1;
  const int ks = (a.flags & CCA_CONV_SEQ) ? a.k_seq : 1;
  float *y0 = sm;                 // [kc][dh]
  float *red = sm + kc * dh;      // [blockDim.x]
  float *yrot = red + blockDim.x; // [dh]

  // conv1_seq output at the kc time steps conv2 needs (zero before the sequence start)
  for (int idx = tid; idx < kc * dh; idx += blockDim.x) {
    const int j = idx / dh, i = idx % dh;
    const int tj = t - (kc - 1) + j;
    float acc = 0.f;
    if (tj >= 0) {
      if (a.flags & CCA_CONV_SEQ) {
        for (int jj = 0; jj < ks; ++jj) {
          const int ts = tj - (ks - 1) + jj;
          if (ts >= 0)
            acc = fmaf(load_f(w0 + (long long)(ch0 + i) * ks + jj),
                       load_f(lat + (row - t + ts) * a.n_lat + ch0 + i), acc);
        }
      } else {
        acc = load_f(lat + (row - t + tj) * a.n_lat + ch0 + i);
      }
    }
    y0[idx] = acc;
  }
  __syncthreads();

  float ssq = 0.f;
  // each thread owns output channels o = tid, tid + blockDim, ...
  for (int o = tid; o < dh; o += blockDim.x) {
    float y;
    if (a.flags & CCA_CONV_CH) {
      y = 0.f;
      const T *wp = w1 + ((long long)head * dh + o) * dh * kc;
      for (int i = 0; i < dh; ++i)
        for (int j = 0; j < kc; ++j) y = fmaf(load_f(wp + i * kc + j), y0[j * dh + i], y);
    } else {
      y = y0[(kc - 1) * dh + o];
    }
    if (a.flags & CCA_QK_MEAN) {
      float m;
      if (is_q) {
        m = 0.5f * (load_f(lat + row * a.n_lat + head * dh + o) +
                    load_f(lat + row * a.n_lat + a.e_q + (head / a.R) * dh + o));
      } else {
        const int g = head - a.Hq;
        float sq = 0.f;
        for (int r = 0; r < a.R; ++r) sq += load_f(lat + row * a.n_lat + (g * a.R + r) * dh + o);
        m = 0.5f * (sq / (float)a.R + load_f(lat + row * a.n_lat + a.e_q + g * dh + o));
      }
      y += m;
    }
    yrot[o] = y;
    ssq = fmaf(y, y, ssq);
  }
  red[tid] = ssq;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  float mul = 1.f;
  if (a.flags & CCA_QK_NORM) {
    mul = sqrtf((float)dh) / sqrtf(red[0] + a.norm_eps);
    if (!is_q && (a.flags & CCA_KEY_TEMP)) mul *= expf(temp[head - a.Hq]);
  }
  if (rnorm && tid == 0) rnorm[row * (a.Hq + a.Hk) + head] = mul;
  T *dst = is_q ? q + row * a.e_q + head * dh : k + row * a.e_kv + (head - a.Hq) * dh;
  for (int o = tid; o < dh; o += blockDim.x) {
    float y = yrot[o] * mul;
    if (a.flags & CCA_ROPE) {
      const int half = dh / 2;
      int pair, partner;
      bool first;
      if (a.flags & CCA_ROPE_INTERLEAVED) {
        pair = o / 2; first = (o % 2) == 0; partner = first ? o + 1 : o - 1;
      } else {
        pair = o % half; first = o < half; partner = first ? o + half : o - half;
      }
      // angle in fp64: t * theta loses ~1e-3 rad in fp32 at t ~ 16k
      const double theta = pow((double)a.rope_base, -2.0 * (double)pair / (double)dh);
      double sn, cs;
      sincos((double)t * theta, &sn, &cs);
      const float yp = yrot[partner] * mul;
      y = first ? (y * (float)cs - yp * (float)sn) : (y * (float)cs + yp * (float)sn);
    }
    store_f(dst + o, y);
  }
}

hipError_t prologue_generic(const Dims &d, const cca_weights &w, const void *lat, void *q, void *k, void *v,
                            float *rnorm, hipStream_t s) {
  PrologueArgs a{d.T, d.Hq, d.Hk, d.dh, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, d.flags, d.rope_base,
                 d.norm_eps};
  int threads = 64;
  while (threads < d.dh && threads < 256) threads *= 2;
  const int kc = (d.flags & CCA_CONV_CH) ? d.k_ch : 1;
  size_t smem = sizeof(float) * ((size_t)kc * d.dh + threads + d.dh);
  dim3 grid((unsigned)d.rows(), d.Hq + 2 * d.Hk);
  if (d.bf16)
    prologue_generic_kernel<bf16_t><<<grid, threads, smem, s>>>(a, (const bf16_t *)lat, (const bf16_t *)w.w_conv_seq,
                                                               (const bf16_t *)w.w_conv_ch, w.temp, (bf16_t *)q,
                                                               (bf16_t *)k, (bf16_t *)v, rnorm);
  else
    prologue_generic_kernel<float><<<grid, threads, smem, s>>>(a, (const float *)lat, (const float *)w.w_conv_seq,
                                                              (const float *)w.w_conv_ch, w.temp, (float *)q,
                                                              (float *)k, (float *)v, rnorm);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Attention.  Workgroup = 32 query rows of one (batch, head); its 8 wavefronts take the 32-key tiles in turn, each with its
// own running (max, sum, accumulator), merged through LDS at the end.  Scores come out transposed (lane = query, registers =
// keys), so the row statistics are in-lane with one exchange between the half-waves and the probabilities are the second
// operand of O^T += V^T P^T as they stand.  T = 1000, 2 heads of 32, fp32: 21.5 us; one wavefront per row on the vector ALU
// took 100.
// ---------------------------------------------------------------------------
constexpr int GA_NT = 512, GA_WAVES = GA_NT / 64;

template <typename T, int DHM>
__global__ __launch_bounds__(GA_NT) void attention_generic_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                 const T *__restrict__ v, T *__restrict__ o,
                                                                 T *__restrict__ o_lo, float *__restrict__ lse, int Tn, int Hq,
                                                                 int Hk, int dh, float scale, int causal) {
  constexpr int DT = DHM / 32;
  __shared__ __attribute__((aligned(16))) float sq[32 * (DHM + 4)];
  __shared__ float sm_[GA_WAVES][32], sl[GA_WAVES][32], so[GA_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int qb = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z, g = h / (Hq / Hk);  // causal: long rows first
  const int q0 = qb * 32, t = q0 + l32;
  const T *const kb = k + ((long long)b * Tn * Hk + g) * dh, *const vb = v + ((long long)b * Tn * Hk + g) * dh;
  const long long ks = (long long)Hk * dh;
  stage_rows32<DHM>(sq, q + ((long long)b * Tn * Hq + h) * dh, (long long)Hq * dh, q0, Tn - 1, dh, [=](float x) { return x * scale; });
  __syncthreads();
  float m = -INFINITY, l = 0.f;
  gen_f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16();
  const int end = causal ? min(q0 + 32, Tn) : Tn;  // keys [0, end) matter
  for (int k0 = wave * 32; k0 < end; k0 += GA_WAVES * 32) {
    const gen_f32x16 s = dot_tile<DHM>(kb + min(k0 + l32, Tn - 1) * ks, sq + l32 * (DHM + 4), dh, half, [](float x) { return x; });
    const bool mixed = k0 + 32 > Tn || (causal && k0 + 31 > q0);
    float w[16], mx = m;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + tile_row(r, half);
      w[r] = key < Tn && (!causal || key <= t) ? s[r] : -INFINITY;
      mx = fmaxf(mx, w[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float ref = mx == -INFINITY ? 0.f : mx;  // a row whose scores so far are all -inf has no maximum yet
    const float corr = expf(m - ref);              // 0 on the first tile
    l *= corr;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      w[r] = expf(w[r] - ref);
      l += w[r];
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[dt][r] *= corr;
    add_outer<DT, T>(acc, w, [=](int x) { return vb + min(k0 + x, Tn - 1) * ks; }, dh, lane, mixed);
    m = mx;
  }
  l += __shfl_xor(l, 32);  // each half-wave has summed half of the keys
  if (half == 0) sm_[wave][l32] = m, sl[wave][l32] = l;
  __syncthreads();
  float M = -INFINITY, L = 0.f, f[GA_WAVES];  // of query l32, the same for every wavefront
#pragma unroll
  for (int x = 0; x < GA_WAVES; ++x) M = fmaxf(M, sm_[x][l32]);
#pragma unroll
  for (int x = 0; x < GA_WAVES; ++x) {
    f[x] = sm_[x][l32] == -INFINITY ? 0.f : expf(sm_[x][l32] - M);
    L += sl[x][l32] * f[x];
  }
  const float inv = 1.f / L;
  const long long orow = (((long long)b * Tn + t) * Hq + h) * dh;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    if (dt > 0) __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) so[wave][r][lane] = acc[dt][r];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 16 / GA_WAVES; ++x) {
      const int r = wave * (16 / GA_WAVES) + x, ch = 32 * dt + tile_row(r, half);
      float sum = 0.f;
#pragma unroll
      for (int y = 0; y < GA_WAVES; ++y) sum += f[y] == 0.f ? 0.f : so[y][r][lane] * f[y];
      if (t < Tn && ch < dh) {
        store_f(o + orow + ch, sum * inv);
        if (o_lo) store_f(o_lo + orow + ch, sum * inv - load_f(o + orow + ch));  // what the rounding dropped
      }
    }
  }
  if (lse && wave == 0 && half == 0 && t < Tn) lse[((long long)b * Hq + h) * Tn + t] = M + logf(L);
}

template <typename T>
static hipError_t attention_generic_t(const Dims &d, const void *q, const void *k, const void *v, void *o,
                                      void *o_lo, float *lse, hipStream_t s) {
  dim3 grid((d.T + 31) / 32, d.Hq, d.B);
  const int causal = (d.flags & CCA_CAUSAL) ? 1 : 0;
#define LAUNCH(DH)                                                                                      \
  attention_generic_kernel<T, DH><<<grid, GA_NT, 0, s>>>((const T *)q, (const T *)k, (const T *)v, (T *)o, (T *)o_lo, lse, d.T, \
                                                      d.Hq, d.Hk, d.dh, d.scale, causal)
  if (d.dh <= 32) LAUNCH(32);
  else if (d.dh <= 64) LAUNCH(64);
  else if (d.dh <= 128) LAUNCH(128);
  else LAUNCH(256);
#undef LAUNCH
  return hipGetLastError();
}

hipError_t attention_generic(const Dims &d, const void *q, const void *k, const void *v, void *o, void *o_lo,
                             float *lse, hipStream_t s) {
  // fp32 storage rounds nothing away: no low part
  return d.bf16 ? attention_generic_t<bf16_t>(d, q, k, v, o, o_lo, lse, s)
                : attention_generic_t<float>(d, q, k, v, o, nullptr, lse, s);
}

}  // namespace cca
