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

template <typename T>
struct GenericProduct {
  const T *A;
  long long lda;
  const T *B;
  long long ldb;
  T *C;
  long long ldc, M;
  int N;
  long long K;
};
typedef float GgSums[GG_WAVES][32][33];

template <typename T, bool TA, bool TB, int AHEAD>
__device__ __forceinline__ void gemm_generic_tile(const T *__restrict__ A, long long lda, const T *__restrict__ Bm, long long ldb,
                                                  T *__restrict__ C, long long ldc, long long M, int N, long long K, unsigned tile,
                                                  GgSums &red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const unsigned tiles_n = (N + 31) / 32;
  const long long m0 = (long long)(tile / tiles_n) * 32;
  const int n0 = tile % tiles_n * 32;
  const long long m = m0 + l32 < M ? m0 + l32 : M - 1;  // rows and columns past the edge feed outputs that are not stored
  const int n = n0 + l32 < N ? n0 + l32 : N - 1;
  gen_f32x16 acc = zero16();
  const long long last = K - 1;
  // AHEAD blocks of 8 terms in flight (the compiler does not unroll a loop of MFMAs whose count it does not know): generic_product_looks_ahead
  for (long long b0 = wave * 8; b0 < K; b0 += AHEAD * GG_WAVES * 8) {
    float a[AHEAD][4], b[AHEAD][4];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (u > 0 && b0 + u * GG_WAVES * 8 >= K) break;
      const long long k0 = b0 + u * GG_WAVES * 8 + 4 * half;
      // terms past K: some readable value, dropped below
      if constexpr (TA) {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[u][i] = load_f(A + (k0 + i < last ? k0 + i : last) * lda + m);
      } else {
        const gen_f32x4 v = load4(A + m * lda + (k0 < K ? k0 : 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) a[u][i] = v[i];
      }
      if constexpr (TB) {
        const gen_f32x4 v = load4(Bm + n * ldb + (k0 < K ? k0 : 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) b[u][i] = v[i];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) b[u][i] = load_f(Bm + (k0 + i < last ? k0 + i : last) * ldb + n);
      }
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (u > 0 && b0 + u * GG_WAVES * 8 >= K) break;
      const long long k0 = b0 + u * GG_WAVES * 8 + 4 * half;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = k0 + i < K;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? a[u][i] : 0.f, in ? b[u][i] : 0.f, acc, 0, 0, 0);
      }
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

template <typename T, bool TA, bool TB, int AHEAD>
__global__ __launch_bounds__(GG_NT) void gemm_generic_kernel(GenericProduct<T> p, unsigned tile0) {
  __shared__ GgSums red;
  gemm_generic_tile<T, TA, TB, AHEAD>(p.A, p.lda, p.B, p.ldb, p.C, p.ldc, p.M, p.N, p.K, tile0 + blockIdx.x, red);
}

// A projection's two adjoints, d_W = A^T d_C (its tiles first: the longer chains) and d_A = d_C W^T: independent, and where the tiles of
// both are on the chip at once (generic_products_share) one launch takes as long as the longer of the two.
template <typename T, int AHEAD_W, int AHEAD_A>
__global__ __launch_bounds__(GG_NT) void gemm_generic_pair_kernel(GenericProduct<T> w, GenericProduct<T> a, unsigned tiles_w) {
  __shared__ GgSums red;
  if (blockIdx.x < tiles_w) gemm_generic_tile<T, true, false, AHEAD_W>(w.A, w.lda, w.B, w.ldb, w.C, w.ldc, w.M, w.N, w.K, blockIdx.x, red);
  else gemm_generic_tile<T, false, true, AHEAD_A>(a.A, a.lda, a.B, a.ldb, a.C, a.ldc, a.M, a.N, a.K, blockIdx.x - tiles_w, red);
}

template <typename T>
static hipError_t gemm_generic_pair_t(const GenericProduct<T> &w, const GenericProduct<T> &a, hipStream_t s) {
  const long long tiles_w = (w.M + 31) / 32 * ((w.N + 31) / 32), tiles_a = (a.M + 31) / 32 * ((a.N + 31) / 32);
  const bool ahead_w = generic_product_looks_ahead(tiles_w, w.K), ahead_a = generic_product_looks_ahead(tiles_a, a.K);
  (ahead_w ? (ahead_a ? gemm_generic_pair_kernel<T, 4, 4> : gemm_generic_pair_kernel<T, 4, 1>)
           : (ahead_a ? gemm_generic_pair_kernel<T, 1, 4> : gemm_generic_pair_kernel<T, 1, 1>))<<<(unsigned)(tiles_w + tiles_a), GG_NT, 0, s>>>(
      w, a, (unsigned)tiles_w);
  return hipGetLastError();
}

bool gemm_generic_pair_supported(long long rows, int n_in, int n_out) {
  const long long rt = (rows + 31) / 32, in = (n_in + 31) / 32, out = (n_out + 31) / 32;
  return generic_products_share(in * out + rt * in);
}

hipError_t gemm_generic_pair(bool bf16, const void *d_C, const void *W, void *d_A, const void *A, void *d_W, long long rows, int n_in,
                             int n_out, hipStream_t s) {
  auto go = [&](auto zero) {
    typedef decltype(zero) T;
    return gemm_generic_pair_t<T>({(const T *)A, n_in, (const T *)d_C, n_out, (T *)d_W, n_out, n_in, n_out, rows},
                                  {(const T *)d_C, n_out, (const T *)W, n_out, (T *)d_A, n_in, rows, n_in, n_out}, s);
  };
  return bf16 ? go(bf16_t{}) : go(float{});
}

template <typename T>
static hipError_t gemm_generic_t(const void *A, long long lda, bool ta, const void *Bm, long long ldb, bool tb, void *C,
                                 long long ldc, long long M, int N, long long K, hipStream_t s) {
  const long long tiles = (M + 31) / 32 * ((N + 31) / 32);
  if (tiles > UINT32_MAX) return hipErrorInvalidValue;  // (2^42 outputs)
  for (long long t = 0; t < tiles; t += GG_GRID) {  // one launch below 2^32 outputs; a second grid dimension cost 0.2 of 2.8 us
    const unsigned grid = (unsigned)(tiles - t < GG_GRID ? tiles - t : GG_GRID);
#define GO(TA, TB)                                                                                                        \
  (generic_product_looks_ahead(tiles, K) ? gemm_generic_kernel<T, TA, TB, 4> : gemm_generic_kernel<T, TA, TB, 1>)<<<grid, GG_NT, 0, s>>>(              \
      GenericProduct<T>{(const T *)A, lda, (const T *)Bm, ldb, (T *)C, ldc, M, N, K}, (unsigned)t)
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
// Prologue: one workgroup per head and TOK = 32 or 8 tokens of a sequence (generic_prologue_takes_8).  Heads 0..Hq-1 are query heads,
// Hq..Hq+Hk-1 key heads, Hq+Hk..Hq+2Hk-1 value heads.  conv2_seq+ch is a product on the fp32 matrix cores (outputs x tokens),
// its terms (input, tap) dealt to the four wavefronts, so a filter is read once per workgroup.  What bounds it is the chain of its
// loads and, on few workgroups, the instructions of one wavefront per SIMD: loads of several channels and of the next outputs' filter rows in
// flight, no division in a loop.  A narrow head (d_h <= 16) keeps fewer in flight, for more wavefronts to a CU.
// us, a workgroup per token on the vector ALU -> this: fp32, 1000 tokens, 2 / 2 heads of 32 21.4 -> 7.4; 500, 2 / 2 x 64 36.2 -> 10.4;
// 4096, 4 / 2 x 128 1422 -> 45; bf16, 64 tokens, 2 / 2 x 40 12.0 -> 9.0; x 200 46.9 -> 34.4; with k_ch = 1 25.5 -> 24.1.
// ---------------------------------------------------------------------------
struct PrologueArgs {
  int T, Hq, Hk, dh, R, e_q, e_kv, n_lat, v_half, k_seq, k_ch;
  uint32_t flags;
  float rope_base, norm_eps;
};

template <typename T, int TOK, bool NARROW>
__global__ __launch_bounds__(GP_NT) void prologue_generic_kernel(PrologueArgs a, const T *__restrict__ lat, const T *__restrict__ w0,
                                                                const T *__restrict__ w1, const float *__restrict__ temp,
                                                                T *__restrict__ q, T *__restrict__ k, T *__restrict__ v,
                                                                float *__restrict__ rnorm, unsigned block0) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int head = blockIdx.y, dh = a.dh, tid = threadIdx.x;
  constexpr int LANES = GP_NT / TOK, U = NARROW ? 2 : 4;  // lanes of a token; channels of a lane whose loads are in flight together
  const unsigned tiles = (a.T + TOK - 1) / TOK, block = block0 + blockIdx.x;
  const long long row0 = (long long)(block / tiles) * a.T;  // the sequence's first row
  const int t0 = block % tiles * TOK, n_tok = min(TOK, a.T - t0);

  if (head >= a.Hq + a.Hk) {  // value head: copy, second stream delayed by one token
    const int g = head - a.Hq - a.Hk;
    for (int id = tid; id < n_tok * dh; id += GP_NT) {
      const int t = t0 + id / dh, c = g * dh + id % dh;  // channel within e_kv
      const bool late = c >= a.v_half && (a.flags & CCA_V_SHIFT);
      const long long row = row0 + t;
      const float val = late && t == 0 ? 0.f : load_f(lat + (late ? row - 1 : row) * a.n_lat + a.e_q + a.e_kv + c);
      store_f(v + row * a.e_kv + c, val);
    }
    return;
  }

  const bool is_q = head < a.Hq;
  const int ch0 = is_q ? head * dh : a.e_q + (head - a.Hq) * dh;  // first packed q|k channel of this head
  const int kc = (a.flags & CCA_CONV_CH) ? a.k_ch : 1;
  const int ks = (a.flags & CCA_CONV_SEQ) ? a.k_seq : 1;
  const int rows = TOK + kc - 1, ldy = dh + 1;
  float *const y0 = sm;                                    // [rows][ldy]: conv1_seq output from token t0 - (kc - 1) on
  float *const z = y0 + rows * ldy;                        // [TOK][ldy]
  float *const sa = z + TOK * ldy, *const red = sa + TOK * dh;  // cos, sin | sums of the wavefronts

  // conv1_seq output at the time steps conv2 needs (zero before the sequence start)
  // The kc - 1 tokens before the first are dealt to all threads.
  const int x = tid / LANES, ln = tid % LANES, t = t0 + x;
  const long long row = row0 + min(t, a.T - 1);
  const bool mean = a.flags & CCA_QK_MEAN;  // z starts as the mean of the row's streams
  const T *const lat_row = lat + row * a.n_lat, *const other = lat_row + (is_q ? a.e_q + head / a.R * dh : (head - a.Hq) * a.R * dh);
  const int n_other = is_q ? 1 : a.R;  // key heads: their query heads
  gp_taps(ks, [&](auto taps_c) __attribute__((always_inline)) {
    constexpr int TAPS = decltype(taps_c)::value;
    const bool conv = a.flags & CCA_CONV_SEQ;
    struct Token {  // the rows its taps read: those outside the sequence are read from the nearest and dropped
      const T *row[TAPS];
      bool in[TAPS];
    };
    auto token = [&](int tj) __attribute__((always_inline)) {
      Token k;
#pragma unroll
      for (int jj = 0; jj < TAPS; ++jj) {
        const int ts = tj - (TAPS - 1) + jj;
        k.row[jj] = lat + (row0 + min(max(ts, 0), a.T - 1)) * a.n_lat + ch0;
        k.in[jj] = ts >= 0 && tj < a.T;
      }
      return k;
    };
    const T *const f0 = conv ? w0 + (long long)ch0 * TAPS : w0;
    auto element = [&](const Token &k, int i) __attribute__((always_inline)) {
      float v[TAPS], f[TAPS], acc = 0.f;
#pragma unroll
      for (int jj = 0; jj < TAPS; ++jj) v[jj] = load_f(k.row[jj] + i), f[jj] = conv ? load_f(f0 + i * TAPS + jj) : 1.f;
#pragma unroll
      for (int jj = 0; jj < TAPS; ++jj) acc = k.in[jj] ? (conv ? fmaf(f[jj], v[jj], acc) : v[jj]) : acc;
      return acc;
    };
    const Token now = token(t0 + x);
    float *const to = y0 + (kc - 1 + x) * ldy;
    for (int i0 = ln; i0 < dh; i0 += U * LANES) {  // (past the head its last channel again)
      float y[U], own[U], sum[U];
      int at[U];
#pragma unroll
      for (int u = 0; u < U; ++u) sum[u] = 0.f, at[u] = min(i0 + u * LANES, dh - 1);
#pragma unroll
      for (int u = 0; u < U; ++u) own[u] = load_f(lat_row + ch0 + at[u]);
      if (mean) {
#pragma unroll 4
        for (int r = 0; r < n_other; ++r)
#pragma unroll
          for (int u = 0; u < U; ++u) sum[u] += load_f(other + r * dh + at[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) y[u] = element(now, at[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u * LANES < dh) {
          to[at[u]] = y[u];
          z[x * ldy + at[u]] = mean ? 0.5f * (is_q ? own[u] + sum[u] : sum[u] / (float)a.R + own[u]) : 0.f;
        }
    }
    for (int i = tid; i < (kc - 1) * dh; i += GP_NT) {
      const int r = (i >= dh) + (i >= 2 * dh);
      y0[r * ldy + i - r * dh] = element(token(t0 - (kc - 1) + r), i - r * dh);
    }
  });
  if (a.flags & CCA_ROPE) rope_angles(sa, a.rope_base, dh, t0, TOK);
  __syncthreads();
  if (a.flags & CCA_CONV_CH) {
    const T *const wh = w1 + (long long)head * dh * dh * kc;
    gp_taps(kc, [&](auto taps_c) __attribute__((always_inline)) {
      constexpr int TAPS = decltype(taps_c)::value;
      const int column = min(tid & 31, TOK - 1);  // (8 tokens: the other columns repeat the last)
      gp_product<TAPS, NARROW ? 2 : 8>(
          dh, dh, red, [&](int o, int n) { return raw4(wh + o * dh * TAPS + n); }, [&](int c, int j) { return y0[(column + j) * ldy + c]; },
          [&](int o, int tok, float sum) {
            if (tok < TOK) z[tok * ldy + o] = mean ? sum + z[tok * ldy + o] : sum;
          });
    });
  } else {
    for (int o = ln; o < dh; o += LANES) z[x * ldy + o] = mean ? y0[x * ldy + o] + z[x * ldy + o] : y0[x * ldy + o];
  }
  __syncthreads();
  float ssq = 0.f;
#pragma unroll 4
  for (int o = ln; o < dh; o += LANES) ssq = fmaf(z[x * ldy + o], z[x * ldy + o], ssq);
#pragma unroll
  for (int e = 1; e < LANES; e *= 2) ssq += __shfl_xor(ssq, e);
  float mul = 1.f;
  if (a.flags & CCA_QK_NORM) {
    mul = sqrtf((float)dh) / sqrtf(ssq + a.norm_eps);
    if (!is_q && (a.flags & CCA_KEY_TEMP)) mul *= expf(temp[head - a.Hq]);
  }
  if (rnorm && ln == 0 && t < a.T) rnorm[row * (a.Hq + a.Hk) + head] = mul;
  __syncthreads();
  if (t >= a.T) return;
  T *const dst = is_q ? q + row * a.e_q + head * dh : k + row * a.e_kv + (head - a.Hq) * dh;
  if (a.flags & CCA_ROPE) {
    const int half = dh / 2;
    const bool il = a.flags & CCA_ROPE_INTERLEAVED;
#pragma unroll 2
    for (int p = ln; p < half; p += LANES) {
      const int first = il ? 2 * p : p, second = il ? 2 * p + 1 : p + half;
      const float cs = sa[2 * (x * half + p)], sn = sa[2 * (x * half + p) + 1];
      const float u = z[x * ldy + first] * mul, w = z[x * ldy + second] * mul;
      store_f(dst + first, u * cs - w * sn);
      store_f(dst + second, w * cs + u * sn);
    }
  } else {
    for (int o = ln; o < dh; o += LANES) store_f(dst + o, z[x * ldy + o] * mul);
  }
}

hipError_t prologue_generic(const Dims &d, const cca_weights &w, const void *lat, void *q, void *k, void *v,
                            float *rnorm, hipStream_t s) {
  PrologueArgs a{d.T, d.Hq, d.Hk, d.dh, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, d.flags, d.rope_base,
                 d.norm_eps};
  const int kc = (d.flags & CCA_CONV_CH) ? d.k_ch : 1;
  auto run = [&](auto tok_c, auto narrow_c, auto t) {
    using T = decltype(t);
    constexpr int TOK = decltype(tok_c)::value;
    constexpr bool NARROW = decltype(narrow_c)::value;
    const size_t smem = sizeof(float) * ((size_t)(2 * TOK + kc - 1) * (d.dh + 1) + (size_t)TOK * d.dh + GP_RED);
    if (hipError_t e = raise_lds_limit<prologue_generic_kernel<T, TOK, NARROW>>(GP_MAX_LDS); e != hipSuccess) return e;
    return gp_launches(d.B, d.T, TOK, [&](unsigned first, unsigned blocks) {
      prologue_generic_kernel<T, TOK, NARROW><<<dim3(blocks, d.Hq + 2 * d.Hk), GP_NT, smem, s>>>(
          a, (const T *)lat, (const T *)w.w_conv_seq, (const T *)w.w_conv_ch, w.temp, (T *)q, (T *)k, (T *)v, rnorm, first);
    });
  };
  auto run_narrow = [&](auto tok_c, auto t) { return d.dh <= 16 ? run(tok_c, std::true_type{}, t) : run(tok_c, std::false_type{}, t); };
  auto run_tok = [&](auto t) {
    return generic_prologue_takes_8(d.B, d.T, d.Hq + d.Hk) ? run_narrow(std::integral_constant<int, 8>{}, t)
                                                               : run_narrow(std::integral_constant<int, 32>{}, t);
  };
  return d.bf16 ? run_tok(bf16_t{}) : run_tok(float{});
}

// ---------------------------------------------------------------------------
// Attention.  Workgroup = 32 query rows of one (batch, head); its 8 wavefronts take the 32-key tiles in turn, each with its
// own running (max, sum, accumulator), merged through LDS at the end.  Scores come out transposed (lane = query, registers =
// keys), so the row statistics are in-lane with one exchange between the half-waves and the probabilities are the second
// operand of O^T += V^T P^T as they stand.  What bounds a small grid is the chain of steps of a wavefront, hence a form with 16 rows
// and up to 16 wavefronts to a workgroup; a large one is bound by the K and V rows loaded per product (generic_attention_rows).
// ---------------------------------------------------------------------------
template <typename T, int DHM>
__global__ __launch_bounds__(G32_NT) void attention_generic32_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                 const T *__restrict__ v, T *__restrict__ o,
                                                                 T *__restrict__ o_lo, float *__restrict__ lse, int Tn, int Hq,
                                                                 int Hk, int dh, float scale, int causal) {
  constexpr int DT = DHM / 32;
  __shared__ __attribute__((aligned(16))) float sq[32 * (DHM + 4)];
  __shared__ float sm_[G32_WAVES][32], sl[G32_WAVES][32], so[G32_WAVES][16][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int qb = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z, g = h / (Hq / Hk);  // causal: long rows first
  const int q0 = qb * 32, t = q0 + l32;
  const T *const kb = k + ((long long)b * Tn * Hk + g) * dh, *const vb = v + ((long long)b * Tn * Hk + g) * dh;
  const long long ks = (long long)Hk * dh;
  stage_rows<DHM, 32>(sq, q + ((long long)b * Tn * Hq + h) * dh, (long long)Hq * dh, q0, Tn - 1, dh, [=](float x) { return x * scale; });
  __syncthreads();
  float m = -INFINITY, l = 0.f;
  gen_f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16();
  const int end = causal ? min(q0 + 32, Tn) : Tn;  // keys [0, end) matter
  for (int k0 = wave * 32; k0 < end; k0 += G32_WAVES * 32) {
    const gen_f32x16 s = dot_tile32<DHM>(kb + min(k0 + l32, Tn - 1) * ks, sq + l32 * (DHM + 4), dh, half, [](float x) { return x; });
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
    add_outer32<DT, T>(acc, w, [=](int x) { return vb + min(k0 + x, Tn - 1) * ks; }, dh, lane, mixed);
    m = mx;
  }
  l += __shfl_xor(l, 32);  // each half-wave has summed half of the keys
  if (half == 0) sm_[wave][l32] = m, sl[wave][l32] = l;
  __syncthreads();
  float M = -INFINITY, L = 0.f, f[G32_WAVES];  // of query l32, the same for every wavefront
#pragma unroll
  for (int x = 0; x < G32_WAVES; ++x) M = fmaxf(M, sm_[x][l32]);
#pragma unroll
  for (int x = 0; x < G32_WAVES; ++x) {
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
    for (int x = 0; x < 16 / G32_WAVES; ++x) {
      const int r = wave * (16 / G32_WAVES) + x, ch = 32 * dt + tile_row(r, half);
      float sum = 0.f;
#pragma unroll
      for (int y = 0; y < G32_WAVES; ++y) sum += f[y] == 0.f ? 0.f : so[y][r][lane] * f[y];
      if (t < Tn && ch < dh) {
        store_f(o + orow + ch, sum * inv);
        if (o_lo) store_f(o_lo + orow + ch, sum * inv - load_f(o + orow + ch));  // what the rounding dropped
      }
    }
  }
  if (lse && wave == 0 && half == 0 && t < Tn) lse[((long long)b * Hq + h) * Tn + t] = M + logf(L);
}

// The same over 16 rows: NT / 64 wavefronts take the 32-key steps, two 16 x 16 tiles each.
template <typename T, int DHM, int NT>
__global__ __launch_bounds__(NT) void attention_generic16_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                const T *__restrict__ v, T *__restrict__ o, T *__restrict__ o_lo,
                                                                float *__restrict__ lse, int Tn, int Hq, int Hk, int dh,
                                                                float scale, int causal) {
  constexpr int DT = DHM / 16, WAVES = NT / 64;
  __shared__ __attribute__((aligned(16))) float sq[16 * (DHM + 4)];
  __shared__ float sm_[WAVES][16], sl[WAVES][16];
  __shared__ G16Partial so[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
  const int qb = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z, g = h / (Hq / Hk);  // causal: long rows first
  const int q0 = qb * 16, t = q0 + l16;
  const T *const kb = k + ((long long)b * Tn * Hk + g) * dh, *const vb = v + ((long long)b * Tn * Hk + g) * dh;
  const long long ks = (long long)Hk * dh;
  stage_rows<DHM, 16>(sq, q + ((long long)b * Tn * Hq + h) * dh, (long long)Hq * dh, q0, Tn - 1, dh, [=](float x) { return x * scale; });
  __syncthreads();
  float m = -INFINITY, l = 0.f;
  gen_f32x4 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
  const int end = causal ? min(q0 + 16, Tn) : Tn;  // keys [0, end) matter
  for (int k0 = wave * 32; k0 < end; k0 += WAVES * 32) {
    const bool mixed = k0 + 32 > Tn || (causal && k0 + 31 > q0);
    gen_f32x4 w[2];
    float mx = m;
#pragma unroll
    for (int x = 0; x < 2; ++x)
      w[x] = dot_tile16<DHM>(kb + min(k0 + 16 * x + l16, Tn - 1) * ks, sq + l16 * (DHM + 4), dh, grp, [](float y) { return y; });
#pragma unroll
    for (int x = 0; x < 2; ++x) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = k0 + 16 * x + 4 * grp + r;
        w[x][r] = key < Tn && (!causal || key <= t) ? w[x][r] : -INFINITY;
        mx = fmaxf(mx, w[x][r]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float ref = mx == -INFINITY ? 0.f : mx;  // a row whose scores so far are all -inf has no maximum yet
    const float corr = expf(m - ref);              // 0 on the first step
    l *= corr;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[dt][r] *= corr;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        w[x][r] = expf(w[x][r] - ref);
        l += w[x][r];
      }
      add_outer16<DT, T>(acc, w[x], [=](int y) { return vb + min(k0 + 16 * x + y, Tn - 1) * ks; }, dh, lane, mixed);
    }
    m = mx;
  }
  l += __shfl_xor(l, 16);  // each lane group has summed a quarter of the keys
  l += __shfl_xor(l, 32);
  if (grp == 0) sm_[wave][l16] = m, sl[wave][l16] = l;
  __syncthreads();
  float M = -INFINITY, L = 0.f;  // of query l16, the same for every wavefront
#pragma unroll
  for (int x = 0; x < WAVES; ++x) M = fmaxf(M, sm_[x][l16]);
  auto weight = [&](int x) { return sm_[x][l16] == -INFINITY ? 0.f : expf(sm_[x][l16] - M); };
#pragma unroll
  for (int x = 0; x < WAVES; ++x) L += sl[x][l16] * weight(x);
  const float inv = 1.f / L;
  const long long orow = (((long long)b * Tn + t) * Hq + h) * dh;
  sum_wavefronts16<WAVES>(acc, so, weight, [&](int ch, float sum) {
    if (t < Tn && ch < dh) {
      store_f(o + orow + ch, sum * inv);
      if (o_lo) store_f(o_lo + orow + ch, sum * inv - load_f(o + orow + ch));  // what the rounding dropped
    }
  });
  if (lse && wave == 0 && grp == 0 && t < Tn) lse[((long long)b * Hq + h) * Tn + t] = M + logf(L);
}

template <typename T>
static hipError_t attention_generic_t(const Dims &d, const void *q, const void *k, const void *v, void *o,
                                      void *o_lo, float *lse, hipStream_t s) {
  const int causal = (d.flags & CCA_CAUSAL) ? 1 : 0;
  auto go = [&](auto kernel, int threads, int rows) {
    kernel<<<dim3((d.T + rows - 1) / rows, d.Hq, d.B), threads, 0, s>>>((const T *)q, (const T *)k, (const T *)v, (T *)o, (T *)o_lo,
                                                                        lse, d.T, d.Hq, d.Hk, d.dh, d.scale, causal);
    return hipGetLastError();
  };
  const GenericRows form = generic_attention_rows((long long)d.B * d.Hq, d.T, d.dh, causal);
#define FORMS(DH)                                                                                        \
  (form == GR_32               ? go(attention_generic32_kernel<T, DH>, G32_NT, 32)                       \
   : form == GR_16_WIDE        ? go(attention_generic16_kernel<T, DH, G16_NT<DH>>, G16_NT<DH>, 16)       \
                               : go(attention_generic16_kernel<T, DH, 512>, 512, 16))
  return d.dh <= 32 ? FORMS(32) : d.dh <= 64 ? FORMS(64) : d.dh <= 128 ? FORMS(128) : FORMS(256);
#undef FORMS
}

hipError_t attention_generic(const Dims &d, const void *q, const void *k, const void *v, void *o, void *o_lo,
                             float *lse, hipStream_t s) {
  // fp32 storage rounds nothing away: no low part
  return d.bf16 ? attention_generic_t<bf16_t>(d, q, k, v, o, o_lo, lse, s)
                : attention_generic_t<float>(d, q, k, v, o, nullptr, lse, s);
}

}  // namespace cca
