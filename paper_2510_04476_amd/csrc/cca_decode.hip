// One autoregressive decode step of the block (Sec. 2.2; the cost table's KV-cache and decode-FLOPs columns):
// what is cached per token are the latent keys and values AFTER every transform, exactly what the prefill
// prologue writes, so prefill and decode share one cache.  By causality the result of a step at position t is
// row t of the whole block applied to the tokens 0..t; that identity is what the tests check.
//
// Per step and sequence:  lat = x W_down (small GEMM);  conv / qk-mean / value-shift / norm / temperature / RoPE
// for the ONE new token from a ring of latent rows (the D-1 earlier rows the D = k_seq + k_ch - 1 taps reach, one
// at least for the value shift, plus the new row, which the projection writes straight into its slot);  k, v appended to the cache;  attention of the new query against the cache;  out = o W_O.
// The attention is bound by reading the cache (2 * len * H_k * d_h elements per sequence), so the key range is
// split over workgroups (each serves all R query heads of one KV head: the cache is read once per group, not
// once per query head) and a second kernel merges the partial softmax states in a fixed order.
#include <type_traits>

#include "cca_internal.h"

namespace cca {

namespace {

constexpr int R_MAX = 8;       // query heads of a group handled per pass over the cache
constexpr int DEC_WAVES = 4;   // wavefronts per workgroup of the attention kernel
constexpr int MAX_SPLITS = 32;

struct DecArgs {
  int B, S, Hq, Hk, dh, R, e_q, e_kv, n_lat, v_half, k_seq, k_ch, P, pos;
  uint32_t flags;
  float rope_base, scale, norm_eps;
  const int *pos_seq;  // per-sequence positions (device, B entries) or null: every sequence at `pos`
};

// Position of sequence b's new token.  With per-sequence positions `pos` is the largest one the host vouched for
// (it is below the cache capacity); a value outside [0, pos] is clamped into that range, so whatever the array
// holds no cache or ring access can leave its allocation.
__device__ __forceinline__ int seq_pos(const DecArgs &a, int b) {
  if (!a.pos_seq) return a.pos;
  const int p = a.pos_seq[b];
  return p < 0 ? 0 : (p > a.pos ? a.pos : p);
}

// N consecutive elements as one vector load (N * sizeof(T) bytes, aligned by construction: head offsets and
// channel offsets are multiples of N elements)
template <int N>
__device__ __forceinline__ void load_vec(const float *p, float *dst) {
  typedef float fv __attribute__((ext_vector_type(N)));
  if constexpr (N == 1) {
    dst[0] = *p;
  } else if constexpr (N == 8) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 a = *reinterpret_cast<const f4 *>(p), b = *reinterpret_cast<const f4 *>(p + 4);
    dst[0] = a.x; dst[1] = a.y; dst[2] = a.z; dst[3] = a.w; dst[4] = b.x; dst[5] = b.y; dst[6] = b.z; dst[7] = b.w;
  } else {
    const fv v = *reinterpret_cast<const fv *>(p);
#pragma unroll
    for (int i = 0; i < N; ++i) dst[i] = v[i];
  }
}
template <int N>
__device__ __forceinline__ void load_vec(const bf16_t *p, float *dst) {
  if constexpr (N == 1) {
    dst[0] = bf16_to_f32(*p);
  } else {
    typedef uint32_t uv __attribute__((ext_vector_type(N / 2)));
    if constexpr (N == 2) {
      const uint32_t w = *reinterpret_cast<const uint32_t *>(p);
      dst[0] = __uint_as_float(w << 16);
      dst[1] = __uint_as_float(w & 0xffff0000u);
    } else {
      const uv v = *reinterpret_cast<const uv *>(p);
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        dst[2 * i] = __uint_as_float(v[i] << 16);
        dst[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
      }
    }
  }
}

// 8 consecutive elements as they lie in memory, converted when they are used: a conversion right behind the load would wait
// for it
template <typename T>
struct Raw8;
template <>
struct Raw8<bf16_t> {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  u4 v;
  __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const u4 *>(p); }
  __device__ __forceinline__ Raw8 keep(bool on) const {  // zeros where not `on`
    Raw8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = on ? v[i] : 0u;
    return r;
  }
  __device__ __forceinline__ float get(int e) const {
    const uint32_t w = v[e >> 1];
    return __uint_as_float((e & 1) ? w & 0xffff0000u : w << 16);
  }
};
template <>
struct Raw8<float> {
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = *reinterpret_cast<const f4 *>(p);
    b = *reinterpret_cast<const f4 *>(p + 4);
  }
  __device__ __forceinline__ Raw8 keep(bool on) const {
    Raw8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r.a[i] = on ? a[i] : 0.f, r.b[i] = on ? b[i] : 0.f;
    return r;
  }
  __device__ __forceinline__ float get(int e) const { return e < 4 ? a[e & 3] : b[e & 3]; }
};

// latent row of token `tok` of sequence b: ring slot tok % P (the new token's row is written there by the projection)
template <typename T>
__device__ __forceinline__ const T *lat_row(const DecArgs &a, const T *hist, int b, int tok) {
  return hist + ((long long)b * a.P + tok % a.P) * a.n_lat;
}

constexpr int MAX_PARTS = 8;
// The new token's latent row: the sum, in index order, of `nparts` fp32 rows that the down-projection left (bf16; (nparts, B, N_lat)),
// rounded to the storage type - or the row itself, where the projection wrote it to its ring slot (fp32: one part).
// Requests and sums are apart so that a caller can request everything before it waits for anything, and no load hides behind a
// condition: a value that two branches load is waited for where they meet (NP >= nparts; addresses past the last part repeat it, the value
// is dropped).  What bounds a small step is this chain of latencies.  Whole step, E = 2048, 8 query and 2 KV heads of 128, before ->
// now: one sequence of 200 tokens 23.4 -> 22.1 us, 32 of 2000 43.5 -> 42.2, 256 of 2000 191.5 -> 186.4 (with eight requests whatever
// nparts is, 96 sequences and more lost 2 ... 6 %).
template <typename T, int NP>
struct NewRow {
  const float *part;    // this sequence's row of the first part
  long long stride;     // from one part to the next
  int nparts;
  template <int N>
  __device__ __forceinline__ void request(const int (&ch)[N], float (&v)[N][NP]) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int s = 0; s < NP; ++s) v[i][s] = part[min(s, nparts - 1) * stride + ch[i]];
  }
  __device__ __forceinline__ float value(const float (&v)[NP]) const {
    float a = 0.f;
#pragma unroll
    for (int s = 0; s < NP; ++s) a += s < nparts ? v[s] : 0.f;
    T r;
    store_f(&r, a);
    return load_f(&r);
  }
  __device__ __forceinline__ float at(int ch) const {
    float v[1][NP];
    request({ch}, v);
    return value(v[0]);
  }
};

// ---------------------------------------------------------------------------
// Transforms of the new token: one workgroup per (sequence, head); heads 0..Hq-1 query, then Hk key, then Hk value.
// What bounds it is latency, so every load that does not depend on something else is requested before the first is used:
// the filter rows of the first outputs, the head's own row and its partners, the rows the taps reach.  The sums of these
// follow, and behind them the rotary angles (fp64, on d_h / 2 threads), which therefore run under none of the loads.  LPO =
// 8 or 16 lanes share an output channel's filter row (128 adjacent bytes per load: the memory pipeline works per cache
// line) and add their parts on the vector ALU; and no load hides behind a condition (each would be waited for). At B = 32,
// d_h = 128: 14.2 us including the sum of the down-projection's parts, against 12.7 + 4.9 us for one thread per filter row
// behind a kernel that added them; at B = 1 7.7 against 8.6 + 3.5.  CH = 16- (fp32: 32-) byte chunks of a filter row per
// lane.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

template <typename T, int CH, int LPO, int NP>
__global__ __launch_bounds__(512) void decode_prologue_kernel(DecArgs a, T *__restrict__ hist, const float *__restrict__ part,
                                                             int nparts, const T *__restrict__ w0, const T *__restrict__ w1,
                                                             const float *__restrict__ temp, float *__restrict__ q_new,
                                                             T *__restrict__ k_cache, T *__restrict__ v_cache) {
  extern __shared__ __attribute__((aligned(16))) float sm[];  // y0[dh][k_ch] | yrot[dh] | cos[dh/2] | sin[dh/2]
  const int b = blockIdx.x, head = blockIdx.y, dh = a.dh, tid = threadIdx.x, t = seq_pos(a, b);
  const long long crow = (long long)b * a.S + t;  // cache row of the new token
  T *const slot = hist + ((long long)b * a.P + t % a.P) * a.n_lat;
  // (fp32: the projection wrote the rows into the ring itself)
  const NewRow<T, NP> now{std::is_same<T, float>::value ? reinterpret_cast<const float *>(slot) : part + (long long)b * a.n_lat,
                      (long long)a.B * a.n_lat, nparts};
  constexpr bool keep = !std::is_same<T, float>::value;  // the new row goes into the ring here

  if (head >= a.Hq + a.Hk) {  // value head: second stream delayed by one token
    const int g = head - a.Hq - a.Hk, v0 = a.e_q + a.e_kv;
    const T *prev = t > 0 ? lat_row(a, hist, b, t - 1) + v0 : nullptr;
    for (int i = tid; i < dh; i += blockDim.x) {
      const int c = g * dh + i;
      const float cur = now.at(v0 + c);
      if (keep) store_f(slot + v0 + c, cur);
      float val;
      if (c < a.v_half || !(a.flags & CCA_V_SHIFT)) val = cur;
      else val = prev ? load_f(prev + c) : 0.f;
      store_f(v_cache + crow * a.e_kv + c, val);
    }
    return;
  }

  const bool is_q = head < a.Hq;
  const int ch0 = is_q ? head * dh : a.e_q + (head - a.Hq) * dh;
  const int kc = (a.flags & CCA_CONV_CH) ? a.k_ch : 1;
  const int ks = (a.flags & CCA_CONV_SEQ) ? a.k_seq : 1;
  float *y0 = sm, *yrot = sm + kc * dh, *cos_t = yrot + dh, *sin_t = cos_t + dh / 2;

  // the first outputs' filter rows: lane lo of an output takes chunks lo, lo + LPO, ...
  const int lo = tid % LPO, opp = blockDim.x / LPO, nch = dh * kc / 8;  // outputs per pass; chunks per filter row
  Raw8<T> wv[2][CH];
  auto load_w = [&](int o, Raw8<T> (&w)[CH]) {
    const T *wp = w1 + ((long long)head * dh + min(o, dh - 1)) * dh * kc;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int c = j * LPO + lo;
      w[j].load(wp + min(c, nch - 1) * 8);  // chunks past the row repeat its last one; dropped below
    }
  };
  const bool conv = a.flags & CCA_CONV_CH;
  if (conv) load_w(tid / LPO, wv[0]);

  // The new row's channels, one output per thread (d_h <= 256 <= threads; the others repeat the last one): the head's own
  // and the qk-mean's other stream.
  // They are requested here and summed behind the requests for the rows the taps reach: one memory latency for both.
  const int oc = min(tid, dh - 1), q0 = (head - a.Hq) * a.R * dh + oc;  // (q0: a key head's first query channel)
  float v_own[1][NP], v_oth[4][NP];
  now.request({ch0 + oc}, v_own);
  const int kv = a.e_q + (head / a.R) * dh + oc;  // a query head's other stream
  now.request({is_q ? kv : q0, is_q ? kv : q0 + min(1, a.R - 1) * dh, is_q ? kv : q0 + min(2, a.R - 1) * dh,
               is_q ? kv : q0 + min(3, a.R - 1) * dh}, v_oth);
  // conv1_seq outputs at the k_ch times conv2 needs, of which one channel and time each: the part from earlier tokens here,
  // the new token's term (always the last tap) once its row is shared
  const int n_y0 = kc * dh;  // <= 1024: two per thread at most
  const bool seq = a.flags & CCA_CONV_SEQ;
  const T *const f0p = seq ? w0 : hist;  // without the convolution: any readable row, the value is dropped
  float y_old[2], w_new[2];
  T xs_[2][4], f0_[2][4];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int idx = min(tid + u * (int)blockDim.x, n_y0 - 1), j = idx / dh, i = idx % dh, tj = t - (kc - 1) + j;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {  // rows outside the sequence (or still to come) are read from some slot and dropped
      const int ts = tj - (ks - 1) + jj;
      xs_[u][jj] = lat_row(a, hist, b, max(ts, 0))[ch0 + i];
      f0_[u][jj] = f0p[(long long)(ch0 + i) * ks + min(jj, ks - 1)];
    }
  }
  __builtin_amdgcn_sched_barrier(0);  // every request stands before the first use
  const float own = now.value(v_own[0]);
  float mean;
  if (is_q) {
    mean = 0.5f * (own + now.value(v_oth[0]));
  } else {
    float sq = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) sq += u < a.R ? now.value(v_oth[u]) : 0.f;
    for (int r = 4; r < a.R; r += 4) {
      float x[4][NP];
      now.request({q0 + r * dh, q0 + min(r + 1, a.R - 1) * dh, q0 + min(r + 2, a.R - 1) * dh, q0 + min(r + 3, a.R - 1) * dh}, x);
#pragma unroll
      for (int u = 0; u < 4; ++u) sq += r + u < a.R ? now.value(x[u]) : 0.f;
    }
    mean = 0.5f * (sq / (float)a.R + own);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int idx = min(tid + u * (int)blockDim.x, n_y0 - 1), j = idx / dh, tj = t - (kc - 1) + j;
    float xs[4], f0[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) xs[jj] = load_f(&xs_[u][jj]), f0[jj] = load_f(&f0_[u][jj]);
    float acc = 0.f;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int ts = tj - (ks - 1) + jj;
      f0[jj] = seq ? f0[jj] : 1.f;
      acc = jj < ks && ts >= 0 && ts < t ? fmaf(f0[jj], xs[jj], acc) : acc;
    }
    y_old[u] = acc;
    w_new[u] = f0[3];  // the last tap (min above)
  }
  if (a.flags & CCA_ROPE) {
    for (int i = tid; i < dh / 2; i += blockDim.x) {
      const double theta = pow((double)a.rope_base, -2.0 * (double)i / (double)dh);
      double sn, cs;
      sincos((double)t * theta, &sn, &cs);
      cos_t[i] = (float)cs;
      sin_t[i] = (float)sn;
    }
  }
  if (tid < dh) {
    yrot[tid] = own;  // shared for the taps; the outputs replace it
    if (keep) store_f(slot + ch0 + tid, own);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int idx = tid + u * blockDim.x;
    if (idx >= n_y0) continue;
    const int j = idx / dh, i = idx % dh;
    // in the order the channel filter stores its (input channel, tap) pairs
    y0[i * kc + j] = j == kc - 1 ? fmaf(w_new[u], yrot[i], y_old[u]) : y_old[u];
  }
  __syncthreads();
  if (tid < dh) yrot[tid] = (a.flags & CCA_QK_MEAN) ? mean : 0.f;
  __syncthreads();

  if (conv) {
    float yv[CH][8];  // this lane's chunks of y0, zero past the row
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int c = j * LPO + lo;
#pragma unroll
      for (int e = 0; e < 8; ++e) yv[j][e] = c < nch ? y0[c * 8 + e] : 0.f;
    }
    auto pass = [&](int o, const Raw8<T> (&w)[CH]) {
      float y = 0.f;
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        const Raw8<T> wj = w[j].keep(j * LPO + lo < nch);  // (a weight may be infinite: zero times it would not be zero)
#pragma unroll
        for (int e = 0; e < 8; ++e) y = fmaf(wj.get(e), yv[j][e], y);
      }
      y = dpp_add<0xB1>(y);   // quad_perm [1,0,3,2]
      y = dpp_add<0x4E>(y);   // quad_perm [2,3,0,1]
      y = dpp_add<0x141>(y);  // row_half_mirror: 8 lanes hold their sum
      if constexpr (LPO == 16) y = dpp_add<0x140>(y);  // row_mirror
      if (lo == 0 && o < dh) yrot[o] += y;
    };
    for (int o = tid / LPO; o < dh; o += 2 * opp) {  // (the lanes of an output agree on the conditions)
      if (o + opp < dh) load_w(o + opp, wv[1]);
      pass(o, wv[0]);
      if (o + opp < dh) {
        if (o + 2 * opp < dh) load_w(o + 2 * opp, wv[0]);
        pass(o + opp, wv[1]);
      }
    }
  } else {
    for (int o = tid; o < dh; o += blockDim.x) yrot[o] += y0[o * kc + (kc - 1)];
  }
  __syncthreads();
  float mul = 1.f;
  if (a.flags & CCA_QK_NORM) {  // every wavefront forms the sum by itself: no further barrier
    float ssq = 0.f;
    for (int o = tid & 63; o < dh; o += 64) ssq = fmaf(yrot[o], yrot[o], ssq);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ssq += __shfl_xor(ssq, off);
    mul = sqrtf((float)dh) / sqrtf(ssq + a.norm_eps);
    if (!is_q && (a.flags & CCA_KEY_TEMP)) mul *= expf(temp[head - a.Hq]);
  }
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
      const float yp = yrot[partner] * mul;
      y = first ? (y * cos_t[pair] - yp * sin_t[pair]) : (y * cos_t[pair] + yp * sin_t[pair]);
    }
    if (is_q) {
      // the query goes through the storage type once, as the prefill's q does, then stays fp32 for the dot products
      T tmp;
      store_f(&tmp, y);
      q_new[((long long)b * a.Hq + head) * dh + o] = load_f(&tmp);
    } else {
      store_f(k_cache + crow * a.e_kv + (head - a.Hq) * dh + o, y);
    }
  }
}

// ---------------------------------------------------------------------------
// Attention of the new queries against the cache.  Workgroup = (sequence, KV head, split of the key range), 4
// wavefronts, each walking its share of the split 64 keys at a time: for the scores a lane owns ONE key (its row
// of K, 8 elements per load) and all R query heads; for P V a lane owns CPL adjacent channels and the probabilities come
// from LDS.  Online softmax per wavefront in log2 units; the wavefronts' states are merged through LDS.
// Partial result per (sequence, query head, split): m, l, o[d_h] in fp32.
// ---------------------------------------------------------------------------
// CPL = channels per lane in the P V phase (d_h <= 64 * CPL); DHC = d_h when it is one of the common widths (the
// loops over channels then unroll and their loads are all in flight together), 0 for any other multiple of 8.
template <typename T, int CPL, int DHC>
__global__ __launch_bounds__(DEC_WAVES * 64) void decode_attn_kernel(DecArgs a, const float *__restrict__ q_new,
                                                                    const T *__restrict__ k_cache,
                                                                    const T *__restrict__ v_cache,
                                                                    float *__restrict__ part, int nsplit, int per, int r0) {
  extern __shared__ float sm[];
  const int dh = DHC ? DHC : a.dh;
  const int split = blockIdx.x % nsplit, g = (blockIdx.x / nsplit) % a.Hk, b = blockIdx.x / (nsplit * a.Hk);
  const int len = seq_pos(a, b) + 1;
  if (split * per >= len) return;  // a short sequence has fewer splits: nobody reads the others' place
  const int nr = min(R_MAX, a.R - r0);  // query heads of this pass: g*R + r0 .. + nr
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float *qs = sm;                             // [R_MAX][dh], scaled to log2 units
  float *ps = qs + R_MAX * dh + wave * 64 * R_MAX;  // [64][R_MAX] probabilities of this wavefront's current keys
  float *mrg = sm + R_MAX * dh + DEC_WAVES * 64 * R_MAX;  // merge area: [DEC_WAVES][R_MAX][2 + dh]
  const float c = a.scale * 1.44269504088896340736f;
  for (int i = tid; i < R_MAX * dh; i += blockDim.x) {
    const int r = i / dh, ch = i % dh;
    qs[i] = r < nr ? q_new[((long long)b * a.Hq + g * a.R + r0 + r) * dh + ch] * c : 0.f;
  }
  __syncthreads();

  // keys of this split, dealt to the wavefronts in blocks of 64
  const int k_begin = split * per, k_end = min(len, k_begin + per);
  float m[R_MAX], l[R_MAX], o[R_MAX][CPL];
#pragma unroll
  for (int r = 0; r < R_MAX; ++r) {
    m[r] = -INFINITY;
    l[r] = 0.f;
#pragma unroll
    for (int x = 0; x < CPL; ++x) o[r][x] = 0.f;
  }
  const long long row_elems = (long long)a.Hk * dh;
  const T *kb = k_cache + ((long long)b * a.S * a.Hk + g) * dh;
  const T *vb = v_cache + ((long long)b * a.S * a.Hk + g) * dh;
  for (int k0 = k_begin + wave * 64; k0 < k_end; k0 += DEC_WAVES * 64) {
    const int key = k0 + lane;
    const bool live = key < k_end;
    float s[R_MAX];
#pragma unroll
    for (int r = 0; r < R_MAX; ++r) s[r] = 0.f;
    if (live) {
      const T *kp = kb + (long long)key * row_elems;
#pragma unroll
      for (int ch = 0; ch < dh; ch += 8) {
        float kv[8];
        load_vec<8>(kp + ch, kv);
#pragma unroll
        for (int r = 0; r < R_MAX; ++r)
          if (r < nr) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s[r] = fmaf(kv[e], qs[r * dh + ch + e], s[r]);
          }
      }
    }
    float alpha[R_MAX];
#pragma unroll
    for (int r = 0; r < R_MAX; ++r) {
      float mx = live ? s[r] : -INFINITY;
      for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      const float mn = fmaxf(m[r], mx), ms = mn == -INFINITY ? 0.f : mn;  // every score so far may be -inf
      const float p = live ? exp2f(s[r] - ms) : 0.f;
      float sum = p;
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
      alpha[r] = exp2f(m[r] - ms);  // 0 on the first block
      l[r] = l[r] * alpha[r] + sum;
      m[r] = mn;
      ps[lane * R_MAX + r] = p;
    }
#pragma unroll
    for (int r = 0; r < R_MAX; ++r)
#pragma unroll
      for (int x = 0; x < CPL; ++x) o[r][x] *= alpha[r];
    // the probabilities written above are read by the same wavefront only: LDS serves a wavefront in order
    const int nk = min(64, k_end - k0);
    constexpr int VB = 16;  // value rows requested together
    for (int j0 = 0; j0 < nk; j0 += VB) {
      float vv[VB][CPL];
#pragma unroll
      for (int u = 0; u < VB; ++u) {
#pragma unroll
        for (int x = 0; x < CPL; ++x) vv[u][x] = 0.f;
        const int j = min(j0 + u, nk - 1);  // rows past the end repeat the last one; their probability is 0
        if (lane * CPL < dh) load_vec<CPL>(vb + (long long)(k0 + j) * row_elems + lane * CPL, vv[u]);
      }
#pragma unroll
      for (int u = 0; u < VB; ++u) {
#pragma unroll
        for (int r = 0; r < R_MAX; ++r) {
          const float p = j0 + u < nk ? ps[(j0 + u) * R_MAX + r] : 0.f;
#pragma unroll
          for (int x = 0; x < CPL; ++x) o[r][x] = fmaf(p, vv[u][x], o[r][x]);
        }
      }
    }
  }
  // merge the wavefronts in a fixed order
  const int stride = 2 + dh;
#pragma unroll
  for (int r = 0; r < R_MAX; ++r) {
    float *dst = mrg + (wave * R_MAX + r) * stride;
    if (lane == 0) {
      dst[0] = m[r];
      dst[1] = l[r];
    }
#pragma unroll
    for (int x = 0; x < CPL; ++x) {
      const int ch = lane * CPL + x;
      if (ch < dh) dst[2 + ch] = o[r][x];
    }
  }
  __syncthreads();
  for (int i = tid; i < nr * dh; i += blockDim.x) {
    const int r = i / dh, ch = i % dh;
    float M = -INFINITY;
    for (int w = 0; w < DEC_WAVES; ++w) M = fmaxf(M, mrg[(w * R_MAX + r) * stride]);
    float L = 0.f, acc = 0.f;
    for (int w = 0; w < DEC_WAVES; ++w) {
      const float *src = mrg + (w * R_MAX + r) * stride;
      const float f = src[0] == -INFINITY ? 0.f : exp2f(src[0] - M);
      L += src[1] * f;
      acc += src[2 + ch] * f;
    }
    float *out = part + (((long long)b * a.Hq + g * a.R + r0 + r) * nsplit + split) * stride;
    if (ch == 0) {
      out[0] = M;
      out[1] = L;
    }
    out[2 + ch] = acc;
  }
}

// Lane exchanges that stay in the vector registers.  The swaps hand (a, b) back as (a's lower half | b's lower half, a's upper
// half | b's upper half) of the wavefront (32) or of each pair of 16-lane rows (16): with a = b = x a sum or maximum over lane
// and lane ^ 32 (16), with two values their two sums, the first in the lower and the second in the upper lanes.
__device__ __forceinline__ float halves32_add(float a, float b) {
  const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}
__device__ __forceinline__ float halves16_add(float a, float b) {
  const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}
__device__ __forceinline__ float xor32_add(float x) { return halves32_add(x, x); }
__device__ __forceinline__ float xor16_add(float x) { return halves16_add(x, x); }
__device__ __forceinline__ float xor32_max(float x) {
  const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(w[0]), __uint_as_float(w[1]));
}
__device__ __forceinline__ float xor16_max(float x) {
  const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(w[0]), __uint_as_float(w[1]));
}
// the value of lane ^ 8 (a rotation by 8 inside each row of 16 lanes)
__device__ __forceinline__ float ror8(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, true));
}

// ---------------------------------------------------------------------------
// The same attention for bf16 caches with d_h in {64, 128, 256}: rows of K and V are read the way they lie in
// memory.  A row is d_h / 8 chunks of 16 bytes; lane = (row of a group of 64 / LPR rows, chunk), so one load
// instruction fetches whole adjacent rows and every byte of every cache line it touches.  A lane's share of a score
// is the dot product over its 8 channels (bf16 pair dot instructions against the query, which the prologue has
// already rounded to bf16, packed in registers); the LPR shares of a row are added with DPP lane exchanges inside a
// row of 16 lanes, after which every lane of the row holds the score.  Each row group of a wavefront keeps its own
// online-softmax state (m, l, o over its 8 channels) so the main loop has no other cross-lane step; the groups, then
// the wavefronts, are merged once at the end.  The next block's K loads are issued as soon as the scores of the
// current one have left the K registers and the next V loads after the P V step, so a wavefront always has one or
// two blocks of loads in flight.  NR = query heads per pass, U = load instructions (groups of rows) per block: 8 for one or
// two heads; 4 above, where the accumulators and 8 groups' rows leave two workgroups on a CU (four heads: 134 registers for
// 4 groups, 200 for 8; eight heads x 128, 20 sequences below 8000 keys: 30.6 us for 4 groups, 33.4 for 2).
// What bounds it: a full batch over long caches the cache itself (32 x 16384 keys of 1 KB: 99.5 us, 5.4 TB/s), a short or
// ragged one the time a workgroup needs besides its keys.  13 sequences of up to 5003 keys, 4 KV heads x 64, 19.5 -> 12.8 us:
// splits past a sequence's end leave at once (they merged and wrote empty states: with every sequence empty the kernel
// took 15 us, now 6), the last block requests no next one, and the merge of the row groups stays in the vector registers (it was 3 x
// 10 lane exchanges through LDS per head).
// ---------------------------------------------------------------------------
template <int NR, int DH, int U>
__global__ __launch_bounds__(DEC_WAVES * 64) void decode_attn_rows_kernel(DecArgs a, const float *__restrict__ q_new,
                                                                         const bf16_t *__restrict__ k_cache,
                                                                         const bf16_t *__restrict__ v_cache,
                                                                         float *__restrict__ part, int nsplit, int per, int r0) {
  constexpr int LPR = DH / 8, RPL = 64 / LPR, BLK = U * RPL;  // lanes per row, rows per load, rows per block
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  __shared__ float mrg[DEC_WAVES][NR][2 + DH];
  const int split = blockIdx.x % nsplit, g = (blockIdx.x / nsplit) % a.Hk, b = blockIdx.x / (nsplit * a.Hk);
  const int nr = min(NR, a.R - r0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rr = lane / LPR, cc = lane % LPR;
  const float c = a.scale * 1.44269504088896340736f;

  f4 ql[NR], qh[NR];  // heads past the last repeat it; nobody stores their results
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float *qp = q_new + ((long long)b * a.Hq + g * a.R + r0 + min(r, nr - 1)) * DH + cc * 8;
    ql[r] = *reinterpret_cast<const f4 *>(qp);
    qh[r] = *reinterpret_cast<const f4 *>(qp + 4);
  }

  const int len = seq_pos(a, b) + 1;  // after the query's loads: one latency for both
  if (split * per >= len) return;     // a short sequence has fewer splits: nobody reads the others' place

  float m[NR], l[NR], o[NR][8];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    m[r] = -INFINITY;
    l[r] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[r][e] = 0.f;
  }
  const int k_begin = split * per, k_end = min(len, k_begin + per);
  int k0 = k_begin + wave * BLK;
  if (k0 < k_end) {  // wave-uniform
    const uint32_t rowb = (uint32_t)a.Hk * DH * 2;  // bytes between consecutive tokens (S * rowb < 2^31: host check)
    const unsigned char *kb = reinterpret_cast<const unsigned char *>(k_cache + ((long long)b * a.S * a.Hk + g) * DH);
    const unsigned char *vb = reinterpret_cast<const unsigned char *>(v_cache + ((long long)b * a.S * a.Hk + g) * DH);
    // byte offsets of this lane's chunk in the U row groups of a block (the same for K and V); rows past the end of
    // the split repeat its last row (in bounds) and their probabilities are set to zero
    uint32_t off[U];
    auto offsets = [&](int kk) {
#pragma unroll
      for (int u = 0; u < U; ++u) off[u] = (uint32_t)min(kk + u * RPL + rr, k_end - 1) * rowb + cc * 16;
    };
    u4 kr[U], vr[U];
    offsets(k0);
#pragma unroll
    for (int u = 0; u < U; ++u) kr[u] = *reinterpret_cast<const u4 *>(kb + off[u]);
    __builtin_amdgcn_sched_barrier(0);  // K before V, as in the loop: the first wait is then for the K loads only
#pragma unroll
    for (int u = 0; u < U; ++u) vr[u] = *reinterpret_cast<const u4 *>(vb + off[u]);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t q2[NR][4];  // this lane's 8 channels of each query head, bf16 pairs (exact: q_new holds bf16 values)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      q2[r][0] = (__float_as_uint(ql[r].x) >> 16) | (__float_as_uint(ql[r].y) & 0xffff0000u);
      q2[r][1] = (__float_as_uint(ql[r].z) >> 16) | (__float_as_uint(ql[r].w) & 0xffff0000u);
      q2[r][2] = (__float_as_uint(qh[r].x) >> 16) | (__float_as_uint(qh[r].y) & 0xffff0000u);
      q2[r][3] = (__float_as_uint(qh[r].z) >> 16) | (__float_as_uint(qh[r].w) & 0xffff0000u);
    }
    // One block: its scores, the next block's K loads, softmax, P V, the next block's V loads.  A wavefront's last block has no
    // next one, and only that one may reach past the end of the split.
    auto block = [&](auto last_) __attribute__((always_inline)) {
      constexpr bool LAST = decltype(last_)::value;
      float s[U][NR];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          float acc = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t kw = kr[u][i], qw = q2[r][i];  // scalars first: a bit cast straight from a vector element is not safe
            acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2, kw), __builtin_bit_cast(bf2, qw), acc, false);
          }
          s[u][r] = acc;
        }
      if constexpr (!LAST) {
        offsets(k0 + DEC_WAVES * BLK);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) kr[u] = *reinterpret_cast<const u4 *>(kb + off[u]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool live = !LAST || k0 + u * RPL + rr < k_end;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          float x = s[u][r];
          x = dpp_add<0xB1>(x);   // quad_perm [1,0,3,2]
          x = dpp_add<0x4E>(x);   // quad_perm [2,3,0,1]
          x = dpp_add<0x141>(x);  // row_half_mirror
          if constexpr (LPR >= 16) x = dpp_add<0x140>(x);  // row_mirror
          if constexpr (LPR >= 32) x = xor16_add(x);
          s[u][r] = live ? x * c : -INFINITY;
        }
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        float mx = s[0][r];
#pragma unroll
        for (int u = 1; u < U; ++u) mx = fmaxf(mx, s[u][r]);
        const float mn = fmaxf(m[r], mx);
        const float ms = mn == -INFINITY ? 0.f : mn;  // a row group that has seen no live key yet
        const float alpha = exp2f(m[r] - ms);
        float sum = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          s[u][r] = exp2f(s[u][r] - ms);
          sum += s[u][r];
        }
        l[r] = l[r] * alpha + sum;
        m[r] = mn;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[r][e] *= alpha;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float vf[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          vf[2 * i] = __uint_as_float(vr[u][i] << 16);
          vf[2 * i + 1] = __uint_as_float(vr[u][i] & 0xffff0000u);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int e = 0; e < 8; ++e) o[r][e] = fmaf(s[u][r], vf[e], o[r][e]);
      }
      if constexpr (!LAST) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) vr[u] = *reinterpret_cast<const u4 *>(vb + off[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    for (; k0 + DEC_WAVES * BLK < k_end; k0 += DEC_WAVES * BLK) block(std::false_type{});
    block(std::true_type{});
  }
  // Merge the row groups of the wavefront: the maximum first, each group's state scaled to it once, then sums over the lanes
  // that hold the same channels, each step leaving half of the channels to either half of the lanes (lane bit 5, then 4, 3).
  constexpr int OWN = 8 * LPR / 64;  // channels of a lane afterwards
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    float M = xor32_max(m[r]);
    if constexpr (LPR <= 16) M = xor16_max(M);
    if constexpr (LPR == 8) M = fmaxf(M, ror8(M));
    const float f = exp2f(m[r] - (M == -INFINITY ? 0.f : M));  // no live key in the wavefront: every state is (-inf, 0, 0)
    float lr = xor32_add(l[r] * f);
    if constexpr (LPR <= 16) lr = xor16_add(lr);
    if constexpr (LPR == 8) lr += ror8(lr);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[r][e] *= f;
    float h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = halves32_add(o[r][e], o[r][e + 4]);
    if constexpr (LPR <= 16) {
      h[0] = halves16_add(h[0], h[2]);
      h[1] = halves16_add(h[1], h[3]);
    }
    if constexpr (LPR == 8) {
      const float keep = (lane & 8) ? h[1] : h[0], give = (lane & 8) ? h[0] : h[1];
      h[0] = keep + ror8(give);
    }
    const int ch = cc * 8 + (lane >> 5) * 4 + (LPR <= 16 ? ((lane >> 4) & 1) * 2 : 0) + (LPR == 8 ? (lane >> 3) & 1 : 0);
#pragma unroll
    for (int e = 0; e < OWN; ++e) mrg[wave][r][2 + ch + e] = h[e];
    if (lane == 0) {
      mrg[wave][r][0] = M;
      mrg[wave][r][1] = lr;
    }
  }
  __syncthreads();
  constexpr int stride = 2 + DH;
  for (int i = tid; i < nr * DH; i += DEC_WAVES * 64) {
    const int r = i / DH, ch = i % DH;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < DEC_WAVES; ++w) M = fmaxf(M, mrg[w][r][0]);
    float L = 0.f, acc = 0.f;
#pragma unroll
    for (int w = 0; w < DEC_WAVES; ++w) {
      const float f = mrg[w][r][0] == -INFINITY ? 0.f : exp2f(mrg[w][r][0] - M);
      L += mrg[w][r][1] * f;
      acc += mrg[w][r][2 + ch] * f;
    }
    float *out = part + (((long long)b * a.Hq + g * a.R + r0 + r) * nsplit + split) * stride;
    if (ch == 0) {
      out[0] = M;
      out[1] = L;
    }
    out[2 + ch] = acc;
  }
}

// o[b, h, :] = sum_s part_o * 2^(m_s - M) / sum_s l_s * 2^(m_s - M), splits in index order.  A thread per channel; its values
// of up to MAX_SPLITS splits are requested with the states, before the length of the sequence is known (a place that no split
// wrote is read, never used): one memory latency for both.
template <typename T>
__global__ __launch_bounds__(256) void decode_combine_kernel(DecArgs a, const float *__restrict__ part, int nsplit, int per,
                                                            T *__restrict__ o) {
  __shared__ float f[MAX_SPLITS];  // 2^(m_s - M) / L per split (0 beyond the sequence's last)
  const int bh = blockIdx.x, dh = a.dh, stride = 2 + dh, tid = threadIdx.x;
  const float *src = part + (long long)bh * nsplit * stride;
  const float *mine = src + 2 + min(tid, dh - 1);
  float val[MAX_SPLITS];
#pragma unroll
  for (int s0 = 0; s0 < MAX_SPLITS; s0 += 8)
    if (s0 < nsplit) {
#pragma unroll
      for (int s = s0; s < s0 + 8; ++s) val[s] = mine[min(s, nsplit - 1) * stride];
    }
  // the state of split `tid` (an even number of floats from a 256-byte boundary)
  const float2 state = *reinterpret_cast<const float2 *>(src + min(tid, nsplit - 1) * stride);
  __builtin_amdgcn_sched_barrier(0);  // requested with the values
  const int len = seq_pos(a, bh / a.Hq) + 1, n = min(nsplit, (len + per - 1) / per);
  if (tid < 64) {  // one wavefront: lane s holds split s
    const float m0 = state.x, l0 = state.y;
    const float ms = tid < n ? m0 : -INFINITY, ls = tid < n ? l0 : 0.f;
    float M = ms;
    for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float w = ms == -INFINITY ? 0.f : exp2f(ms - M);
    float L = 0.f;
    for (int s = 0; s < n; ++s) L += __shfl(ls * w, s);  // index order
    if (tid < MAX_SPLITS) f[tid] = w / L;
  }
  __syncthreads();
  float acc = 0.f;
#pragma unroll
  for (int s0 = 0; s0 < MAX_SPLITS; s0 += 8)
    if (s0 < n) {
#pragma unroll
      for (int s = s0; s < s0 + 8; ++s) acc = s < n ? fmaf(val[s], f[s], acc) : acc;
    }
  if (tid < dh) store_f(o + (long long)bh * dh + tid, acc);
}

// ---------------------------------------------------------------------------
// Projections of a decode step in fp32 (bf16: gemm_panel_kernel): C (M, N) = A (M, K) W (K, N) with M = batch size, bound by
// reading W once.  Workgroup = 128 columns x one slice of K; a lane owns 2 adjacent columns (one 4- or 8-byte load
// per row of W), the 4 wavefronts take quarters of the slice and are added through LDS, rows of A go through LDS
// 16 or 32 at a time ([k][rows] floats, so one 16-byte broadcast read feeds 4 rows).  K slices write fp32 partial sums
// that a second kernel adds in index order (no atomics).
// ---------------------------------------------------------------------------
constexpr int SK_COLS = 128, SK_MAXCHUNK = 128, SK_KB = 16, SK_PAD = 4;

// ROWS = rows of A per pass (16 or 32).  A wavefront requests SK_KB rows of W at a time and the next batch before it
// multiplies the current one, so its loads overlap the arithmetic instead of being waited for one by one.
template <typename T, int ROWS>
__global__ __launch_bounds__(256) void gemm_skinny_kernel(const T *__restrict__ A, const T *__restrict__ W,
                                                         float *__restrict__ part, int M, int N, int K, int chunk) {
  constexpr int XS = ROWS + SK_PAD;  // padded row of the A tile: the transposing store spreads over 8 banks
  constexpr int XS_FLOATS = SK_MAXCHUNK * XS, RED_FLOATS = 3 * 64 * ROWS * 2;
  __shared__ float buf[XS_FLOATS > RED_FLOATS ? XS_FLOATS : RED_FLOATS];
  float *xs = buf;   // [klen][XS] A tile, fp32
  float *red = buf;  // [3][64][2 * ROWS] sums of wavefronts 1..3 (after the A tile is no longer read)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.x * SK_COLS + lane * 2;
  const int k_begin = blockIdx.y * chunk, k_end = min(K, k_begin + chunk);
  const int klen = k_end - k_begin;
  const int per_wave = (klen + 3) / 4;
  const int kw0 = wave * per_wave, kw1 = min(klen, kw0 + per_wave);
  const bool col_ok = n0 < N;
  // rows of W past the wavefront's range are read from its last row (in bounds) and multiplied by nothing
  const T *wp = W + (long long)k_begin * N + (col_ok ? n0 : 0);
  auto load_rows = [&](int kk0, float (&wv)[SK_KB][2]) {
#pragma unroll
    for (int j = 0; j < SK_KB; ++j) load_vec<2>(wp + (long long)min(kk0 + j, max(kw1 - 1, 0)) * N, wv[j]);
  };
  for (int m0 = 0; m0 < M; m0 += ROWS) {
    __syncthreads();  // the previous pass no longer reads buf
    for (int i = tid; i < klen * ROWS; i += 256) {
      const int m = i / klen, kk = i % klen;  // consecutive threads read consecutive k of one row
      xs[kk * XS + m] = m0 + m < M ? load_f(A + (long long)(m0 + m) * K + k_begin + kk) : 0.f;
    }
    __syncthreads();
    float acc[ROWS][2];
#pragma unroll
    for (int m = 0; m < ROWS; ++m) acc[m][0] = acc[m][1] = 0.f;
    if (kw0 < kw1) {
      float wa[SK_KB][2], wb[SK_KB][2];
      load_rows(kw0, wa);
      for (int kk0 = kw0; kk0 < kw1; kk0 += SK_KB) {
        load_rows(kk0 + SK_KB, wb);
#pragma unroll
        for (int j = 0; j < SK_KB; ++j) {
          if (kk0 + j < kw1) {  // wave-uniform
#pragma unroll
            for (int m4 = 0; m4 < ROWS; m4 += 4) {
              typedef float f4 __attribute__((ext_vector_type(4)));
              const f4 xv = *reinterpret_cast<const f4 *>(&xs[(kk0 + j) * XS + m4]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                acc[m4 + e][0] = fmaf(xv[e], wa[j][0], acc[m4 + e][0]);
                acc[m4 + e][1] = fmaf(xv[e], wa[j][1], acc[m4 + e][1]);
              }
            }
          }
        }
#pragma unroll
        for (int j = 0; j < SK_KB; ++j) wa[j][0] = wb[j][0], wa[j][1] = wb[j][1];
      }
    }
    __syncthreads();  // every wavefront is done with the A tile: its memory now takes the partial sums
    if (wave > 0) {
#pragma unroll
      for (int m = 0; m < ROWS; ++m) {
        red[((wave - 1) * 64 + lane) * 2 * ROWS + 2 * m] = acc[m][0];
        red[((wave - 1) * 64 + lane) * 2 * ROWS + 2 * m + 1] = acc[m][1];
      }
    }
    __syncthreads();
    if (wave == 0 && col_ok) {
#pragma unroll
      for (int m = 0; m < ROWS; ++m) {
        if (m0 + m < M) {
          float a0 = acc[m][0], a1 = acc[m][1];
          for (int w = 0; w < 3; ++w) a0 += red[(w * 64 + lane) * 2 * ROWS + 2 * m], a1 += red[(w * 64 + lane) * 2 * ROWS + 2 * m + 1];
          float *dst = part + ((long long)blockIdx.y * M + m0 + m) * N + n0;
          dst[0] = a0;
          dst[1] = a1;
        }
      }
    }
  }
}

// The same product on the matrix cores for bf16 (N and K multiples of 8), in one launch without partial sums in memory.
// Workgroup = 32 columns x all of K: its panel of W (64 bytes per row) and the rows of A are requested together, straight
// into LDS, as much of K at a time as fits (all 2048 for up to 8 rows, 1024 for 32), so one memory latency is paid per
// pass - what bounds a product this small is latency and launches, not bytes.  The panel is read as MFMA fragments with the
// transposing LDS read (rows lie 64 bytes apart, so the 8 rows a read touches are 512 adjacent bytes: no bank conflicts, no
// padding); A lies row-major with chunk c of row r at c ^ (r mod 16).  (Read as fragments straight from memory, 32 rows x
// 32 bytes per load instruction, A cost 9 of 14.6 us at 32 rows and K = 2048: the memory pipeline works per cache line.)
// The 8 wavefronts take an eighth of the k each and their sums are added through LDS in order.  A CU takes in about 29 GB/s
// of 64-byte pieces, so the grid is split over K as well where the next kernel adds the parts anyway (the down-projection:
// K = 2048 whole 6.7 us at one row, in 5 slices 4.4).  Up-projection, K x N = 1024 x 2048: 3.4 us at one row, 5.8 at 32,
// against 6.4 + 4.7 us for one workgroup per CU with partial sums and a kernel to add them.  More than 32 rows: a workgroup per
// 32 (each reads its panel of W again, mostly from the L2), and the down-projection in fewer slices.  One workgroup for all rows in
// turn was slower than W staged once (step of 128 sequences over 200 keys, E = 2048, 8 / 2 heads of 128: W staged once 68.3,
// in turn 70.6, side by side 55.3 us; 512: 177, 234, 167; 40 x 1000, E = 4096: 78, 85, 71).
typedef __bf16 sk_bf16x8 __attribute__((ext_vector_type(8)));
typedef float sk_f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t sk_u32x4 __attribute__((ext_vector_type(4)));
typedef short sk_v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) sk_v4i16 sk_lds_v4i16;
constexpr int PN_COLS = 32, PN_NT = 512, PN_WAVES = PN_NT / 64;
constexpr size_t PN_LDS = 160 * 1024, PN_SUMS = (size_t)PN_WAVES * 32 * 33 * 4;

// rows of W per pass: all of K in as few equal passes as the LDS allows, in whole 256-byte lines of A
int panel_rows(int M, int K) {
  const int fit = (int)(PN_LDS / (PN_COLS * 2 + 2 * (size_t)(M < 32 ? M : 32))) / 128 * 128;
  const int passes = (K + fit - 1) / fit;
  return ((K + passes - 1) / passes + 127) / 128 * 128;
}

// C row m starts at C + m * ldc (the rows of a projection may go straight into a strided destination).  With `row_pos`
// row m goes to ring slot clamp(row_pos[m], 0, pos_max) % ring of its sequence: C + m * ldc + slot * N.
struct RowDest {
  long long ldc;
  const int *row_pos;
  int pos_max, ring;
  __device__ __forceinline__ long long at(int m, int N) const {
    long long o = m * ldc;
    if (row_pos) {
      const int p = row_pos[m];
      o += (long long)((p < 0 ? 0 : (p > pos_max ? pos_max : p)) % ring) * N;
    }
    return o;
  }
};

// (a body inlined with restrict arguments: without them the compiler makes the transposing LDS reads of a later pass wait
// for loads into LDS that they do not touch)
// COMBINE: A is not in memory yet, its rows are the sums over the splits of the attention (`cmb`, as decode_combine_kernel forms them),
// made here while the panel of W is on its way; one pass over all of K, B * H_q d_h <= 4 PN_NT, d_h >= 64, at most COMBINE_SPLITS splits.
constexpr int COMBINE_SPLITS = 8;
struct CombineArgs {
  DecArgs a;
  const float *part;
  int nsplit, per;
};
// Rows of A into LDS: a thread per four channels, the values of all splits requested with the states, before the length of the
// sequence is known
__device__ __forceinline__ void combine_rows(const CombineArgs &c, int M, int K, int kp, unsigned char *sA) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  __shared__ float f[4 * PN_NT / 64 * COMBINE_SPLITS];  // 2^(m_s - M) / L of every row, head and split (0 beyond the sequence's last); d_h >= 64 here
  const int tid = threadIdx.x, dh = c.a.dh, Hq = c.a.Hq, stride = 2 + dh, per_row = K / 4;
  const int item = min(tid, M * per_row - 1), row = item / per_row, k = item % per_row * 4, head = k / dh;
  const float *const mine = c.part + (long long)(row * Hq + head) * c.nsplit * stride + 2 + k % dh;  // (8-byte aligned: dh is even)
  f2 lo[COMBINE_SPLITS], hi[COMBINE_SPLITS];
#pragma unroll
  for (int s0 = 0; s0 < COMBINE_SPLITS; s0 += 4)
    if (s0 < c.nsplit) {
#pragma unroll
      for (int s = s0; s < s0 + 4; ++s) {
        const f2 *const at = reinterpret_cast<const f2 *>(mine + min(s, c.nsplit - 1) * stride);
        lo[s] = at[0], hi[s] = at[1];
      }
    }
  // the factors: COMBINE_SPLITS lanes per row and head, lane = split
  for (int bh0 = 0; bh0 < M * Hq; bh0 += PN_NT / COMBINE_SPLITS) {
    const int bh = min(bh0 + tid / COMBINE_SPLITS, M * Hq - 1), s = tid % COMBINE_SPLITS;
    const f2 state = *reinterpret_cast<const f2 *>(c.part + ((long long)bh * c.nsplit + min(s, c.nsplit - 1)) * stride);
    const int len = seq_pos(c.a, bh / Hq) + 1, n = min(c.nsplit, (len + c.per - 1) / c.per);
    const float ms = s < n ? state.x : -INFINITY, ls = s < n ? state.y : 0.f;
    float m = ms;
#pragma unroll
    for (int off = COMBINE_SPLITS / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    const float w = ms == -INFINITY ? 0.f : exp2f(ms - m);
    float l = 0.f;
#pragma unroll
    for (int x = 0; x < COMBINE_SPLITS; ++x) {  // index order; past the last split nothing
      const float lx = __shfl(ls * w, (tid & 63) / COMBINE_SPLITS * COMBINE_SPLITS + x);
      l = x < n ? l + lx : l;
    }
    f[bh * COMBINE_SPLITS + s] = s < n ? w / l : 0.f;
  }
  __syncthreads();
  const int len = seq_pos(c.a, row) + 1, n = min(c.nsplit, (len + c.per - 1) / c.per);
  f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < COMBINE_SPLITS; ++s)
    if (s < n) {
      const float w = f[(row * Hq + head) * COMBINE_SPLITS + s];
      acc.x = fmaf(lo[s].x, w, acc.x), acc.y = fmaf(lo[s].y, w, acc.y);
      acc.z = fmaf(hi[s].x, w, acc.z), acc.w = fmaf(hi[s].y, w, acc.w);
    }
  unsigned char *const at = sA + row * (kp * 2);
  if (tid < M * per_row) {
    const uint32_t p[2] = {(uint32_t)f32_to_bf16(acc.x) | (uint32_t)f32_to_bf16(acc.y) << 16, (uint32_t)f32_to_bf16(acc.z) | (uint32_t)f32_to_bf16(acc.w) << 16};
    uint32_t *const to = reinterpret_cast<uint32_t *>(at + (((k / 8) ^ (row & 15)) * 16) + (k & 4) * 2);
    to[0] = p[0], to[1] = p[1];
  }
}

template <bool COMBINE>
__device__ __forceinline__ void gemm_panel_body(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W, bf16_t *__restrict__ C,
                                                RowDest dest, int M, int N, int K, int kp, int k_slice, float *__restrict__ part,
                                                const CombineArgs &cmb, unsigned char *smem) {
  typedef __attribute__((address_space(3))) void lds_void;
  typedef __attribute__((address_space(1))) void glb_void;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int n0 = blockIdx.x * PN_COLS;
  const int col = n0 + (lane & 3) * 8 < N ? n0 + (lane & 3) * 8 : 0;  // columns past N feed outputs that are not stored
  unsigned char *const sA = smem + kp * (PN_COLS * 2);
  // transposing read: this lane's 8 bytes of row 8 * half + (lane & 15) / 4 (+ 4) of a group, column block (lane >> 4) & 1
  const unsigned char *const pw = smem + (8 * half + ((lane & 15) >> 2)) * 64 + (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2;
  const int cpr = kp / 8;  // 16-byte chunks of a row of A
  const int k_begin = blockIdx.y * k_slice, k_end = min(K, k_begin + k_slice);
  for (int m0 = blockIdx.z * 32; m0 < M; m0 += gridDim.z * 32) {
    const int mrows = min(32, M - m0);
    sk_f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    for (int k0 = k_begin; k0 < k_end; k0 += kp) {
      const int rows = min(kp, k_end - k0), groups = (rows + 15) / 16;
      __syncthreads();  // what lies in LDS is no longer read
      // whole groups of 16 k: k past the end are zero in both operands
      for (int g = wave; g < groups; g += PN_WAVES) {
        const int r = g * 16 + (lane >> 2);
        if (r < rows)
          __builtin_amdgcn_global_load_lds((glb_void *)(W + (long long)(k0 + r) * N + col), (lds_void *)(smem + g * 1024), 16, 0, 0);
        else
          *reinterpret_cast<sk_u32x4 *>(smem + g * 1024 + lane * 16) = sk_u32x4{0, 0, 0, 0};
      }
      if constexpr (COMBINE) combine_rows(cmb, M, K, kp, sA);
      else for (int i = wave; i < (mrows * cpr + 63) / 64; i += PN_WAVES) {
        const int pos = i * 64 + lane, r = pos / cpr, p = pos % cpr, k = (p ^ (r & 15)) * 8;
        if (r < mrows) {
          if (k < rows)
            __builtin_amdgcn_global_load_lds((glb_void *)(A + (long long)(m0 + r) * K + k0 + k), (lds_void *)(sA + i * 1024), 16, 0, 0);
          else
            *reinterpret_cast<sk_u32x4 *>(sA + pos * 16) = sk_u32x4{0, 0, 0, 0};
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      const int per = (groups + PN_WAVES - 1) / PN_WAVES, g_end = min(groups, (wave + 1) * per);
      const int ra = min(l32, mrows - 1);  // rows past M repeat the last one; they are not stored
      const unsigned char *const pa = sA + ra * (kp * 2);
#pragma unroll 4
      for (int g = wave * per; g < g_end; ++g) {
        const unsigned char *const q = pw + g * 1024;
        const sk_bf16x8 fa = __builtin_bit_cast(sk_bf16x8, *reinterpret_cast<const sk_u32x4 *>(pa + (((2 * g + half) ^ (ra & 15)) * 16)));
        const sk_v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((sk_lds_v4i16 *)q);
        const sk_v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((sk_lds_v4i16 *)(q + 256));
        const sk_bf16x8 fw = __builtin_bit_cast(sk_bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw, fa, acc, 0, 0, 0);
      }
    }
    // acc[r] = this wavefront's part of C[m0 + l32][n0 + 8*(r/4) + 4*half + r%4]
    float *const red = reinterpret_cast<float *>(smem);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(wave * 32 + l32) * 33 + 8 * (r >> 2) + 4 * half + (r & 3)] = acc[r];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int m = (tid >> 5) + 16 * x, c = tid & 31;
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < PN_WAVES; ++w) sum += red[(w * 32 + m) * 33 + c];
      if (m < mrows && n0 + c < N) {
        if (part) part[((long long)blockIdx.y * M + m0 + m) * N + n0 + c] = sum;
        else C[dest.at(m0 + m, N) + n0 + c] = f32_to_bf16(sum);
      }
    }
  }
}

__global__ __launch_bounds__(PN_NT) void gemm_panel_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W,
                                                          bf16_t *__restrict__ C, RowDest dest, int M, int N, int K, int kp,
                                                          int k_slice, float *__restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char psm[];
  gemm_panel_body<false>(A, W, C, dest, M, N, K, kp, k_slice, part, CombineArgs{}, psm);
}

// The up-projection of a few rows whose attention ran in a few splits: the launch that combines them saved (figures: decode_up_combines)
__global__ __launch_bounds__(PN_NT) void gemm_panel_combine_kernel(CombineArgs cmb, const bf16_t *__restrict__ W, bf16_t *__restrict__ C, RowDest dest,
                                                                  int M, int N, int K, int kp) {
  extern __shared__ __attribute__((aligned(16))) unsigned char psm[];
  gemm_panel_body<true>(nullptr, W, C, dest, M, N, K, kp, K, nullptr, cmb, psm);
}

template <typename T>
__global__ void skinny_reduce_kernel(const float *__restrict__ part, T *__restrict__ C, RowDest dest, long long mn, int N,
                                     int splits) {
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= mn) return;
  float a = 0.f;
  int s = 0;
  for (; s + 8 <= splits; s += 8) {  // 8 loads in flight, added in split order
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(long long)(s + u) * mn + id];
#pragma unroll
    for (int u = 0; u < 8; ++u) a += v[u];
  }
  for (; s < splits; ++s) a += part[(long long)s * mn + id];
  store_f(C + dest.at((int)(id / N), N) + id % N, a);
}

int skinny_splits(int N, int K) {
  const int col_blocks = (N + SK_COLS - 1) / SK_COLS;
  int splits = (256 + col_blocks - 1) / col_blocks;          // about one workgroup per CU
  const int min_splits = (K + SK_MAXCHUNK - 1) / SK_MAXCHUNK;  // a slice must fit the LDS tile
  splits = splits < min_splits ? min_splits : splits;
  return splits > K / 16 ? (K / 16 > min_splits ? K / 16 : min_splits) : splits;
}
size_t skinny_scratch_bytes(int M, int N, int K) { return (size_t)skinny_splits(N, K) * M * N * sizeof(float); }

// N and K are multiples of 8, as every bf16 width is (make_dims).  `part` gets `slices` partial sums (slices, M, N) for the caller's next
// kernel to add; without it (one slice) the rows go to C.
hipError_t gemm_panel(const bf16_t *A, const bf16_t *W, bf16_t *C, RowDest dest, float *part, int slices, int M, int N, int K,
                      hipStream_t s) {
  if (hipError_t e = raise_lds_limit<gemm_panel_kernel>(PN_LDS); e != hipSuccess) return e;
  const int row_blocks = (M + 31) / 32, k_slice = ((K + slices - 1) / slices + 127) / 128 * 128;
  const int kp = panel_rows(M, K < k_slice ? K : k_slice);
  const size_t pass = (size_t)kp * (PN_COLS * 2 + 2 * (M < 32 ? M : 32)), lds = pass > PN_SUMS ? pass : PN_SUMS;
  gemm_panel_kernel<<<dim3((N + PN_COLS - 1) / PN_COLS, slices, row_blocks < 4096 ? row_blocks : 4096), PN_NT, lds, s>>>(A, W, C, dest, M, N, K, kp, k_slice,
                                                                                 part);
  return hipGetLastError();
}

hipError_t up_combined(const DecArgs &a, const float *attn, int nsplit, int per, const bf16_t *W, bf16_t *out, int N, int K, hipStream_t s) {
  static_assert(PN_COLS == 32 && PN_SUMS <= DECODE_UP_LDS && DECODE_UP_LDS + 4 * PN_NT / 64 * COMBINE_SPLITS * sizeof(float) <= PN_LDS, "LDS");
  if (hipError_t e = raise_lds_limit<gemm_panel_combine_kernel>(DECODE_UP_LDS); e != hipSuccess) return e;
  const int kp = (K + 127) / 128 * 128;
  const size_t pass = decode_up_lds(a.B, K), lds = pass > PN_SUMS ? pass : PN_SUMS;
  if (lds > DECODE_UP_LDS) return hipErrorInvalidValue;
  gemm_panel_combine_kernel<<<(N + PN_COLS - 1) / PN_COLS, PN_NT, lds, s>>>(CombineArgs{a, attn, nsplit, per}, W, out, RowDest{N, nullptr, 0, 1}, a.B, N, K, kp);
  return hipGetLastError();
}

template <typename T>
hipError_t gemm_skinny(const T *A, const T *W, T *C, RowDest dest, float *part, int M, int N, int K, hipStream_t s) {
  if constexpr (std::is_same<T, bf16_t>::value) {
    return gemm_panel(A, W, C, dest, nullptr, 1, M, N, K, s);
  } else {
    const int splits = skinny_splits(N, K);
    const int chunk = (K + splits - 1) / splits;
    const dim3 grid((N + SK_COLS - 1) / SK_COLS, (K + chunk - 1) / chunk);
    if (M > 16) gemm_skinny_kernel<T, 32><<<grid, 256, 0, s>>>(A, W, part, M, N, K, chunk);
    else gemm_skinny_kernel<T, 16><<<grid, 256, 0, s>>>(A, W, part, M, N, K, chunk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long mn = (long long)M * N;
    skinny_reduce_kernel<T><<<(unsigned)((mn + 255) / 256), 256, 0, s>>>(part, C, dest, mn, N, (int)grid.y);
    return hipGetLastError();
  }
}

// slots of the latent ring: the taps - 1 earlier rows the convolutions reach back to (one at least, for the value
// shift) plus the slot the new row is written to
int ring_rows(const Dims &d) {
  const int ks = (d.flags & CCA_CONV_SEQ) ? d.k_seq : 1, kc = (d.flags & CCA_CONV_CH) ? d.k_ch : 1;
  const int taps = ks + kc - 1;
  return (taps - 1 > 1 ? taps - 1 : 1) + 1;
}

// K slices of the down-projection on the matrix cores: enough workgroups for the chip (with one per 32 rows), slices of 256 k at least, and no
// more than the scratch of the split form holds (skinny_scratch_bytes)
int down_slices(const Dims &d) {
  const int cols = (d.n_lat + PN_COLS - 1) / PN_COLS, most = skinny_splits(d.n_lat, d.E);
  int s = 256 / (cols * ((d.B + 31) / 32));
  s = s < d.E / 256 ? s : d.E / 256;
  s = s < most ? s : most;
  s = s < MAX_PARTS ? s : MAX_PARTS;
  return s < 1 ? 1 : s;
}

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

struct DecLayout {
  size_t q_new, o, part, gemm, total;
};
DecLayout layout(const Dims &d) {
  DecLayout L;
  size_t off = 0;
  auto take = [&](size_t n) {
    const size_t at = off;
    off += align256(n);
    return at;
  };
  L.q_new = take((size_t)d.B * d.e_q * sizeof(float));
  L.o = take((size_t)d.B * d.e_q * d.esize());
  L.part = take((size_t)d.B * d.Hq * MAX_SPLITS * (2 + d.dh) * sizeof(float));
  const size_t g1 = skinny_scratch_bytes(d.B, d.n_lat, d.E), g2 = skinny_scratch_bytes(d.B, d.E, d.e_q);
  L.gemm = take(g1 > g2 ? g1 : g2);
  L.total = off;
  return L;
}

template <typename T>
hipError_t step_t(const Dims &d, const cca_weights &w, const void *x_new, void *k_cache, void *v_cache, void *hist,
                  int pos, const int *pos_seq, void *out, unsigned char *ws, hipStream_t s) {
  // pos: the position of every sequence, or with pos_seq (device, one entry per sequence) the largest of them
  const DecLayout L = layout(d);
  const int P = ring_rows(d);
  DecArgs a{d.B, d.T, d.Hq, d.Hk, d.dh, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, P, pos,
            d.flags, d.rope_base, d.scale, d.norm_eps, pos_seq};
  float *q_new = reinterpret_cast<float *>(ws + L.q_new);
  T *o = reinterpret_cast<T *>(ws + L.o);
  float *part = reinterpret_cast<float *>(ws + L.part);
  float *gpart = reinterpret_cast<float *>(ws + L.gemm);
  // The down-projection.  On the matrix cores (bf16) it is split over K so that more CUs pull the weight (one CU takes in about 29
  // GB/s of 64-byte pieces): the prologue adds the parts and writes the new latent rows into their ring slot.  In fp32 the
  // rows go straight into the ring.
  int nparts = 1;
  hipError_t e;
  if constexpr (std::is_same<T, bf16_t>::value) {
    nparts = down_slices(d);
    e = gemm_panel((const bf16_t *)x_new, (const bf16_t *)w.w_down, nullptr, RowDest{}, gpart, nparts, d.B, d.n_lat, d.E, s);
  } else {
    const long long ring_stride = (long long)P * d.n_lat;
    const RowDest ring = pos_seq ? RowDest{ring_stride, pos_seq, pos, P} : RowDest{ring_stride, nullptr, 0, 1};
    T *const ring_c = (T *)hist + (pos_seq ? 0 : (long long)(pos % P) * d.n_lat);
    e = gemm_skinny<T>((const T *)x_new, (const T *)w.w_down, ring_c, ring, gpart, d.B, d.n_lat, d.E, s);
  }
  if (e != hipSuccess) return e;
  {
    const int kc = (d.flags & CCA_CONV_CH) ? d.k_ch : 1;
    const int threads = d.dh <= 64 ? 256 : 512, per_lane = (d.dh * kc / 8 + 7) / 8;  // filter chunks per lane of 8
    const size_t smem = sizeof(float) * ((size_t)kc * d.dh + 2 * d.dh);
#define CCA_DEC_PRO_NP(CH, LPO, NP)                                                                                       \
  decode_prologue_kernel<T, CH, LPO, NP><<<dim3(d.B, d.Hq + 2 * d.Hk), threads, smem, s>>>(                                \
      a, (T *)hist, gpart, nparts, (const T *)w.w_conv_seq, (const T *)w.w_conv_ch, w.temp, q_new, (T *)k_cache, (T *)v_cache)
#define CCA_DEC_PRO(CH, LPO)                                                                                              \
  if (std::is_same<T, float>::value || nparts == 1) CCA_DEC_PRO_NP(CH, LPO, 1);                                            \
  else if (nparts == 2) CCA_DEC_PRO_NP(CH, LPO, (std::is_same<T, float>::value ? 1 : 2));                                  \
  else if (nparts <= 5) CCA_DEC_PRO_NP(CH, LPO, (std::is_same<T, float>::value ? 1 : 5));                                  \
  else CCA_DEC_PRO_NP(CH, LPO, (std::is_same<T, float>::value ? 1 : MAX_PARTS))
    if (per_lane <= 2) { CCA_DEC_PRO(2, 8); }
    else if (per_lane <= 4) { CCA_DEC_PRO(4, 8); }
    else if (per_lane <= 8) { CCA_DEC_PRO(8, 8); }
    else { CCA_DEC_PRO(8, 16); }
#undef CCA_DEC_PRO
#undef CCA_DEC_PRO_NP
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    const int len = pos + 1;  // the longest sequence sizes the splits
    // (the row kernel addresses a sequence's cache with 32-bit byte offsets)
    const bool rows_kernel = std::is_same<T, bf16_t>::value && (d.dh == 64 || d.dh == 128 || d.dh == 256) &&
                             (long long)d.T * d.Hk * d.dh * 2 < (1ll << 31);
    const int per = decode_keys_per_split((long long)d.B * d.Hk, len, d.dh, rows_kernel, MAX_SPLITS);
    const int nsplit = (len + per - 1) / per;
    const size_t smem = sizeof(float) * ((size_t)R_MAX * d.dh + DEC_WAVES * 64 * R_MAX + DEC_WAVES * R_MAX * (2 + d.dh));
    const unsigned grid = (unsigned)((long long)d.B * d.Hk * nsplit);
    if constexpr (std::is_same<T, bf16_t>::value) {
      if (rows_kernel) {
        for (int r0 = 0; r0 < d.R; r0 += R_MAX) {
          const int left = d.R - r0;
#define CCA_DEC_ROWS(NR, DH, U)                                                                                    \
  decode_attn_rows_kernel<NR, DH, U><<<grid, DEC_WAVES * 64, 0, s>>>(a, q_new, (const bf16_t *)k_cache,             \
                                                                     (const bf16_t *)v_cache, part, nsplit, per, r0)
#define CCA_DEC_ROWS_DH(NR, U)                                                                                     \
  {                                                                                                                \
    if (d.dh == 64) CCA_DEC_ROWS(NR, 64, U);                                                                       \
    else if (d.dh == 128) CCA_DEC_ROWS(NR, 128, U);                                                                \
    else CCA_DEC_ROWS(NR, 256, U);                                                                                 \
  }
          if (left == 1) CCA_DEC_ROWS_DH(1, 8)
          else if (left == 2) CCA_DEC_ROWS_DH(2, 8)
          else if (left <= 4) CCA_DEC_ROWS_DH(4, 4)
          else CCA_DEC_ROWS_DH(8, 4)
#undef CCA_DEC_ROWS_DH
#undef CCA_DEC_ROWS
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if constexpr (std::is_same<T, bf16_t>::value)
          if (decode_up_combines(d.B, d.e_q, nsplit, COMBINE_SPLITS)) return up_combined(a, part, nsplit, per, (const bf16_t *)w.w_out, (bf16_t *)out, d.E, d.e_q, s);
        decode_combine_kernel<T><<<(unsigned)(d.B * d.Hq), (d.dh + 63) / 64 * 64, 0, s>>>(a, part, nsplit, per, o);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        return gemm_skinny<T>(o, (const T *)w.w_out, (T *)out, RowDest{d.E, nullptr, 0, 1}, gpart, d.B, d.E, d.e_q, s);
      }
    }
    for (int r0 = 0; r0 < d.R; r0 += R_MAX) {
#define CCA_DEC_ATTN(CPL, DHC)                                                                                  \
  {                                                                                                             \
    e = raise_lds_limit<decode_attn_kernel<T, CPL, DHC>>(smem);                                                 \
    if (e != hipSuccess) return e;                                                                              \
    decode_attn_kernel<T, CPL, DHC><<<grid, DEC_WAVES * 64, smem, s>>>(a, q_new, (const T *)k_cache,              \
                                                                           (const T *)v_cache, part, nsplit, per, r0); \
  }
      if (d.dh == 64) CCA_DEC_ATTN(1, 64)
      else if (d.dh == 128) CCA_DEC_ATTN(2, 128)
      else if (d.dh == 256) CCA_DEC_ATTN(4, 256)
      else if (d.dh <= 64) CCA_DEC_ATTN(1, 0)
      else if (d.dh <= 128) CCA_DEC_ATTN(2, 0)
      else CCA_DEC_ATTN(4, 0)
#undef CCA_DEC_ATTN
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    decode_combine_kernel<T><<<(unsigned)(d.B * d.Hq), (d.dh + 63) / 64 * 64, 0, s>>>(a, part, nsplit, per, o);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return gemm_skinny<T>(o, (const T *)w.w_out, (T *)out, RowDest{d.E, nullptr, 0, 1}, gpart, d.B, d.E, d.e_q, s);
}

}  // namespace

int decode_ring_rows(const Dims &d) { return ring_rows(d); }
size_t decode_scratch_bytes(const Dims &d) { return layout(d).total; }

hipError_t decode_step(const Dims &d, const cca_weights &w, const void *x_new, void *k_cache, void *v_cache, void *hist,
                       int pos, const int *pos_seq, void *out, void *workspace, hipStream_t s) {
  unsigned char *ws = static_cast<unsigned char *>(workspace);
  return d.bf16 ? step_t<bf16_t>(d, w, x_new, k_cache, v_cache, hist, pos, pos_seq, out, ws, s)
                : step_t<float>(d, w, x_new, k_cache, v_cache, hist, pos, pos_seq, out, ws, s);
}

}  // namespace cca
