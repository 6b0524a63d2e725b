// Backward of the fused latent-space prologue for gfx950, bf16 storage,
// d_h = 256, 128 or 64 (adjoint of the convolution, qk-mean and value-shift equations
// and of the first two lines of the final equation block of Sec. 2.2; the
// paper states these steps forward only).
//
//   1. pointwise kernel: undoes RoPE (a rotation: rotate back) and the norm /
//      temperature step on the gradients of q and k.  With y = x * mul,
//      mul = sqrt(d_h) beta / |x|:   dx = mul * (dy - y <y,dy> / (d_h beta^2)),
//      where y is the saved q / k (the dot product is invariant under RoPE, so
//      it is taken on the rotated vectors), mul the saved norm factor.  Result
//      d3 (B*T, e_q + e_kv) bf16 = gradient of the conv2 output; also
//      <dk,k> per (token, KV head), whose sum over tokens is d temp.
//   2. d_lat: the forward kernel run as its own adjoint (cca_prologue.hip).
//   3. filter gradients: dWc[h,o,d,i] = sum_t d3[t,h,o] * u[t-(D-1-d),h,i] for
//      the folded filter Wc of width D = k_seq + k_ch - 1, as an MFMA
//      contraction over tokens (both operands fetched from row-major LDS tiles
//      with the transposing read), split over chunks of tokens into fp32
//      partial sums that a second kernel adds in a fixed order; Wc is bilinear
//      in (w0, w1), so d w1[h,o,i,j] = sum_jj dWc[h,o,j+jj,i] w0[c,jj] and
//      d w0[c,jj] = sum_o sum_j dWc[h,o,j+jj,i] w1[h,o,i,j].
// No atomics anywhere: a repeated call gives the same bits.
#include "cca_dwc.h"

namespace cca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// from cca_prologue.hip
bool prologue_fused_supported(const Dims &d);
size_t prologue_fused_scratch_bytes(const Dims &d);
PrologueSetup prologue_fused_bwd_setup(const Dims &d, const cca_weights &w, void *scratch);
hipError_t prologue_set_up(const PrologueSetup &setup, hipStream_t s);
hipError_t prologue_fused_bwd_dlat(const Dims &d, const void *d3, const void *d_v, void *d_lat, void *scratch, const DwcArgs *dwc,
                                   hipStream_t s);

namespace {

// ROW below = DH * 2 + 16: padded LDS row of one token, bytes

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

struct PointArgs {
  int T, Hq, Hk, e_q, e_kv;
  long long rows;
  uint32_t flags;
};

// ---------------------------------------------------------------------------
// 1. pointwise: d_h / 8 lanes per (token, head); lane j holds channels 4j..4j+3 and d_h/2 + 4j .. + 3, so the
//    rotate-half partner sits in the same lane and the row dot product is a butterfly over those lanes.
//    PARTS: the attention left dK and dV as fp32 per query head (KvParts); a key item adds its group's dK, in head order, and
//    rounds it once, as group_sum_kernel does, and Hk more items per token add and store dV.  At length the 32-bit
//    halves of dK and dV are read here instead of by a launch of their own (4 us and a bf16 pass less).
// ---------------------------------------------------------------------------
template <int DH, bool PARTS>
__global__ __launch_bounds__(256) void pro_bwd_point_kernel(PointArgs a, KvParts kv, const bf16_t *__restrict__ q,
                                                           const bf16_t *__restrict__ k,
                                                           const float *__restrict__ rnorm,
                                                           const float *__restrict__ temp,
                                                           const bf16_t *__restrict__ dq, const bf16_t *__restrict__ dk,
                                                           const float2 *__restrict__ ropeA,
                                                           const float2 *__restrict__ ropeB, bf16_t *__restrict__ d3,
                                                           float *__restrict__ rowdot) {
  const int NH = a.Hq + a.Hk, NI = PARTS ? NH + a.Hk : NH;
  constexpr int LPI = DH / 8, HALF = DH / 2;  // lanes per item
  const long long item = (long long)blockIdx.x * (256 / LPI) + threadIdx.x / LPI;  // row * NI + head
  const int j = threadIdx.x % LPI;
  const bool live = item < a.rows * NI;
  const long long it = live ? item : 0;
  const long long row = it / NI;
  const int head = (int)(it % NI);
  const int tpos = (int)(row % a.T);
  const bool is_q = head < a.Hq;
  const int g = min(head, NH - 1) - a.Hq;  // (an item of dV leaves before its key row is used)
  const bf16_t *y5 = is_q ? q + (row * a.Hq + head) * DH : k + (row * a.Hk + g) * DH;
  const bf16_t *dy5 = is_q ? dq + (row * a.Hq + head) * DH : dk + (row * a.Hk + g) * DH;
  const u32x2 ya = *reinterpret_cast<const u32x2 *>(y5 + 4 * j), yb = *reinterpret_cast<const u32x2 *>(y5 + HALF + 4 * j);
  u32x2 da, db;
  if (PARTS && !is_q) {
    const int R = a.Hq / a.Hk, gg = head < NH ? g : head - NH;
    const float *p = (head < NH ? kv.k : kv.v) + (row * a.Hq + gg * R) * DH + 4 * j;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
    int r = 0;
    for (; r + 2 <= R; r += 2) {  // two heads' loads in flight
      const f32x4 l0 = *reinterpret_cast<const f32x4 *>(p + r * DH), h0 = *reinterpret_cast<const f32x4 *>(p + r * DH + HALF);
      const f32x4 l1 = *reinterpret_cast<const f32x4 *>(p + r * DH + DH), h1 = *reinterpret_cast<const f32x4 *>(p + r * DH + DH + HALF);
#pragma unroll
      for (int e = 0; e < 4; ++e) lo[e] = lo[e] + l0[e] + l1[e], hi[e] = hi[e] + h0[e] + h1[e];
    }
    if (r < R) {
      const f32x4 l0 = *reinterpret_cast<const f32x4 *>(p + r * DH), h0 = *reinterpret_cast<const f32x4 *>(p + r * DH + HALF);
#pragma unroll
      for (int e = 0; e < 4; ++e) lo[e] += l0[e], hi[e] += h0[e];
    }
    da.x = pack2(lo[0], lo[1]), da.y = pack2(lo[2], lo[3]);
    db.x = pack2(hi[0], hi[1]), db.y = pack2(hi[2], hi[3]);
    if (head >= NH) {
      if (live) {
        bf16_t *const to = kv.d_v + (row * a.Hk + gg) * DH;
        *reinterpret_cast<u32x2 *>(to + 4 * j) = da;
        *reinterpret_cast<u32x2 *>(to + HALF + 4 * j) = db;
      }
      return;
    }
  } else {
    da = *reinterpret_cast<const u32x2 *>(dy5 + 4 * j), db = *reinterpret_cast<const u32x2 *>(dy5 + HALF + 4 * j);
  }
  float y[8] = {bf_lo(ya.x), bf_hi(ya.x), bf_lo(ya.y), bf_hi(ya.y), bf_lo(yb.x), bf_hi(yb.x), bf_lo(yb.y), bf_hi(yb.y)};
  float dy[8] = {bf_lo(da.x), bf_hi(da.x), bf_lo(da.y), bf_hi(da.y), bf_lo(db.x), bf_hi(db.x), bf_lo(db.y), bf_hi(db.y)};
  float dot = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) dot = fmaf(y[e], dy[e], dot);
#pragma unroll
  for (int off = LPI / 2; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
  float mul = 1.f, c = 0.f;
  if (a.flags & CCA_QK_NORM) {
    mul = rnorm[row * NH + head];
    const float beta2 = (!is_q && (a.flags & CCA_KEY_TEMP)) ? expf(2.f * temp[g]) : 1.f;
    c = dot / ((float)DH * beta2);
  }
  if (live && !is_q && rowdot && j == 0) rowdot[row * a.Hk + g] = dot;
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = dy[e] - y[e] * c;
  if (a.flags & CCA_ROPE) {
    const int thi = tpos >> 7, tlo = tpos & 127;
    const f32x4 *pa = reinterpret_cast<const f32x4 *>(ropeA + thi * (DH / 2) + 4 * j);
    const f32x4 *pb = reinterpret_cast<const f32x4 *>(ropeB + (j * 128 + tlo) * 4);
    const f32x4 a01 = pa[0], a23 = pa[1], b01 = pb[0], b23 = pb[1];
    const float ca[4] = {a01.x, a01.z, a23.x, a23.z}, sa[4] = {a01.y, a01.w, a23.y, a23.w};
    const float cb[4] = {b01.x, b01.z, b23.x, b23.z}, sb[4] = {b01.y, b01.w, b23.y, b23.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float cs = ca[e] * cb[e] - sa[e] * sb[e];
      const float sn = sa[e] * cb[e] + ca[e] * sb[e];
      // forward: (x1, x2) -> (x1 c - x2 s, x2 c + x1 s); the adjoint rotates back
      const float g1 = r[e], g2 = r[e + 4];
      r[e] = g1 * cs + g2 * sn;
      r[e + 4] = g2 * cs - g1 * sn;
    }
  }
  if (live) {
    bf16_t *dst = d3 + row * (a.e_q + a.e_kv) + (is_q ? head * DH : a.e_q + g * DH);
    u32x2 lo, hi;
    lo.x = pack2(r[0] * mul, r[1] * mul);
    lo.y = pack2(r[2] * mul, r[3] * mul);
    hi.x = pack2(r[4] * mul, r[5] * mul);
    hi.y = pack2(r[6] * mul, r[7] * mul);
    *reinterpret_cast<u32x2 *>(dst + 4 * j) = lo;
    *reinterpret_cast<u32x2 *>(dst + HALF + 4 * j) = hi;
  }
}

// out[col] = sum over rows of src[row*ncol + col]; one workgroup of 256 threads per column, fixed summation order
struct ColumnSum {
  const float *src;
  float *out;
  long long rows;
  int ncol;  // columns = workgroups; 0: nothing to do
};
__device__ __forceinline__ void column_sum_block(const ColumnSum &c, int col, float *red) {
  const int tid = threadIdx.x;
  float acc = 0.f;
  long long r = tid;
  for (; r + 7 * 256 < c.rows; r += 8 * 256) {  // 8 loads in flight, added in row order
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = c.src[(r + u * 256) * c.ncol + col];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; r < c.rows; r += 256) acc += c.src[r * c.ncol + col];
  red[tid] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) c.out[col] = red[0];
}
__global__ __launch_bounds__(256) void column_sum_f32_kernel(ColumnSum c) {
  __shared__ float red[256];
  column_sum_block(c, blockIdx.x, red);
}

// ---------------------------------------------------------------------------
// 3. folded-filter gradient, partial sums per chunk of tokens: dwc_body (cca_dwc.h), in a launch of its own at d_h = 256, else beside
//    the adjoint of the prologue (prologue_fused_bwd_dlat).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(dwc_threads(256)) void pro_bwd_dwc_kernel(DwcArgs w) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[dwc_lds(256, D)];
  dwc_body<256, D>(w, blockIdx.x, blockIdx.y, threadIdx.x, smem);
}

// The last `csum.ncol` workgroups add the columns of d temp instead (a launch of its own cost 5 us).
// dwc[h][o][d][i] = sum over chunks (fixed order); then d w1[h,o,i,j] = sum_jj dwc[h,o,j+jj,i] * w0[c(h,i),jj]
__global__ __launch_bounds__(256) void pro_bwd_unfold_w1_kernel(const float *__restrict__ part, int n_chunks, int NH,
                                                               int D, int ks, int kc, int use_w0,
                                                               const bf16_t *__restrict__ w0, float *__restrict__ dwc,
                                                               bf16_t *__restrict__ dw1, int DH, ColumnSum csum) {
  __shared__ float red[256];
  if ((int)blockIdx.x >= (int)gridDim.x - csum.ncol) {
    column_sum_block(csum, (int)blockIdx.x - ((int)gridDim.x - csum.ncol), red);
    return;
  }
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;  // (h*DH + o)*DH + i
  if (id >= (long long)NH * DH * DH) return;
  const int i = (int)(id % DH), o = (int)((id / DH) % DH), h = (int)(id / (DH * DH));
  float sum[4] = {0.f, 0.f, 0.f, 0.f};  // D <= 3 on this path
  const long long cstride = (long long)NH * DH * D * DH;
  const float *p0 = part + ((long long)h * DH + o) * D * DH + i;
  int c = 0;
  for (; c + 8 <= n_chunks; c += 8) {  // 8 chunks of loads in flight, added in chunk order
    float v[8][3];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int d = 0; d < 3; ++d) v[u][d] = d < D ? p0[(c + u) * cstride + d * DH] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int d = 0; d < 3; ++d) sum[d] += v[u][d];
  }
  if (c < n_chunks) {  // the rest, again all in flight: past the last chunk they repeat it and are not added
    float v[7][3];
    const float *p = p0 + c * cstride;
#pragma unroll
    for (int u = 0; u < 7; ++u) {
#pragma unroll
      for (int d = 0; d < 3; ++d) v[u][d] = p[(d < D ? d : 0) * DH];
      if (c + u + 1 < n_chunks) p += cstride;
    }
#pragma unroll
    for (int u = 0; u < 7; ++u)
#pragma unroll
      for (int d = 0; d < 3; ++d) sum[d] += c + u < n_chunks ? v[u][d] : 0.f;
  }
  for (int d = 0; d < D; ++d) dwc[(((long long)h * DH + o) * D + d) * DH + i] = sum[d];
  if (!dw1) return;
  for (int j = 0; j < kc; ++j) {
    float acc = 0.f;
    for (int jj = 0; jj < ks; ++jj) {
      const float f0 = use_w0 ? bf16_to_f32(w0[(long long)(h * DH + i) * ks + jj]) : 1.f;
      acc = fmaf(sum[j + jj], f0, acc);
    }
    dw1[(((long long)h * DH + o) * DH + i) * kc + j] = f32_to_bf16(acc);
  }
}

// d w0[c(h,i), jj] = sum_o sum_j dwc[h,o,j+jj,i] * w1[h,o,i,j].  Workgroup = (head, 16 input channels): 8 groups of
// d_h / 8 output channels x 16 input channels; the 8 partial sums are added through LDS in a fixed order.
constexpr int W0_IW = 16;
template <int DH>
__global__ __launch_bounds__(W0_IW * 8) void pro_bwd_unfold_w0_kernel(const float *__restrict__ dwc, int D, int ks, int kc,
                                                                     const bf16_t *__restrict__ w1, bf16_t *__restrict__ dw0) {
  __shared__ float red[8][4][W0_IW];
  const int h = blockIdx.x, il = threadIdx.x % W0_IW, i = blockIdx.y * W0_IW + il, og = threadIdx.x / W0_IW;
  // D = ks + kc - 1 <= 3 on this path: every load of the d_h / 8 output channels is issued before the first use, so the
  // thread waits for memory once instead of once per channel.  Absent taps read the last one and count as zero: a load
  // behind a condition is waited for before the next condition (T = 16384, d_h = 128: 15.6 us that way, 4.8 this way).
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float pv[DH / 8][3], wv[DH / 8][3];
#pragma unroll
  for (int x = 0; x < DH / 8; ++x) {
    const int o = og * (DH / 8) + x;
    const float *p = dwc + (((long long)h * DH + o) * D) * DH + i;
    const bf16_t *wp = w1 + (((long long)h * DH + o) * DH + i) * kc;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      pv[x][t] = p[min(t, D - 1) * DH];
      wv[x][t] = bf16_to_f32(wp[min(t, kc - 1)]);
    }
  }
#pragma unroll
  for (int x = 0; x < DH / 8; ++x)
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int jj = 0; jj < 3; ++jj)
        if (j + jj < 3) acc[jj] = j < kc && j + jj < D ? fmaf(pv[x][j + jj], wv[x][j], acc[jj]) : acc[jj];
  for (int jj = 0; jj < 4; ++jj) red[og][jj][il] = acc[jj];
  __syncthreads();
  if (og == 0)
    for (int jj = 0; jj < ks; ++jj) {
      float sum = 0.f;
      for (int x = 0; x < 8; ++x) sum += red[x][jj][il];
      dw0[(long long)(h * DH + i) * ks + jj] = f32_to_bf16(sum);
    }
}

int taps(const Dims &d) { return ((d.flags & CCA_CONV_SEQ) ? d.k_seq : 1) + d.k_ch - 1; }

int dwc_chunk(const Dims &d) { return filter_gradient_chunk(d.B, d.T, d.Hq + d.Hk, dwc_slices(d.dh, taps(d)), d.dh); }

struct BwdScratch {
  size_t fused, d3, rowdot, part, dwc, total;  // byte offsets
};
BwdScratch bwd_layout(const Dims &d) {
  BwdScratch L;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) / 256 * 256; return o; };
  const int D = taps(d), NH = d.Hq + d.Hk, chunk = dwc_chunk(d), DH = d.dh;
  const size_t n_chunks = (size_t)d.B * ((d.T + chunk - 1) / chunk);
  L.fused = take(prologue_fused_scratch_bytes(d));
  L.d3 = take((size_t)d.rows() * (d.e_q + d.e_kv) * 2);
  L.rowdot = take((size_t)d.rows() * d.Hk * 4);
  L.part = take(n_chunks * NH * DH * D * DH * 4);
  L.dwc = take((size_t)NH * DH * D * DH * 4);
  L.total = off;
  return L;
}

}  // namespace

bool prologue_bwd_fused_supported(const Dims &d) { return prologue_fused_supported(d); }

size_t prologue_bwd_fused_scratch_bytes(const Dims &d) {
  return prologue_bwd_fused_supported(d) ? bwd_layout(d).total : 0;
}

template <int DH>
static hipError_t prologue_bwd_run(const Dims &d, const cca_weights &w, const void *lat, const void *q, const void *k,
                                   const float *rnorm, const void *d_q, const void *d_k, const void *d_v, void *d_lat,
                                   const cca_grads *gr, void *scratch, hipStream_t s, bool set_up, const KvParts *parts) {
  const BwdScratch L = bwd_layout(d);
  char *base = static_cast<char *>(scratch);
  bf16_t *d3 = reinterpret_cast<bf16_t *>(base + L.d3);
  float *rowdot = reinterpret_cast<float *>(base + L.rowdot);
  float *part = reinterpret_cast<float *>(base + L.part);
  float *dwc = reinterpret_cast<float *>(base + L.dwc);
  const int D = taps(d), NH = d.Hq + d.Hk;

  const PrologueSetup setup = prologue_fused_bwd_setup(d, w, base + L.fused);
  hipError_t e = set_up ? hipSuccess : prologue_set_up(setup, s);
  if (e != hipSuccess) return e;

  const bool want_temp = (d.flags & CCA_KEY_TEMP) && gr && gr->temp;
  PointArgs pa{d.T, d.Hq, d.Hk, d.e_q, d.e_kv, d.rows(), d.flags};
  const long long items = d.rows() * (parts ? NH + d.Hk : NH);
  constexpr int IPB = 256 / (DH / 8);  // items per workgroup of the pointwise kernel
  (parts ? pro_bwd_point_kernel<DH, true> : pro_bwd_point_kernel<DH, false>)<<<(unsigned)((items + IPB - 1) / IPB), 256, 0, s>>>(
      pa, parts ? *parts : KvParts{}, (const bf16_t *)q, (const bf16_t *)k, rnorm, w.temp, (const bf16_t *)d_q, (const bf16_t *)d_k,
      setup.ropeA, setup.ropeB, d3, want_temp ? rowdot : nullptr);
  ColumnSum csum{rowdot, want_temp ? gr->temp : nullptr, d.rows(), want_temp ? d.Hk : 0};
  e = hipGetLastError();
  if (e != hipSuccess) return e;

  const bool want_w1 = gr && gr->w_conv_ch;  // CONV_CH is on whenever this path runs
  const bool want_w0 = (d.flags & CCA_CONV_SEQ) && gr && gr->w_conv_seq;
  const int chunk = dwc_chunk(d), cps = (d.T + chunk - 1) / chunk, n_chunks = d.B * cps;
  const DwcArgs dwc_args{d3, (const bf16_t *)lat, part, d.T, d.Hq, d.Hk, d.e_q, d.e_kv, d.n_lat, chunk, cps, n_chunks * NH};
  const bool filters = want_w1 || want_w0;
  e = prologue_fused_bwd_dlat(d, d3, d_v, d_lat, base + L.fused, DH <= 128 && filters ? &dwc_args : nullptr, s);
  if (e != hipSuccess) return e;
  if (!filters) {
    if (want_temp) column_sum_f32_kernel<<<d.Hk, 256, 0, s>>>(csum);
    return hipGetLastError();
  }
  if constexpr (DH == 256) {
    const dim3 grid(n_chunks * NH, dwc_slices(DH, D));
    switch (D) {
      case 1: pro_bwd_dwc_kernel<1><<<grid, dwc_threads(DH), 0, s>>>(dwc_args); break;
      case 2: pro_bwd_dwc_kernel<2><<<grid, dwc_threads(DH), 0, s>>>(dwc_args); break;
      default: pro_bwd_dwc_kernel<3><<<grid, dwc_threads(DH), 0, s>>>(dwc_args); break;
    }
  }
  const int ks = (d.flags & CCA_CONV_SEQ) ? d.k_seq : 1;
  pro_bwd_unfold_w1_kernel<<<(NH * DH * DH + 255) / 256 + csum.ncol, 256, 0, s>>>(part, n_chunks, NH, D, ks, d.k_ch,
                                                                     (d.flags & CCA_CONV_SEQ) ? 1 : 0,
                                                                     (const bf16_t *)w.w_conv_seq, dwc,
                                                                     want_w1 ? (bf16_t *)gr->w_conv_ch : nullptr, DH, csum);
  if (want_w0)
    pro_bwd_unfold_w0_kernel<DH><<<dim3(NH, DH / W0_IW), W0_IW * 8, 0, s>>>(dwc, D, ks, d.k_ch, (const bf16_t *)w.w_conv_ch,
                                               (bf16_t *)gr->w_conv_seq);
  return hipGetLastError();
}

hipError_t prologue_bwd_fused_bf16(const Dims &d, const cca_weights &w, const void *lat, const void *q, const void *k,
                                   const float *rnorm, const void *d_q, const void *d_k, const void *d_v, void *d_lat,
                                   const cca_grads *gr, void *scratch, hipStream_t s, bool set_up, const KvParts *parts) {
  return d.dh == 64    ? prologue_bwd_run<64>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s, set_up, parts)
         : d.dh == 128 ? prologue_bwd_run<128>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s, set_up, parts)
                       : prologue_bwd_run<256>(d, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat, gr, scratch, s, set_up, parts);
}

PrologueSetup prologue_bwd_fused_setup(const Dims &d, const cca_weights &w, void *scratch) {
  return prologue_fused_bwd_setup(d, w, static_cast<char *>(scratch) + bwd_layout(d).fused);
}

}  // namespace cca
