// Fused latent-space prologue for gfx950, bf16 storage (Sec. 2.2: convolution
// equation, qk-mean equation, value-shift equation and the first two lines of
// the final equation block).  One pass over the down-projected latents yields
// the q, k, v that enter attention.
//
// The two causal convolutions have no bias and no nonlinearity between them,
// so conv2_seq+ch(conv1_seq(u)) is one causal convolution of width
// D = k_seq + k_ch - 1 with per-head filters
//     Wc[h,o,i,d] = sum_{j + jj = d} w1[h,o,i,j] * w0[c(h,i),jj].
// A small set-up kernel forms Wc (fp32, rounded once to bf16) and the RoPE
// tables; the main kernel then runs the convolution as a bf16 MFMA
// contraction per head (M = d_h outputs, N = tokens, K = D*d_h), straight on
// the latent rows: the filter of one head lives in LDS for the lifetime of a
// workgroup, the token operands are the latent rows of tokens t-D+1..t.
//
// The MFMA is issued with the filter as its first operand, so each lane ends
// up with half of the d_h output channels of ONE token (the other half-wave has
// the rest; d_h = 128 or 64): the L2 norm is an in-lane sum plus one half-wave exchange, and
// the rotate-half RoPE partner (o, o + d_h/2) sits in the same lane.  The
// qk-mean skip branch is added by the matrix core as well (a scaled identity
// times the pre-conv latent rows), so it needs no loads in another layout.
//
// RoPE angles: t * theta_i is split as (t >> 7) * 128 * theta_i + (t & 127) *
// theta_i; both parts come from tables made in fp64, combined by the angle
// addition formulas in fp32 (an fp32 product t * theta_i alone is off by up to
// 1e-3 rad at t ~ 16k).
#include "cca_internal.h"
#include "cca_dwc.h"
#include "cca_setup.h"
#include "cca_transpose.h"

namespace cca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int NT = 512;
constexpr int MAX_TILES_PER_WAVE = 3;  // a workgroup takes 256 * tiles_per_wave tokens, tiles dealt round-robin

struct FusedArgs {
  int T, Hq, Hk, R, e_q, e_kv, n_lat, v_half, k_seq, k_ch;
  long long rows;
  uint32_t flags;
  int n_conv_blocks;
  int tiles_per_wave;
  float rope_base, norm_eps;
  // Row strides (elements).  Forward: the source is the latent (n_lat), q / k / v are dense.  Backward: the source
  // is the gradient entering the convolutions (e_q + e_kv wide), q / k destinations are column ranges of d_lat,
  // the value role reads d_v (e_kv) and writes the value columns of d_lat.
  int src_stride, q_stride, k_stride, vsrc_stride, vdst_stride;
  // qk-mean weights of the other stream: a q head adds mean_q_other * (k row of its group), a k head adds
  // mean_k_other * (each q row of its group).  Forward 1/2 and 1/(2R); the adjoint swaps them.
  float mean_q_other, mean_k_other;
  // Key-head workgroups come first in the grid and take tiles_per_wave_k tiles per wavefront (a key-head tile
  // costs more: its qk-mean adds the rows of all R query heads of the group); `tiles_per_wave` is the query heads'.
  int n_k_blocks, tiles_per_wave_k;
};

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float lo_f(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// ---------------------------------------------------------------------------
// set-up (cca_setup.h), and the transposes of the projection weights where a pass derives everything at once
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prologue_setup_kernel(PrologueSetup setup, TransposePair weights) {
  __shared__ TransposeTile tile;
  if ((int)blockIdx.x >= setup.n_blocks) transpose_block(weights, blockIdx.x - setup.n_blocks, tile);
  else setup_block(setup, blockIdx.x);
}

// ---------------------------------------------------------------------------
// main kernel: one workgroup = one head x (256 * tiles per wavefront) tokens, 8 wavefronts x 32-token tiles.
// BWD = false: the forward prologue.  BWD = true: its adjoint from the gradient d3 of the conv2 output to
// d_lat: the same contraction with the transposed filter and the taps reaching FORWARD in time (token t reads
// rows t .. t+D-1, zero past the end of its sequence), the qk-mean adjoint through the same identity MFMAs, no
// norm / RoPE (those are undone by a pointwise kernel before), and the value role running the shift backwards.
// ---------------------------------------------------------------------------
// DH = d_h (64 or 128): KK fragments of 16 input channels, NTL tiles of 32 output channels, CPR 16-byte chunks per
// tap of a filter row.
template <int DH, int D, bool BWD>
__device__ __forceinline__ void prologue_fused_body(
    const FusedArgs &a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp,
    bf16_t *__restrict__ q, bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm, int block, unsigned char *smem) {
  constexpr int KK = DH / 16, NTL = DH / 32, CPR = DH / 8;
  constexpr int WROW = D * CPR;  // 16-byte chunks per filter row (one output channel)
  u32x4 *sW = reinterpret_cast<u32x4 *>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;

  if (block >= a.n_conv_blocks) {
    // ---- value-shift role: v[t] = [vc[t] | vp[t-1]], 16 bytes per thread, whole rows per wavefront
    const int cpr = a.e_kv / 8;  // chunks per row
    const long long total = a.rows * cpr;
    const long long first = ((long long)block - a.n_conv_blocks) * (NT * 4);
    for (int it = 0; it < 4; ++it) {
      const long long id = first + it * NT + tid;
      if (id >= total) break;
      const long long row = id / cpr;
      const int ch = (int)(id % cpr) * 8;
      const int t = (int)(row % a.T);
      u32x4 val = {0, 0, 0, 0};
      const bool shifted = (a.flags & CCA_V_SHIFT) && ch >= a.v_half;
      // forward: the shifted half comes from token t-1; adjoint: its gradient goes back to token t, read at t+1
      const bool live = !shifted || (BWD ? t + 1 < a.T : t > 0);
      if (live) val = *reinterpret_cast<const u32x4 *>(vsrc + (row + (shifted ? (BWD ? 1 : -1) : 0)) * a.vsrc_stride + ch);
      *reinterpret_cast<u32x4 *>(v + row * a.vdst_stride + ch) = val;
    }
    return;
  }

  const int NH = a.Hq + a.Hk;
  const bool is_q = block >= a.n_k_blocks;
  const int bid = is_q ? block - a.n_k_blocks : block;
  const int head = is_q ? bid % a.Hq : a.Hq + bid % a.Hk;
  const int tiles_per_wave = is_q ? a.tiles_per_wave : a.tiles_per_wave_k;
  const long long row_begin = (long long)(bid / (is_q ? a.Hq : a.Hk)) * (256 * tiles_per_wave);
  const int g = is_q ? head / a.R : head - a.Hq;
  const int ch0 = is_q ? head * DH : a.e_q + g * DH;

  // ---- filter of this head -> LDS, chunk-swizzled by output channel
  {
    const u32x4 *src = wc + (long long)head * DH * WROW;
#pragma unroll 4
    for (int id = tid; id < DH * WROW; id += NT) {
      const int o = id / WROW, c = id % WROW;
      sW[o * WROW + ((c & ~(CPR - 1)) | ((c ^ o) & (CPR - 1)))] = src[id];
    }
  }
  __syncthreads();  // the only workgroup-wide synchronisation
  const float beta = (!is_q && (a.flags & CCA_KEY_TEMP)) ? expf(temp[g]) : 1.f;
  bf16_t *dst = is_q ? q + head * DH : k + g * DH;
  const int dst_stride = is_q ? a.q_stride : a.k_stride;

  // ---- qk-mean through the matrix core: m = c * I * u adds c times a latent row, already in the
  // accumulator layout, with no extra loads or conversions.  Fragment j of c*I for output tile nt pairs with
  // operand fragment kk = 2*nt + j of the source row; lane (l32, half) is non-zero in fragment l32 >> 4 when
  // (l32 >> 3) & 1 == half, element l32 & 7.
  const bool mean = a.flags & CCA_QK_MEAN;
  // The weight of the other stream, 1/2 or 1/(2R), is an exact mean in the qk-mean equation.  As a single bf16
  // it is exact only for R a power of two, so it is fed as the sum of two bf16 numbers, w = hi + lo (the MFMA forms
  // bf16 products exactly and adds in fp32, so hi*u + lo*u carries w to 2^-17 relative); the second pass is skipped
  // when lo is zero.
  // c * I as fragments: lane (l32, half) holds c in ONE half-word of fragment j = l32 >> 4 (when (l32 >> 3) & 1 == half:
  // element l32 & 7) and zeros elsewhere, so one mask per fragment is kept and c is and-ed in where it is used.
  const float w_other = is_q ? a.mean_q_other : a.mean_k_other;
  const bf16_t w_other_hi = f32_to_bf16(w_other);
  const bf16_t w_other_lo = f32_to_bf16(w_other - bf16_to_f32(w_other_hi));
  const bool grp_lo = (w_other_lo & 0x7fffu) != 0;  // uniform over the workgroup
  u32x4 id_sel[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const bool on = ((l32 >> 4) == j) && (((l32 >> 3) & 1) == half);
    const int e = l32 & 7;
    id_sel[j] = u32x4{0, 0, 0, 0};
    if (on) id_sel[j][e >> 1] = 0xffffu << ((e & 1) * 16);
  }
  auto identity_frag = [&](bf16_t c, int j) {
    const uint32_t cc = (uint32_t)c | ((uint32_t)c << 16);
    const u32x4 w = {id_sel[j].x & cc, id_sel[j].y & cc, id_sel[j].z & cc, id_sel[j].w & cc};
    return __builtin_bit_cast(bf16x8, w);
  };

  for (int tt = 0; tt < tiles_per_wave; ++tt) {
    const long long trow0 = row_begin + (tt * 8 + wave) * 32;
    if (trow0 >= a.rows) break;  // wave-uniform; nothing below synchronises across wavefronts
    const long long row = trow0 + l32;
    const long long rowc = row < a.rows ? row : a.rows - 1;
    const int tpos = (int)(rowc % a.T);
    // Taps outside the token's sequence contribute zeros.  Only the first (adjoint: last) tile of a sequence
    // has such taps: everywhere else the loads are unconditional and all in flight together.
    const bool any_pad = __any(BWD ? tpos + D - 1 >= a.T : tpos < D - 1) != 0;

    // ---- operands: source rows of tokens t-D+1 .. t (adjoint: t .. t+D-1) of this head.  The taps of a tile are
    //      the same 32 rows shifted by a token, so the rows are fetched ONCE, whole (16 bytes per lane, 64 / CPR rows
    //      per load instruction: every cache line touched is used in full), parked in this wavefront's staging rows
    //      in LDS (chunk c of row r at position c ^ (r mod CPR)) and read from there as MFMA fragments, tap by tap.
    //      Fetched as fragments straight from memory, each tap cost 8 load instructions that touch 32 rows with 32
    //      bytes each; the vector memory pipeline works per cache line touched (timing without the D-1 earlier taps'
    //      loads: 56 -> 46 us).  The D-1 rows before the tile (adjoint: after it) are handled below (`halo`).
    constexpr int RPI = 64 / CPR, NLD = 32 / RPI, ROWB = DH * 2;
    unsigned char *const stg = smem + (size_t)DH * WROW * 16 + wave * (32 * ROWB);
    // Addresses of the whole-row transfers: a wave-uniform pointer to the tile's first row plus a 32-bit offset per
    // lane (row it * RPI + lane / CPR of the tile, clamped to the last row of the tensor on a ragged last tile).
    const int rows_left = (int)(a.rows - trow0 < 32 ? a.rows - trow0 : 32);  // >= 1
    auto stage_rows = [&](const bf16_t *tile_src, int stride) {  // rows of `tile_src` -> staging rows (swizzled)
      u32x4 rreg[NLD];
#pragma unroll
      for (int it = 0; it < NLD; ++it) {
        const int rr = it * RPI + lane / CPR, p = lane % CPR, c = p ^ (rr & (CPR - 1));
        const int rs = rr < rows_left ? rr : rows_left - 1;
        rreg[it] = *reinterpret_cast<const u32x4 *>(tile_src + rs * stride + c * 8);
      }
#pragma unroll
      for (int it = 0; it < NLD; ++it) {
        const int rr = it * RPI + lane / CPR, p = lane % CPR;
        *reinterpret_cast<u32x4 *>(stg + rr * ROWB + p * 16) = rreg[it];
      }
    };
    stage_rows(lat + trow0 * a.src_stride + ch0, a.src_stride);
    // The D-1 rows before the tile (adjoint: after it), which the first (last) D-1 tokens' taps reach: fetched whole as
    // well, one 16-byte chunk per lane - halo row j, chunk c in lane j * CPR + c - and handed to the lane that needs a
    // fragment of them by a lane gather (4 registers instead of a set of fragments in every lane).
    u32x4 halo = {0, 0, 0, 0};
    if (D > 1 && lane < (D - 1) * CPR) {
      const long long lo = -trow0, hi = a.rows - 1 - trow0;  // clamped in bounds; a clamped row is zeroed below:
      int hrel = BWD ? 32 + lane / CPR : lane / CPR - (D - 1);  // it lies outside the token's sequence
      hrel = hrel < lo ? (int)lo : (hrel > hi ? (int)hi : hrel);
      const bf16_t *tile_src = lat + trow0 * a.src_stride + ch0;  // wave-uniform
      halo = *reinterpret_cast<const u32x4 *>(tile_src + hrel * a.src_stride + (lane % CPR) * 8);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS handles a wavefront's accesses in order
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // fragment kk of tap `back` for this lane's token: row l32 -+ back of the tile, or the halo row
    auto row_frag = [&](auto back_c, int kk, int l32v) {
      constexpr int back = decltype(back_c)::value;
      const int r = BWD ? l32v + back : l32v - back;
      const bool inside = BWD ? r < 32 : r >= 0;
      const int rc = inside ? r : l32v;  // the lanes that take the halo read their own row and drop it
      u32x4 raw = *reinterpret_cast<const u32x4 *>(stg + rc * ROWB + (((2 * kk + half) ^ (rc & (CPR - 1))) * 16));
      if constexpr (back > 0) {
        // halo row of this lane's tap: index r + (D-1) (adjoint: r - 32); its chunk 2 kk + half sits in lane
        // index * CPR + chunk (the index is clamped for the lanes that do not take the halo)
        int hj = BWD ? r - 32 : r + (D - 1);
        hj = hj < 0 ? 0 : (hj > D - 2 ? D - 2 : hj);
        const int src = (hj * CPR + 2 * kk + half) * 4;
        u32x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)halo[e]);
        if (!inside) raw = h;
      }
      return __builtin_bit_cast(bf16x8, raw);
    };

    // ---- y1^T = Wc * [u(t-D+1) .. u(t)]^T
    f32x16 acc[NTL];
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;
    bf16x8 uf[KK];  // the fragments of the tap being multiplied; after the loop: the token's own row (back = 0)
    auto conv_tap = [&](auto d_c) {
      constexpr int d = decltype(d_c)::value;
      constexpr int back = D - 1 - d;
      // the LDS addresses of a tap (one per k-step: the swizzle is an XOR, not an offset) are formed here, per tap
      // and tile, from a copy of the lane index the compiler cannot see through: hoisted out of the tile loop as
      // loop invariants they cost 8 registers per tap for the whole kernel
      int l32v = l32;
      asm volatile("" : "+v"(l32v));
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) uf[kk] = row_frag(std::integral_constant<int, back>{}, kk, l32v);
      if (back > 0 && any_pad) {  // wave-uniform and rare: a tap that reaches outside the token's sequence is zero
        const bool outside = BWD ? tpos + back >= a.T : tpos < back;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          if (outside) uf[kk] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
      }
      // the tap's KK * NTL products in a fixed order, the filter fragment of product i + PFW requested before product
      // i is issued (left to the compiler each fragment is read, waited for and consumed one at a time, and the LDS
      // latency of every read is paid in full)
      constexpr int NPW = KK * NTL, PFW = 4;
      bf16x8 wfr[PFW + 1];  // ring: fragment i lives in slot i mod (PFW + 1)
      auto fetch_w = [&](int i) {
        const int kk = i / NTL, nt = i % NTL;
        const int o = nt * 32 + l32v;
        const int c = d * CPR + kk * 2 + half;
        wfr[i % (PFW + 1)] = __builtin_bit_cast(bf16x8, sW[o * WROW + ((c & ~(CPR - 1)) | ((c ^ o) & (CPR - 1)))]);
      };
#pragma unroll
      for (int i = 0; i < PFW; ++i) fetch_w(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NPW; ++i) {
        if (i + PFW < NPW) fetch_w(i + PFW);
        acc[i % NTL] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfr[i % (PFW + 1)], uf[i / NTL], acc[i % NTL], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);  // one tap's fragments at a time: the next tap's reads stay behind this one's products
    };
    conv_tap(std::integral_constant<int, 0>{});
    if constexpr (D > 1) conv_tap(std::integral_constant<int, 1>{});
    if constexpr (D > 2) conv_tap(std::integral_constant<int, 2>{});

    // ---- qk-mean.  q head: + (q0 + k0[g]) / 2.  k head: + (mean_r q0[gR + r] + k0) / 2.
    //      Adjoint: q head + d3_q / 2 + d3_k[g] / (2R);  k head: + (sum_r d3_q[gR + r] + d3_k) / 2.
    if (mean) {
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(identity_frag(f32_to_bf16(0.5f), j), uf[2 * nt + j], acc[nt], 0, 0, 0);
      const int nsrc = is_q ? 1 : a.R;
      for (int sidx = 0; sidx < nsrc; ++sidx) {
        // the other stream's rows of this tile travel like the tile's own: whole rows -> staging rows -> fragments
        const int col = is_q ? a.e_q + g * DH : (g * a.R + sidx) * DH;
        __builtin_amdgcn_sched_barrier(0);  // not hoisted above the products before: their registers are needed there
        stage_rows(lat + trow0 * a.src_stride + col, a.src_stride);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int l32v = l32;
        asm volatile("" : "+v"(l32v));
        bf16x8 mf[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          mf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
                                                  stg + l32v * ROWB + (((2 * kk + half) ^ (l32v & (CPR - 1))) * 16)));
#pragma unroll
        for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(identity_frag(w_other_hi, j), mf[2 * nt + j], acc[nt], 0, 0, 0);
        if (grp_lo) {
#pragma unroll
          for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(identity_frag(w_other_lo, j), mf[2 * nt + j], acc[nt], 0, 0, 0);
        }
      }
    }

    __builtin_amdgcn_sched_barrier(0);
    // ---- per token: norm, temperature, RoPE.  Lane (l32, half) holds channels
    //      o = 32*nt + 8*rg + 4*half + e of token l32 in acc[nt][4*rg + e].
    if (!BWD && (a.flags & CCA_QK_NORM)) {
      float ssq = 0.f;
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) ssq = fmaf(acc[nt][r], acc[nt][r], ssq);
      ssq += __shfl_xor(ssq, 32);
      const float mul = sqrtf((float)DH) / sqrtf(ssq + a.norm_eps) * beta;
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nt][r] *= mul;
      if (rnorm && half == 0 && row < a.rows) rnorm[row * NH + head] = mul;
    } else if (!BWD && rnorm && half == 0 && row < a.rows) {
      rnorm[row * NH + head] = 1.f;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!BWD && (a.flags & CCA_ROPE)) {
      const int thi = tpos >> 7, tlo = tpos & 127;
#pragma unroll
      for (int nt = 0; nt < NTL / 2; ++nt)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const int i0 = nt * 32 + rg * 8 + half * 4;  // 4 consecutive pair indices
          const f32x4 *pa = reinterpret_cast<const f32x4 *>(ropeA + thi * (DH / 2) + i0);
          const f32x4 *pb = reinterpret_cast<const f32x4 *>(ropeB + ((i0 >> 2) * 128 + tlo) * 4);
          const f32x4 a01 = pa[0], a23 = pa[1], b01 = pb[0], b23 = pb[1];
          const float ca[4] = {a01.x, a01.z, a23.x, a23.z}, sa[4] = {a01.y, a01.w, a23.y, a23.w};
          const float cb[4] = {b01.x, b01.z, b23.x, b23.z}, sb[4] = {b01.y, b01.w, b23.y, b23.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float cs = ca[e] * cb[e] - sa[e] * sb[e];
            const float sn = sa[e] * cb[e] + ca[e] * sb[e];
            const float x1 = acc[nt][rg * 4 + e], x2 = acc[nt + NTL / 2][rg * 4 + e];
            acc[nt][rg * 4 + e] = x1 * cs - x2 * sn;
            acc[nt + NTL / 2][rg * 4 + e] = x2 * cs + x1 * sn;
          }
        }
    }
    // ---- round once to bf16 and store.  In the accumulator layout a lane holds 4 consecutive channels (8 bytes) of
    //      one token per (nt, rg): stored from there, a wavefront's store instruction would touch 32 rows with 16
    //      bytes each, and the vector memory pipeline works per cache line touched (timing the kernel with 1 such
    //      store per lane instead of 16: 56 -> 45 us).  So the tile is transposed through this wavefront's private
    //      staging rows in LDS (16-byte chunk c of row r at position c ^ (r mod CPR): conflict-free both ways) and
    //      leaves as whole rows, 16 bytes per lane, 64 / CPR rows per instruction.
    {
      int l32w = l32;  // as for the tap reads: the 16 swizzled positions are formed here, not kept across tiles
      asm volatile("" : "+v"(l32w));
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          u32x2 w;
          w.x = pack2(acc[nt][rg * 4 + 0], acc[nt][rg * 4 + 1]);
          w.y = pack2(acc[nt][rg * 4 + 2], acc[nt][rg * 4 + 3]);
          const int pos = (nt * 4 + rg) ^ (l32w & (CPR - 1));
          *reinterpret_cast<u32x2 *>(stg + l32w * (DH * 2) + pos * 16 + half * 8) = w;
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS handles a wavefront's accesses in order
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      bf16_t *const tile_dst = dst + trow0 * dst_stride;
#pragma unroll
      for (int it = 0; it < 32 / RPI; ++it) {
        const int rr = it * RPI + lane / CPR, p = lane % CPR, c = p ^ (rr & (CPR - 1));
        const u32x4 val = *reinterpret_cast<const u32x4 *>(stg + rr * (DH * 2) + p * 16);
        if (rr < rows_left) *reinterpret_cast<u32x4 *>(tile_dst + rr * dst_stride + c * 8) = val;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // the next tile's writes come after these reads
      __builtin_amdgcn_wave_barrier();
    }
  }
}

template <int DH, int D, bool BWD>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void prologue_fused_kernel(
    FusedArgs a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp,
    bf16_t *__restrict__ q, bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  prologue_fused_body<DH, D, BWD>(a, lat, vsrc, wc, ropeA, ropeB, temp, q, k, v, rnorm, blockIdx.x, smem);
}

// The adjoint and, beside it, the partial sums of the filter gradients (cca_dwc.h; two units of 256 threads to a workgroup at d_h = 64):
// both follow from d3 alone, and on short sequences each leaves most CUs idle.  Workgroups [0, n_adjoint) do the former.  Backward
// pass, the prologue's adjoint in seven launches -> four (us; set-up beside Delta, group sums in the pointwise pass, these two
// together): 2 x 512 tokens, 8 query and 2 KV heads of 128: 121.9 -> 109.9; 1 x 512, 8 heads of 64: 62.5 -> 54.3; 2 x 4096: 621 -> 596.
template <int DH, int D>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void prologue_adjoint_pair_kernel(
    FusedArgs a, const bf16_t *__restrict__ d3, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc, bf16_t *__restrict__ dq,
    bf16_t *__restrict__ dk, bf16_t *__restrict__ dv, DwcArgs w, int n_adjoint) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x < n_adjoint) {
    prologue_fused_body<DH, D, true>(a, d3, vsrc, wc, nullptr, nullptr, nullptr, dq, dk, dv, nullptr, blockIdx.x, smem);
  } else {
    constexpr int PER = NT / dwc_threads(DH);
    const int sub = PER == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / dwc_threads(DH));
    dwc_body<DH, D, (PER > 1)>(w, ((int)blockIdx.x - n_adjoint) * PER + sub, 0, threadIdx.x % dwc_threads(DH), smem + sub * dwc_lds(DH, D));
  }
}

// ---------------------------------------------------------------------------
// The same prologue for d_h = 256, where one head's folded filter (D x 256 x 256 bf16 = 128 KB per tap) cannot
// stay in LDS: the filter is STREAMED through a ring of four LDS slabs (16 KB each, requested straight into LDS with
// one bare barrier per slab), all 4 wavefronts of a workgroup walking the slabs in step.  Workgroup = one head x 128
// tokens, wavefront = 32 tokens x all 256 outputs (8 accumulator tiles), one wavefront per SIMD.  The token rows of a
// wavefront (its 32 and the D - 1 its taps reach) are fetched once, whole, into its own staging rows in LDS and read
// from there tap by tap, and results leave through the same rows: as fragments straight from memory a load instruction
// touches 32 rows with 32 bytes each, and the memory pipeline takes about 4.6 cycles per cache line.
// With one wavefront per SIMD nothing else covers a wait, so the fragments of one k-step are read between the products
// of the one before (a slab's barrier stands between its two k-steps, so the next slab's come as early), the rows of the
// qk-mean's other stream follow the filter through the ring as further slabs, and the rotary table's entries are on
// their way under the norm.  Read, multiplied and rotated one after the other: 16 workgroups 24.4 us, now 17.6 (adjoint
// 19.3 and 15.0); 235 (6000 tokens, 4 / 1 heads, one per CU) 32.8 and 27.5 (28.5 and 25.4), where the row traffic,
// 45 MB that all workgroups ask for at the same times, is the larger part; 3000 tokens, 8 / 2 heads, 32.7 and 27.3.
// In LDS a slab's reads take 576 cycles, its products 512.
// BWD = true is the adjoint, as for the kernel above:
// transposed filter, taps reaching forward in time, the value shift running backwards; the host passes only the
// qk-mean and value-shift flags, so the norm and RoPE steps are skipped.
// ---------------------------------------------------------------------------
constexpr int ST_NT = 256, ST_WAVES = ST_NT / 64, ST_RING = 4;
constexpr int stream_rows(int D) { return (32 + D - 1 + 1) / 2 * 2; }  // staged rows of a wavefront, whole load instructions
constexpr size_t stream_lds(int D) { return (size_t)ST_RING * SLAB_BYTES + (size_t)ST_WAVES * stream_rows(D) * 512; }

// ---- pieces of the two d_h = 256 kernels
// Value role: 4 x NTH chunks of 16 bytes from `first` on; the shifted half of the channels one token later (adjoint: earlier).
template <bool BWD, int NTH>
__device__ __forceinline__ void value_role(const FusedArgs &a, const bf16_t *__restrict__ vsrc, bf16_t *__restrict__ v, long long first) {
  const int cpr = a.e_kv / 8;
  const long long total = a.rows * cpr;
  for (int it = 0; it < 4; ++it) {
    const long long id = first + it * NTH + threadIdx.x;
    if (id >= total) break;
    const long long row = id / cpr;
    const int ch = (int)(id % cpr) * 8;
    const int t = (int)(row % a.T);
    u32x4 val = {0, 0, 0, 0};
    const bool shifted = (a.flags & CCA_V_SHIFT) && ch >= a.v_half;
    const bool live = !shifted || (BWD ? t + 1 < a.T : t > 0);
    if (live) val = *reinterpret_cast<const u32x4 *>(vsrc + (row + (shifted ? (BWD ? 1 : -1) : 0)) * a.vsrc_stride + ch);
    *reinterpret_cast<u32x4 *>(v + row * a.vdst_stride + ch) = val;
  }
}

// ---------------------------------------------------------------------------
// The prologue of short sequences, d_h = 64 and 128.  What bounds the kernel above there is one workgroup's chain: the filter in three
// batches, the rows, R partner rows one after the other, the RoPE tables, each a memory latency, and 256 tokens on one CU while
// most are idle.  Here a workgroup takes 64 tokens of one head with d_h / 16 wavefronts, wavefront = 32 tokens x 32 output channels,
// and asks for everything it reads at once: the filter (straight into LDS), the token rows and the halo, the partner rows and the RoPE
// table entries.  The sums of a token meet in LDS as fp32, where d_h / 16 lanes take its norm, rotate and store.
// Prologue with its set-up, the kernel above -> this one, us: 1 x 512 tokens, 8 query and 2 KV heads of 128: 18.8 -> 12.4; 8 + 1 heads:
// 21.0 -> 13.9; 16 + 4 heads of 64: 11.8 -> 8.7.  Prologue's adjoint with its gradients: 35.5 -> 31.8, 37.7 -> 32.3, 27.0 -> 24.0.
// ---------------------------------------------------------------------------
constexpr int SH_TOK = 64, SH_SRC = 4;  // tokens of a workgroup; partner rows requested at a time
constexpr size_t short_u_bytes(int DH, int D) { return (size_t)(SH_TOK + D - 1) * (DH * 2 + 16); }
constexpr size_t short_lds(int DH, int D) {
  return (size_t)DH * D * DH * 2 + short_u_bytes(DH, D) + (size_t)SH_TOK * (DH + 4) * sizeof(float);
}

template <int DH, int D, bool BWD, bool IS_Q>
__device__ __forceinline__ void prologue_short_head(
    const FusedArgs &a, const bf16_t *__restrict__ lat, const u32x4 *__restrict__ wc, const float2 *__restrict__ ropeA,
    const float2 *__restrict__ ropeB, const float *__restrict__ temp, bf16_t *__restrict__ dst_, float *__restrict__ rnorm, int bid,
    unsigned char *smem) {
  constexpr int NTH = DH * 4, NW = NTH / 64, KK = DH / 16, NTL = DH / 32, CPR = DH / 8, WROW = D * CPR;
  constexpr int UROW = DH * 2 + 16, XROW = DH + 4, U_CHUNKS = (SH_TOK + D - 1) * CPR, NU = (U_CHUNKS + NTH - 1) / NTH;
  constexpr int W_LOADS = DH * WROW / 64 / NW, LPT = DH / 16;  // load instructions of a wavefront; lanes of a token at the end
  unsigned char *const sW = smem, *const sU = sW + DH * WROW * 16;
  float *const sX = reinterpret_cast<float *>(sU + short_u_bytes(DH, D));
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = wave % NTL, rg = wave / NTL;
  const int n_heads = IS_Q ? a.Hq : a.Hk, hl = bid % n_heads, head = IS_Q ? hl : a.Hq + hl, g = IS_Q ? hl / a.R : hl;
  const long long row0 = (long long)(bid / n_heads) * SH_TOK, last = a.rows - 1;
  const int ch0 = IS_Q ? hl * DH : a.e_q + g * DH;
  const long long row = row0 + rg * 32 + l32, rowc = row < last ? row : last;
  const int tk = tid / LPT, i0 = tid % LPT * 8;  // the token and the pairs of channels this lane finishes
  const long long rowf = row0 + tk, rowfc = rowf < last ? rowf : last;

  // ---- requests
  u32x4 u[NU];
#pragma unroll
  for (int i = 0; i < NU; ++i) {  // rows outside the tensor repeat its first or last: the taps that reach them are zeroed below
    const int id = min(tid + i * NTH, U_CHUNKS - 1), r = id / CPR;
    long long gr = BWD ? row0 + r : row0 + r - (D - 1);
    gr = gr < 0 ? 0 : gr > last ? last : gr;
    u[i] = *reinterpret_cast<const u32x4 *>(lat + gr * a.src_stride + ch0 + id % CPR * 8);
  }
  const int n_src = IS_Q ? 1 : a.R;
  constexpr int NS = IS_Q ? 1 : SH_SRC;
  u32x4 mf[NS][2];
  auto request_sources = [&](int s0) {  // sources past the last repeat it and are not added
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int col = IS_Q ? a.e_q + g * DH : (g * a.R + min(s0 + s, n_src - 1)) * DH;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        mf[s][j] = *reinterpret_cast<const u32x4 *>(lat + rowc * a.src_stride + col + ((2 * nt + j) * 2 + half) * 8);
    }
  };
  request_sources(0);
  f32x4 pa[4], pb[4];
  float beta = 1.f;
  if constexpr (!BWD) {  // (the tables are set up whatever the flags)
    const int tpos = (int)(rowfc % a.T), thi = tpos >> 7, tlo = tpos & 127;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      pa[e] = reinterpret_cast<const f32x4 *>(ropeA + thi * (DH / 2) + i0)[e];
      pb[e] = reinterpret_cast<const f32x4 *>(ropeB + (((i0 >> 2) + (e >> 1)) * 128 + tlo) * 4)[e & 1];
    }
    if (!IS_Q && (a.flags & CCA_KEY_TEMP)) beta = expf(temp[g]);
  }
  {
    typedef __attribute__((address_space(3))) void lds_void;
    typedef __attribute__((address_space(1))) void glb_void;
    const u32x4 *const src = wc + (long long)head * DH * WROW;
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i) {  // instruction p of the filter deposits chunks [64 p, 64 p + 64): chunk c of row o at c ^ o
      const int at = (i * NW + wave) * 64 + lane, o = at / WROW, c = at % WROW;
      __builtin_amdgcn_global_load_lds((glb_void *)(src + o * WROW + ((c & ~(CPR - 1)) | ((c ^ o) & (CPR - 1)))),
                                       (lds_void *)(sW + (i * NW + wave) * 1024), 16, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < NU; ++i) {
    const int id = tid + i * NTH;
    if (id < U_CHUNKS) *reinterpret_cast<u32x4 *>(sU + id / CPR * UROW + id % CPR * 16) = u[i];
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // ---- this wavefront's 32 channels of 32 tokens: the taps in order, then the means, all on one accumulator
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int tposw = (int)(rowc % a.T), o = nt * 32 + l32;
  const unsigned char *const ur = sU + (rg * 32 + l32 + (BWD ? 0 : D - 1)) * UROW + half * 16;  // the token's own row
  auto tap = [&](auto d_c) {
    constexpr int d = decltype(d_c)::value, back = D - 1 - d;
    const bool outside = BWD ? tposw + back >= a.T : tposw < back;  // reaches out of the token's sequence
    const unsigned char *const row_at = ur + (BWD ? back : -back) * UROW;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      u32x4 x = *reinterpret_cast<const u32x4 *>(row_at + kk * 32);
      if (back > 0 && outside) x = u32x4{0, 0, 0, 0};
      const int c = d * CPR + kk * 2 + half;
      const u32x4 w = *reinterpret_cast<const u32x4 *>(sW + (o * WROW + ((c & ~(CPR - 1)) | ((c ^ o) & (CPR - 1)))) * 16);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
    }
  };
  tap(std::integral_constant<int, 0>{});
  if constexpr (D > 1) tap(std::integral_constant<int, 1>{});
  if constexpr (D > 2) tap(std::integral_constant<int, 2>{});
  if (a.flags & CCA_QK_MEAN) {  // c * I times the rows (prologue_fused_body): lane (l32, half) holds c in element l32 & 7 of one fragment
    const float w_other = IS_Q ? a.mean_q_other : a.mean_k_other;
    const bf16_t hi = f32_to_bf16(w_other), lo = f32_to_bf16(w_other - bf16_to_f32(hi));
    auto add = [&](bf16_t c, int j, u32x4 x) {
      const uint32_t cc = ((l32 >> 4) == j && ((l32 >> 3) & 1) == half) ? (uint32_t)c << (l32 & 1) * 16 : 0u;
      const int e = (l32 & 7) >> 1;
      const u32x4 w = {e == 0 ? cc : 0u, e == 1 ? cc : 0u, e == 2 ? cc : 0u, e == 3 ? cc : 0u};
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < 2; ++j) add(f32_to_bf16(0.5f), j, *reinterpret_cast<const u32x4 *>(ur + (2 * nt + j) * 32));
    for (int s0 = 0;;) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (s0 + s >= n_src) break;
#pragma unroll
        for (int j = 0; j < 2; ++j) add(hi, j, mf[s][j]);
        if ((lo & 0x7fffu) != 0) {
#pragma unroll
          for (int j = 0; j < 2; ++j) add(lo, j, mf[s][j]);
        }
      }
      s0 += NS;
      if (s0 >= n_src) break;
      request_sources(s0);
    }
  }
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const f32x4 x = {acc[q4 * 4], acc[q4 * 4 + 1], acc[q4 * 4 + 2], acc[q4 * 4 + 3]};
    *reinterpret_cast<f32x4 *>(sX + (rg * 32 + l32) * XROW + nt * 32 + q4 * 8 + half * 4) = x;
  }
  __syncthreads();

  // ---- per token: norm, temperature, RoPE, one rounding
  float x1[8], x2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x1[e] = sX[tk * XROW + i0 + e], x2[e] = sX[tk * XROW + DH / 2 + i0 + e];
  if constexpr (!BWD) {
    float mul = 1.f;
    if (a.flags & CCA_QK_NORM) {
      float ssq = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) ssq = fmaf(x1[e], x1[e], fmaf(x2[e], x2[e], ssq));
#pragma unroll
      for (int m = 1; m < LPT; m *= 2) ssq += __shfl_xor(ssq, m);
      mul = sqrtf((float)DH) / sqrtf(ssq + a.norm_eps) * beta;
#pragma unroll
      for (int e = 0; e < 8; ++e) x1[e] *= mul, x2[e] *= mul;
    }
    if (rnorm && i0 == 0 && rowf <= last) rnorm[rowf * (a.Hq + a.Hk) + head] = mul;
    if (a.flags & CCA_ROPE) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ca = pa[e >> 1][(e & 1) * 2], sa = pa[e >> 1][(e & 1) * 2 + 1], cb = pb[e >> 1][(e & 1) * 2], sb = pb[e >> 1][(e & 1) * 2 + 1];
        const float cs = ca * cb - sa * sb, sn = sa * cb + ca * sb, y1 = x1[e], y2 = x2[e];
        x1[e] = y1 * cs - y2 * sn;
        x2[e] = y2 * cs + y1 * sn;
      }
    }
  }
  if (rowf <= last) {
    bf16_t *const to = dst_ + hl * DH + rowf * (IS_Q ? a.q_stride : a.k_stride) + i0;
    *reinterpret_cast<u32x4 *>(to) = u32x4{pack2(x1[0], x1[1]), pack2(x1[2], x1[3]), pack2(x1[4], x1[5]), pack2(x1[6], x1[7])};
    *reinterpret_cast<u32x4 *>(to + DH / 2) = u32x4{pack2(x2[0], x2[1]), pack2(x2[2], x2[3]), pack2(x2[4], x2[5]), pack2(x2[6], x2[7])};
  }
}

template <int DH, int D, bool BWD>
__device__ __forceinline__ void prologue_short_body(
    const FusedArgs &a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp, bf16_t *__restrict__ q,
    bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm, int block, unsigned char *smem) {
  if (block >= a.n_conv_blocks) value_role<BWD, DH * 4>(a, vsrc, v, ((long long)block - a.n_conv_blocks) * (DH * 16));
  else if (block < a.n_k_blocks) prologue_short_head<DH, D, BWD, false>(a, lat, wc, ropeA, ropeB, temp, k, rnorm, block, smem);
  else prologue_short_head<DH, D, BWD, true>(a, lat, wc, ropeA, ropeB, temp, q, rnorm, block - a.n_k_blocks, smem);
}

template <int DH, int D, bool BWD>
__global__ __launch_bounds__(DH * 4) void prologue_short_kernel(
    FusedArgs a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp,
    bf16_t *__restrict__ q, bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  prologue_short_body<DH, D, BWD>(a, lat, vsrc, wc, ropeA, ropeB, temp, q, k, v, rnorm, blockIdx.x, smem);
}

// Its adjoint beside the filter gradients' partial sums, as prologue_adjoint_pair_kernel (a unit is a workgroup's d_h * 4 threads)
template <int DH, int D>
__global__ __launch_bounds__(DH * 4) void prologue_short_pair_kernel(
    FusedArgs a, const bf16_t *__restrict__ d3, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc, bf16_t *__restrict__ dq,
    bf16_t *__restrict__ dk, bf16_t *__restrict__ dv, DwcArgs w, int n_adjoint) {
  static_assert(dwc_threads(DH) == DH * 4, "threads of both roles");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x < n_adjoint)
    prologue_short_body<DH, D, true>(a, d3, vsrc, wc, nullptr, nullptr, nullptr, dq, dk, dv, nullptr, blockIdx.x, smem);
  else
    dwc_body<DH, D>(w, (int)blockIdx.x - n_adjoint, 0, threadIdx.x, smem);
}

// The workgroup's head and its streams
struct StreamHead {
  bool is_q;
  int bid, head, g, ch0;
  __device__ __forceinline__ explicit StreamHead(const FusedArgs &a) {
    is_q = (int)blockIdx.x >= a.n_k_blocks;
    bid = is_q ? (int)blockIdx.x - a.n_k_blocks : (int)blockIdx.x;
    head = is_q ? bid % a.Hq : a.Hq + bid % a.Hk;
    g = is_q ? head / a.R : head - a.Hq;
    ch0 = is_q ? head * 256 : a.e_q + g * 256;
    bid /= is_q ? a.Hq : a.Hk;  // token block
  }
};

// Per token: norm, temperature, RoPE (lane (l32, half): channels 32*nt + 8*rg + 4*half + e).  The table entries of AHEAD of the 16 groups
// of pairs are on their way at a time, the first ones under the norm: fetched group by group they were 16 latencies one after the other,
// 6 us of the 128-token kernel (0: they are, where registers are short and the SIMD has another wavefront)
template <int AHEAD>
__device__ __forceinline__ void norm_and_rope_256(f32x16 (&acc)[8], const FusedArgs &a, int head, float beta, long long row, int tpos,
                                                  int half, const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB,
                                                  float *__restrict__ rnorm) {
  constexpr int DH = 256, NTL = DH / 32, GROUPS = NTL / 2 * 4;
  const int NH = a.Hq + a.Hk;
  const bool rope = a.flags & CCA_ROPE;
  f32x4 table[AHEAD ? AHEAD : 1][4];
  const int thi = tpos >> 7, tlo = tpos & 127;
  auto fetch = [&](int i) __attribute__((always_inline)) {
    const int i0 = i * 8 + half * 4;  // 4 consecutive pair indices
    const f32x4 *pa = reinterpret_cast<const f32x4 *>(ropeA + thi * (DH / 2) + i0);
    const f32x4 *pb = reinterpret_cast<const f32x4 *>(ropeB + ((i0 >> 2) * 128 + tlo) * 4);
    f32x4 (&t)[4] = table[AHEAD ? i % AHEAD : 0];
    t[0] = pa[0], t[1] = pa[1], t[2] = pb[0], t[3] = pb[1];
    if (AHEAD) __builtin_amdgcn_sched_barrier(0);
  };
  if (rope) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(i);
  }
  if (a.flags & CCA_QK_NORM) {
    float ssq = 0.f;
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) ssq = fmaf(acc[nt][r], acc[nt][r], ssq);
    ssq += __shfl_xor(ssq, 32);
    const float mul = sqrtf((float)DH) / sqrtf(ssq + a.norm_eps) * beta;
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nt][r] *= mul;
    if (rnorm && half == 0 && row < a.rows) rnorm[row * NH + head] = mul;
  } else if (rnorm && half == 0 && row < a.rows) {
    rnorm[row * NH + head] = 1.f;
  }
  if (rope) {
#pragma unroll
    for (int i = 0; i < GROUPS; ++i) {
      const int nt = i / 4, rg = i % 4;
      if (!AHEAD) fetch(i);
      const f32x4 (&t)[4] = table[AHEAD ? i % AHEAD : 0];
      const float ca[4] = {t[0].x, t[0].z, t[1].x, t[1].z}, sa[4] = {t[0].y, t[0].w, t[1].y, t[1].w};
      const float cb[4] = {t[2].x, t[2].z, t[3].x, t[3].z}, sb[4] = {t[2].y, t[2].w, t[3].y, t[3].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // (which product is rounded is written out: left to the compiler it differed between groups)
        const float cs = fmaf(ca[e], cb[e], -(sa[e] * sb[e]));
        const float sn = fmaf(sa[e], cb[e], ca[e] * sb[e]);
        const float x1 = acc[nt][rg * 4 + e], x2 = acc[nt + NTL / 2][rg * 4 + e];
        acc[nt][rg * 4 + e] = fmaf(x1, cs, -(x2 * sn));
        acc[nt + NTL / 2][rg * 4 + e] = fmaf(x1, sn, x2 * cs);
      }
      if (AHEAD && i + AHEAD < GROUPS) fetch(i + AHEAD);
    }
  }
}

// (a body inlined with restrict arguments and dynamic LDS: otherwise the compiler makes LDS reads wait for the loads into
// LDS in flight)
template <int D, bool BWD>
__device__ __forceinline__ void prologue_stream_body(
    const FusedArgs &a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp,
    bf16_t *__restrict__ q, bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm, unsigned char *smem) {
  constexpr int DH = 256, NTL = DH / 32, CPR = DH / 8, ROWB = DH * 2;
  constexpr int QS = DH / SLAB_K, NSLAB = D * QS;              // slabs per tap, slabs
  constexpr int SLAB_INSTR = SLAB_BYTES / 1024 / ST_WAVES;     // load instructions of a wavefront per slab
  static_assert(NSLAB % ST_RING == 0 && ST_RING == 4 && SLAB_INSTR == 4, "a source of the qk-mean is one turn of the ring");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;

  if ((int)blockIdx.x >= a.n_conv_blocks) {
    value_role<BWD, ST_NT>(a, vsrc, v, ((long long)blockIdx.x - a.n_conv_blocks) * (ST_NT * 4));
    return;
  }

  const StreamHead hd(a);
  const bool is_q = hd.is_q;
  const int g = hd.g, ch0 = hd.ch0;
  const float beta = (!is_q && (a.flags & CCA_KEY_TEMP)) ? expf(temp[g]) : 1.f;
  bf16_t *dst = is_q ? q + hd.head * DH : k + g * DH;
  const int dst_stride = is_q ? a.q_stride : a.k_stride;

  // this wavefront's 32 tokens (a wavefront past the end keeps walking the slabs: it loads filter chunks too)
  const int first_wave = __builtin_amdgcn_readfirstlane(wave);  // the wavefront, as the scalar that the loads' addresses are made of
  const long long trow0 = (long long)hd.bid * (ST_WAVES * 32) + first_wave * 32;
  const long long row = trow0 + l32;
  const long long rowc = row < a.rows ? row : a.rows - 1;
  const int tpos = (int)(rowc % a.T);
  const bool any_pad = __any(BWD ? tpos + D - 1 >= a.T : tpos < D - 1) != 0;

  // Rows outside the tensor repeat an end row (they lie outside the token's sequence: zeroed or dropped below).  Rows count from the
  // wavefront's first token, a load's offset from row_from, the first row that it touches (scalars: 64-bit minima are made in vector
  // registers)
  const int row_min = __builtin_amdgcn_readfirstlane((int)max(-trow0, -64ll)), row_max = __builtin_amdgcn_readfirstlane((int)min(a.rows - 1 - trow0, 64ll));
  auto clamp_row = [&](int r) { return min(max(r, row_min), row_max); };
  const int row_from = clamp_row(BWD ? 0 : -(D - 1));
  const bf16_t *const lat_from = lat + (trow0 + row_from) * a.src_stride;
  auto row_off = [&](int r) { return (unsigned)(clamp_row(r) - row_from) * (unsigned)a.src_stride * 2; };
  constexpr unsigned NO_BOUND = 0x7fffffff;  // (the rows are clamped)

  unsigned char *const ring = smem, *const stg = smem + ST_RING * SLAB_BYTES + first_wave * (stream_rows(D) * ROWB);
  // the token rows, 2 per load instruction; chunk c of staged row j lies at c ^ (j mod 16)
  constexpr int FIRST = BWD ? 0 : -(D - 1);
#pragma unroll
  for (int i = 0; i < stream_rows(D) / 2; ++i) {
    const int j = 2 * i + (lane >> 5), p = lane & 31;
    load_to_lds(lat_from, NO_BOUND, row_off(FIRST + j) + (p ^ (j & 15)) * 16, ch0 * 2, stg + i * 1024);
  }
  auto row_frag = [&](int j, int kk) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(stg + j * ROWB + (((2 * kk + half) ^ (j & 15)) * 16)));
  };
  const bool mean = a.flags & CCA_QK_MEAN;
  // Ring slab s_ < NSLAB: the filter's.  Slab NSLAB + 4 x + c: of the qk-mean's source x (another head's rows) the workgroup's 128 tokens
  // x 64 channels from 64 c on, each wavefront its own 32 rows, chunk c of row j at c ^ (j mod 8); beyond the last source, or without
  // the qk-mean, nothing is read for it.
  const int n_src = mean ? (is_q ? 1 : a.R) : 0;
  int src_col = (is_q ? a.e_q + g * DH : g * a.R * DH) * 2, src_bound = mean ? NO_BOUND : 0;
  asm volatile("" : "+s"(src_col), "+s"(src_bound));  // (settled here: chosen at the loads they would be branches between the products)
  unsigned src_off[SLAB_INSTR];
#pragma unroll
  for (int u = 0; u < SLAB_INSTR; ++u) src_off[u] = row_off(8 * u + (lane >> 3)) + ((lane & 7) ^ (lane >> 3)) * 16;
  const u32x4 *const wsrc = wc + (long long)hd.head * NSLAB * (SLAB_BYTES / 16);
  auto fetch_filter = [&](int s_, int u) __attribute__((always_inline)) {
    const int i = first_wave * SLAB_INSTR + u;
    load_to_lds(wsrc, NSLAB * SLAB_BYTES, lane * 16, s_ * SLAB_BYTES + i * 1024, ring + (s_ % ST_RING) * SLAB_BYTES + i * 1024);
  };
  auto fetch_source = [&](int x, int bound, int c, int u) __attribute__((always_inline)) {
    load_to_lds(lat_from, bound, src_off[u], src_col + x * (DH * 2) + c * 128, ring + c * SLAB_BYTES + (first_wave * SLAB_INSTR + u) * 1024);
  };
  auto fetch = [&](int s_, int u) __attribute__((always_inline)) { s_ < NSLAB ? fetch_filter(s_, u) : fetch_source(0, src_bound, s_ - NSLAB, u); };
#pragma unroll
  for (int s_ = 0; s_ < ST_RING; ++s_)
#pragma unroll
    for (int u = 0; u < SLAB_INSTR; ++u) fetch(s_, u);

  f32x16 acc[NTL];
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;

  // this lane's two 16-byte reads of row l32 of a slab (k-steps 0 and 1); output tile nt lies 2 KB further per tile
  uint32_t woff[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) woff[kk] = ((l32 >> 1) * 8 + ((((l32 & 1) << 2) | (2 * kk + half)) ^ ((l32 >> 2) & 3))) * 16;
  // Two sets of fragments, one per k-step of 16 channels; the other set is read between the products of one
  bf16x8 uf[2], wf[2][NTL];
  auto read = [&](int s_, int kk, int i) __attribute__((always_inline)) {
    const int back = D - 1 - s_ / QS;
    if (i == 0) uf[kk] = row_frag(BWD ? l32 + back : l32 + D - 1 - back, 2 * (s_ % QS) + kk);
    else wf[kk][i - 1] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(ring + (s_ % ST_RING) * SLAB_BYTES + woff[kk] + (i - 1) * 2048));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int s_, int kk, int nt) __attribute__((always_inline)) {
    const int back = D - 1 - s_ / QS;
    if (nt == 0 && back > 0 && any_pad && (BWD ? tpos + back >= a.T : tpos < back)) uf[kk] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[kk][nt], uf[kk], acc[nt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // qk-mean weights as identity fragments (see prologue_fused_kernel)
  auto identity_frag = [&](bf16_t wbits, int j) {
    const bool on = ((l32 >> 4) == j) && (((l32 >> 3) & 1) == half);
    u32x4 w = {0, 0, 0, 0};
    const int e = l32 & 7;
    if (on) w[e >> 1] = (uint32_t)wbits << ((e & 1) * 16);
    return __builtin_bit_cast(bf16x8, w);
  };
  const bf16x8 id_half[2] = {identity_frag(f32_to_bf16(0.5f), 0), identity_frag(f32_to_bf16(0.5f), 1)};
  __builtin_amdgcn_s_waitcnt(wait_vm((ST_RING - 1) * SLAB_INSTR) & WAIT_LDS_TOO);  // the token rows and slab 0
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i <= NTL; ++i) read(0, 0, i);
#pragma unroll
  for (int s_ = 0; s_ < NSLAB; ++s_) {
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt) {
      multiply(s_, 0, nt);
      if (nt == 0) read(s_, 1, 0);
      read(s_, 1, nt + 1);
    }
    const bf16x8 own = uf[0];
    // every wavefront holds its last fragments of slab s_, and slab s_ + 1 has landed when only the two behind it are outstanding
    __builtin_amdgcn_s_waitcnt(wait_vm((ST_RING - 2) * SLAB_INSTR) & WAIT_LDS_TOO);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt) {
      multiply(s_, 1, nt);
      if (s_ + 1 < NSLAB) {
        if (nt == 0) read(s_ + 1, 0, 0);
        read(s_ + 1, 0, nt + 1);
      }
      if (nt % 2 == 1) fetch(s_ + ST_RING, nt / 2);
    }
    // own stream of the qk-mean: + 1/2 of the token's own row, whose fragments the last tap holds; channels 32 c .. lie in tile c
    if (s_ >= NSLAB - QS && mean) {
      const int c = s_ - (NSLAB - QS);
      acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_half[0], own, acc[c], 0, 0, 0);
      acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_half[1], uf[1], acc[c], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  if (mean) {
    // ---- other stream of the qk-mean: the sources' slabs, the wavefront's own rows of each
    const float w_other = is_q ? a.mean_q_other : a.mean_k_other;
    const bf16_t w_other_hi = f32_to_bf16(w_other);
    const bf16_t w_other_lo = f32_to_bf16(w_other - bf16_to_f32(w_other_hi));
    const bool grp_lo = (w_other_lo & 0x7fffu) != 0;  // uniform over the workgroup
    const bf16x8 id_hi[2] = {identity_frag(w_other_hi, 0), identity_frag(w_other_hi, 1)};
    const bf16x8 id_lo[2] = {identity_frag(w_other_lo, 0), identity_frag(w_other_lo, 1)};
    for (int x = 0; x < n_src; ++x) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        __builtin_amdgcn_s_waitcnt(wait_vm((ST_RING - 1) * SLAB_INSTR));
        asm volatile("" ::: "memory");
        bf16x8 m[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          m[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(ring + c * SLAB_BYTES + first_wave * (SLAB_BYTES / ST_WAVES) + l32 * 128 + (((2 * kk + half) ^ (l32 & 7)) * 16)));
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < SLAB_INSTR; ++u) fetch_source(x + 1, x + 1 < n_src ? NO_BOUND : 0, c, u);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          acc[2 * c + kk / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_hi[kk & 1], m[kk], acc[2 * c + kk / 2], 0, 0, 0);
          if (grp_lo) acc[2 * c + kk / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_lo[kk & 1], m[kk], acc[2 * c + kk / 2], 0, 0, 0);
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(0));  // no load into LDS outlives the workgroup

  norm_and_rope_256<4>(acc, a, hd.head, beta, row, tpos, half, ropeA, ropeB, rnorm);
  // ---- round once to bf16; through this wavefront's staging rows (16-byte chunk c of row r at c ^ r), out as whole rows
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows' last readers are done
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      u32x2 w;
      w.x = pack2(acc[nt][rg * 4 + 0], acc[nt][rg * 4 + 1]);
      w.y = pack2(acc[nt][rg * 4 + 2], acc[nt][rg * 4 + 3]);
      *reinterpret_cast<u32x2 *>(stg + l32 * ROWB + ((nt * 4 + rg) ^ l32) * 16 + half * 8) = w;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS handles a wavefront's accesses in order
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  bf16_t *const to = dst + trow0 * dst_stride;
  const int rows_left = (int)min(a.rows - trow0, 32ll);
#pragma unroll
  for (int it = 0; it < 16; it += 8) {
    u32x4 out[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) out[u] = *reinterpret_cast<const u32x4 *>(stg + ((it + u) * 2 + (lane >> 5)) * ROWB + (lane & 31) * 16);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int rr = (it + u) * 2 + (lane >> 5), c = (lane & 31) ^ rr;
      if (rr < rows_left) *reinterpret_cast<u32x4 *>(to + rr * dst_stride + c * 8) = out[u];
    }
  }
}

template <int D, bool BWD>
__global__ __launch_bounds__(ST_NT) __attribute__((amdgpu_waves_per_eu(1, 1))) void prologue_stream_kernel(
    FusedArgs a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp,
    bf16_t *__restrict__ q, bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm) {
  extern __shared__ __attribute__((aligned(16))) unsigned char stream_smem[];
  prologue_stream_body<D, BWD>(a, lat, vsrc, wc, ropeA, ropeB, temp, q, k, v, rnorm, stream_smem);
}

// ---------------------------------------------------------------------------
// The form for grids of several rounds: 256 tokens per workgroup, 8 wavefronts x 32 tokens, two per SIMD.  Each filter byte
// that comes into LDS serves twice as many tokens, and a wavefront's waits hide under its SIMD's other one; there is no room
// for staged token rows, so their fragments come straight from the latent rows, and the filter goes through registers into two
// buffers of two slabs (64 input channels).  Bound by the filter reads from LDS and the waits between barriers: 16384 tokens, 8 / 2
// heads 129 us against 132 for the kernel above (6000 tokens, 4 / 1 heads: 48 against 27.5; the rule is stream_takes_256).
// ---------------------------------------------------------------------------
template <int D, bool BWD>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void prologue_stream_long_kernel(
    FusedArgs a, const bf16_t *__restrict__ lat, const bf16_t *__restrict__ vsrc, const u32x4 *__restrict__ wc,
    const float2 *__restrict__ ropeA, const float2 *__restrict__ ropeB, const float *__restrict__ temp,
    bf16_t *__restrict__ q, bf16_t *__restrict__ k, bf16_t *__restrict__ v, float *__restrict__ rnorm) {
  constexpr int DH = 256, NTL = DH / 32;
  constexpr int KC = 2 * SLAB_K, KCK = KC / 16;  // input channels per step, MFMA k-steps per step
  constexpr int NCH = DH / KC, NSTEP = D * NCH, STEP = 2 * SLAB_BYTES;
  constexpr int W_PER_THREAD = STEP / 16 / NT;  // 16-byte chunks of a step per thread
  constexpr int SROW = KC * 2 + 16, BUF = DH * SROW;  // padded row in LDS: conflict-free 16-byte reads down a column of rows
  static_assert(W_PER_THREAD == 4 && NT * 4 == 2 * DH * 4, "two chunks of each slab per thread, 128 rows apart");
  __shared__ __attribute__((aligned(16))) unsigned char sW[2 * BUF];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  if ((int)blockIdx.x >= a.n_conv_blocks) {
    value_role<BWD, NT>(a, vsrc, v, ((long long)blockIdx.x - a.n_conv_blocks) * (NT * 4));
    return;
  }
  const StreamHead hd(a);
  const bool is_q = hd.is_q;
  const float beta = (!is_q && (a.flags & CCA_KEY_TEMP)) ? expf(temp[hd.g]) : 1.f;

  // qk-mean weights as identity fragments (see prologue_fused_kernel); the other stream's are made after the
  // convolution, when fewer registers are live
  const bool mean = a.flags & CCA_QK_MEAN;
  auto identity_frag = [&](bf16_t wbits, int j) {
    const bool on = ((l32 >> 4) == j) && (((l32 >> 3) & 1) == half);
    u32x4 w = {0, 0, 0, 0};
    const int e = l32 & 7;
    if (on) w[e >> 1] = (uint32_t)wbits << ((e & 1) * 16);
    return __builtin_bit_cast(bf16x8, w);
  };
  bf16x8 id_half[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) id_half[j] = identity_frag(f32_to_bf16(0.5f), j);

  // this wavefront's 32 tokens (a wavefront past the end keeps walking the slabs: it stages filter chunks too)
  const long long row = (long long)hd.bid * 256 + wave * 32 + l32;
  const long long rowc = row < a.rows ? row : a.rows - 1;
  const int tpos = (int)(rowc % a.T);

  // step s = (tap s / NCH, channels (s % NCH) * 64 ...): two slabs, one after the other in memory and in LDS
  const u32x4 *const wsrc = wc + (long long)hd.head * NSTEP * (STEP / 16) + tid;
  // chunk tid of a slab (slab_elem): row 2 * (tid / 8) + u / 4, chunk u mod 4 of it, with u = tid mod 8 ^ (tid / 16) mod 4
  const int w_u = (tid & 7) ^ ((tid >> 4) & 3), w_to = (2 * (tid >> 3) + (w_u >> 2)) * SROW + (w_u & 3) * 16;
  u32x4 wreg[W_PER_THREAD];
  auto load_step = [&](int s_) {
#pragma unroll
    for (int i = 0; i < W_PER_THREAD; ++i) wreg[i] = wsrc[(long long)s_ * (STEP / 16) + i * NT];
  };
  auto store_step = [&](int buf) {
#pragma unroll
    for (int i = 0; i < W_PER_THREAD; ++i)
      *reinterpret_cast<u32x4 *>(sW + buf * BUF + w_to + (i & 1) * (DH / 2) * SROW + (i >> 1) * SLAB_K * 2) = wreg[i];
  };

  f32x16 acc[NTL];
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;

  load_step(0);
  store_step(0);
#pragma unroll  // tap and channel group must be compile-time: they pick accumulator tiles
  for (int s_ = 0; s_ < NSTEP; ++s_) {
    const int d = s_ / NCH, c = s_ % NCH, back = D - 1 - d;
    if (s_ + 1 < NSTEP) load_step(s_ + 1);
    // token operands: row t - (D-1-d) (adjoint: t + (D-1-d)), channels c*64 .. c*64+63; rows outside the sequence are zero
    bf16x8 uf[KCK];
    {
      long long src_row = BWD ? rowc + back : rowc - back;
      src_row = src_row < 0 ? 0 : (src_row > a.rows - 1 ? a.rows - 1 : src_row);
      const bf16_t *p = lat + src_row * a.src_stride + hd.ch0 + c * KC + half * 8;
#pragma unroll
      for (int kk = 0; kk < KCK; ++kk) {
        u32x4 raw = *reinterpret_cast<const u32x4 *>(p + kk * 16);
        if (BWD ? tpos + back >= a.T : tpos < back) raw = u32x4{0, 0, 0, 0};
        uf[kk] = __builtin_bit_cast(bf16x8, raw);
      }
    }
    __syncthreads();  // step s_ is in LDS (stored one step ago); the other buffer is no longer read
    if (s_ + 1 < NSTEP) store_step((s_ + 1) & 1);
    const unsigned char *const sw = sW + (s_ & 1) * BUF + l32 * SROW + half * 16;
#pragma unroll
    for (int kk = 0; kk < KCK; ++kk)
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt) {
        const bf16x8 wf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(sw + nt * 32 * SROW + kk * 32));
        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, uf[kk], acc[nt], 0, 0, 0);
      }
    if (mean && back == 0) {  // own stream of the qk-mean: + 1/2 of the token's own row; channels c*64 + kk*16 .. lie in tile 2c + kk/2
#pragma unroll
      for (int kk = 0; kk < KCK; ++kk)
        acc[2 * c + kk / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_half[kk & 1], uf[kk], acc[2 * c + kk / 2], 0, 0, 0);
    }
  }

  // ---- other stream of the qk-mean, a quarter of the head width at a time
  if (mean) {
    const float w_other = is_q ? a.mean_q_other : a.mean_k_other;
    const bf16_t w_other_hi = f32_to_bf16(w_other);
    const bf16_t w_other_lo = f32_to_bf16(w_other - bf16_to_f32(w_other_hi));
    const bool grp_lo = (w_other_lo & 0x7fffu) != 0;  // uniform over the workgroup
    bf16x8 id_grp[2], id_grp_lo[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      id_grp[j] = identity_frag(w_other_hi, j);
      id_grp_lo[j] = identity_frag(w_other_lo, j);
    }
    const int nsrc = is_q ? 1 : a.R;
    for (int x = 0; x < nsrc; ++x) {
      const bf16_t *p = lat + rowc * a.src_stride + (is_q ? a.e_q + hd.g * DH : (hd.g * a.R + x) * DH) + half * 8;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        bf16x8 mf[KCK];
#pragma unroll
        for (int kk = 0; kk < KCK; ++kk)
          mf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p + c * KC + kk * 16));
#pragma unroll
        for (int kk = 0; kk < KCK; ++kk) {
          acc[2 * c + kk / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_grp[kk & 1], mf[kk], acc[2 * c + kk / 2], 0, 0, 0);
          if (grp_lo)
            acc[2 * c + kk / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id_grp_lo[kk & 1], mf[kk], acc[2 * c + kk / 2], 0, 0, 0);
        }
      }
    }
  }

  norm_and_rope_256<0>(acc, a, hd.head, beta, row, tpos, half, ropeA, ropeB, rnorm);
  if (row < a.rows) {
    bf16_t *const orow = is_q ? q + hd.head * DH + row * a.q_stride : k + hd.g * DH + row * a.k_stride;
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        u32x2 w;
        w.x = pack2(acc[nt][rg * 4 + 0], acc[nt][rg * 4 + 1]);
        w.y = pack2(acc[nt][rg * 4 + 2], acc[nt][rg * 4 + 3]);
        *reinterpret_cast<u32x2 *>(orow + nt * 32 + rg * 8 + half * 4) = w;
      }
  }
}

// ---------------------------------------------------------------------------
// No transform selected (plain MHA / GQA, Sec. 2.1): q, k, v are column slices
// of the latent rows; only the optional value-shift moves data in time.
// 16 bytes per thread, storage-type agnostic (`es` = bytes per element).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void split_copy_kernel(const unsigned char *__restrict__ lat,
                                                        unsigned char *__restrict__ q, unsigned char *__restrict__ k,
                                                        unsigned char *__restrict__ v, long long rows, int T, int e_q,
                                                        int e_kv, int v_half, int es, int v_shift) {
  const int n_lat = e_q + 2 * e_kv;
  const int cpr = n_lat * es / 16;  // chunks per latent row
  const long long total = rows * cpr;
  for (long long id = (long long)blockIdx.x * 256 + threadIdx.x; id < total; id += (long long)gridDim.x * 256) {
    const long long row = id / cpr;
    const int col = (int)(id % cpr) * (16 / es);  // first element of the chunk
    const int t = (int)(row % T);
    u32x4 val = {0, 0, 0, 0};
    const bool shifted = v_shift && col >= e_q + e_kv + v_half;
    if (!shifted || t > 0)
      val = *reinterpret_cast<const u32x4 *>(lat + ((row - (shifted ? 1 : 0)) * n_lat + col) * es);
    unsigned char *dstp;
    if (col < e_q) dstp = q + (row * e_q + col) * es;
    else if (col < e_q + e_kv) dstp = k + (row * e_kv + (col - e_q)) * es;
    else dstp = v + (row * e_kv + (col - e_q - e_kv)) * es;
    *reinterpret_cast<u32x4 *>(dstp) = val;
  }
}

// Adjoint of split_copy_kernel: d_lat is d_q | d_k | d_v side by side, the shifted half of d_v read one token later
// (zero for the last token of a sequence).
__global__ __launch_bounds__(256) void split_copy_bwd_kernel(const unsigned char *__restrict__ dq,
                                                            const unsigned char *__restrict__ dk,
                                                            const unsigned char *__restrict__ dv,
                                                            unsigned char *__restrict__ d_lat, long long rows, int T,
                                                            int e_q, int e_kv, int v_half, int es, int v_shift) {
  const int n_lat = e_q + 2 * e_kv;
  const int cpr = n_lat * es / 16;
  const long long total = rows * cpr;
  for (long long id = (long long)blockIdx.x * 256 + threadIdx.x; id < total; id += (long long)gridDim.x * 256) {
    const long long row = id / cpr;
    const int col = (int)(id % cpr) * (16 / es);
    const int t = (int)(row % T);
    u32x4 val = {0, 0, 0, 0};
    if (col < e_q) {
      val = *reinterpret_cast<const u32x4 *>(dq + (row * e_q + col) * es);
    } else if (col < e_q + e_kv) {
      val = *reinterpret_cast<const u32x4 *>(dk + (row * e_kv + (col - e_q)) * es);
    } else {
      const int cc = col - e_q - e_kv;
      const bool shifted = v_shift && cc >= v_half;
      if (!shifted || t + 1 < T) val = *reinterpret_cast<const u32x4 *>(dv + ((row + (shifted ? 1 : 0)) * e_kv + cc) * es);
    }
    *reinterpret_cast<u32x4 *>(d_lat + (row * n_lat + col) * es) = val;
  }
}

template <int DH, int D, bool BWD>
hipError_t launch_main(const FusedArgs &a, const void *lat, const void *vsrc, const void *wc, const float2 *ropeA,
                       const float2 *ropeB, const float *temp, void *q, void *k, void *v, float *rnorm, int grid,
                       hipStream_t s) {
  // the head's filter, then 32 staging rows of d_h channels per wavefront (160 KB at d_h = 128 with 3 taps)
  constexpr size_t smem = (size_t)DH * D * (DH / 8) * 16 + (size_t)(NT / 64) * 32 * DH * 2;
  static_assert(smem <= 160 * 1024, "filter and staging rows must fit the LDS");
  if (hipError_t e = raise_lds_limit<prologue_fused_kernel<DH, D, BWD>>(smem); e != hipSuccess) return e;
  prologue_fused_kernel<DH, D, BWD><<<grid, NT, smem, s>>>(a, (const bf16_t *)lat, (const bf16_t *)vsrc, (const u32x4 *)wc,
                                                       ropeA, ropeB, temp, (bf16_t *)q, (bf16_t *)k, (bf16_t *)v, rnorm);
  return hipGetLastError();
}

template <int DH, int D>
hipError_t launch_adjoint_pair(const FusedArgs &a, const void *d3, const void *vsrc, const void *wc, void *dq, void *dk, void *dv,
                               const DwcArgs &w, int grid, hipStream_t s) {
  constexpr size_t adjoint = (size_t)DH * D * (DH / 8) * 16 + (size_t)(NT / 64) * 32 * DH * 2, per = NT / dwc_threads(DH);
  constexpr size_t smem = adjoint > per * dwc_lds(DH, D) ? adjoint : per * dwc_lds(DH, D);
  static_assert(smem <= 160 * 1024, "LDS");
  if (hipError_t e = raise_lds_limit<prologue_adjoint_pair_kernel<DH, D>>(smem); e != hipSuccess) return e;
  prologue_adjoint_pair_kernel<DH, D><<<grid + (w.units + (int)per - 1) / (int)per, NT, smem, s>>>(
      a, (const bf16_t *)d3, (const bf16_t *)vsrc, (const u32x4 *)wc, (bf16_t *)dq, (bf16_t *)dk, (bf16_t *)dv, w, grid);
  return hipGetLastError();
}

// Tokens per workgroup: each workgroup first loads its head's filter (about one tile's worth of time), and one
// workgroup fits per CU, so minimise rounds-on-256-CUs x (1 + tiles per wavefront).  Returns the grid size.
int plan_grid(const Dims &d, FusedArgs &a) {
  // One workgroup = one head x 256 * tiles tokens.  Cost of a workgroup in units of a query-head tile: about one
  // for loading its filter, one per query-head tile, 1 + 0.11 R per key-head tile when the qk-mean is on (measured
  // 1.43 at R = 4).  The slowest workgroup of a round sets the round's length, so key heads take fewer tiles.
  const double ck = (a.flags & CCA_QK_MEAN) ? 1.0 + 0.11 * d.R : 1.0;
  double best_cost = -1.0;
  long long best_q = 0, best_k = 0;
  for (int tq = 1; tq <= MAX_TILES_PER_WAVE; ++tq)
    for (int tk = 1; tk <= MAX_TILES_PER_WAVE; ++tk) {
      const long long nq = d.Hq * ((d.rows() + 256 * tq - 1) / (256 * tq));
      const long long nk = d.Hk * ((d.rows() + 256 * tk - 1) / (256 * tk));
      const double slowest = 1.0 + (tq > ck * tk ? (double)tq : ck * tk);
      const double cost = (double)((nq + nk + 255) / 256) * slowest;
      if (best_cost < 0 || cost < best_cost - 1e-9) {
        best_cost = cost;
        a.tiles_per_wave = tq;
        a.tiles_per_wave_k = tk;
        best_q = nq;
        best_k = nk;
      }
    }
  a.n_k_blocks = (int)best_k;
  a.n_conv_blocks = (int)(best_q + best_k);
  const long long v_chunks = d.rows() * (d.e_kv / 8);
  const int v_blocks = (int)((v_chunks + NT * 4 - 1) / (NT * 4));
  return a.n_conv_blocks + v_blocks;
}

// The short form: 64 tokens of one head per workgroup.  Returns the grid size.
int plan_short(const Dims &d, FusedArgs &a) {
  const long long blocks = (d.rows() + SH_TOK - 1) / SH_TOK, per_v = d.dh * 16;
  a.n_k_blocks = (int)(d.Hk * blocks);
  a.n_conv_blocks = (int)((d.Hq + d.Hk) * blocks);
  return a.n_conv_blocks + (int)((d.rows() * (d.e_kv / 8) + per_v - 1) / per_v);
}

template <int DH, int D, bool BWD>
hipError_t launch_short(const FusedArgs &a, const void *lat, const void *vsrc, const void *wc, const float2 *ropeA,
                        const float2 *ropeB, const float *temp, void *q, void *k, void *v, float *rnorm, int grid, hipStream_t s) {
  static_assert(short_lds(DH, D) <= 160 * 1024, "LDS");
  if (hipError_t e = raise_lds_limit<prologue_short_kernel<DH, D, BWD>>(short_lds(DH, D)); e != hipSuccess) return e;
  prologue_short_kernel<DH, D, BWD><<<grid, DH * 4, short_lds(DH, D), s>>>(a, (const bf16_t *)lat, (const bf16_t *)vsrc, (const u32x4 *)wc, ropeA,
                                                                           ropeB, temp, (bf16_t *)q, (bf16_t *)k, (bf16_t *)v, rnorm);
  return hipGetLastError();
}

template <int DH, int D>
hipError_t launch_short_pair(const FusedArgs &a, const void *d3, const void *vsrc, const void *wc, void *dq, void *dk, void *dv,
                             const DwcArgs &w, int grid, hipStream_t s) {
  constexpr size_t smem = short_lds(DH, D) > dwc_lds(DH, D) ? short_lds(DH, D) : dwc_lds(DH, D);
  if (hipError_t e = raise_lds_limit<prologue_short_pair_kernel<DH, D>>(smem); e != hipSuccess) return e;
  prologue_short_pair_kernel<DH, D><<<grid + w.units, DH * 4, smem, s>>>(a, (const bf16_t *)d3, (const bf16_t *)vsrc, (const u32x4 *)wc,
                                                                         (bf16_t *)dq, (bf16_t *)dk, (bf16_t *)dv, w, grid);
  return hipGetLastError();
}

struct FusedScratch {
  bf16_t *wc;
  float2 *ropeA, *ropeB;
  size_t bytes;
};
FusedScratch carve(const Dims &d, void *scratch, int D) {
  const int NH = d.Hq + d.Hk, n_thi = (d.T + 127) / 128, DH = d.dh;
  const size_t wc_bytes = ((size_t)NH * DH * D * DH * 2 + 255) / 256 * 256;
  const size_t ra_bytes = ((size_t)n_thi * (DH / 2) * 8 + 255) / 256 * 256;
  const size_t rb_bytes = (size_t)(DH / 2) * 128 * 8;
  char *base = static_cast<char *>(scratch);
  return FusedScratch{reinterpret_cast<bf16_t *>(base), reinterpret_cast<float2 *>(base + wc_bytes),
                      reinterpret_cast<float2 *>(base + wc_bytes + ra_bytes), wc_bytes + ra_bytes + rb_bytes};
}

PrologueSetup make_setup(const Dims &d, const cca_weights &w, const FusedScratch &fs, int D, bool transposed) {
  const int NH = d.Hq + d.Hk, n_thi = (d.T + 127) / 128, DH = d.dh;
  const int n_fold = (NH * DH * DH + 255) / 256, n_rope = (n_thi * (DH / 2) + (DH / 2) * 128 + 255) / 256;
  return PrologueSetup{(d.flags & CCA_CONV_SEQ) ? (const bf16_t *)w.w_conv_seq : nullptr, (const bf16_t *)w.w_conv_ch, fs.wc, fs.ropeA,
                       fs.ropeB, d.rope_base, NH, DH, D, (d.flags & CCA_CONV_SEQ) ? d.k_seq : 1, d.k_ch, n_thi, transposed ? 1 : 0,
                       n_fold, n_fold + n_rope};
}

hipError_t run_setup(const PrologueSetup &setup, hipStream_t s, const TransposePair *weights = nullptr) {
  const TransposePair pair = weights ? *weights : TransposePair{};
  prologue_setup_kernel<<<setup.n_blocks + pair.n1 + pair.n2, 256, 0, s>>>(setup, pair);
  return hipGetLastError();
}

int taps(const Dims &d) { return ((d.flags & CCA_CONV_SEQ) ? d.k_seq : 1) + d.k_ch - 1; }

}  // namespace

bool prologue_is_split_copy(const Dims &d) {
  const uint32_t transforms = CCA_CONV_SEQ | CCA_CONV_CH | CCA_QK_MEAN | CCA_QK_NORM | CCA_KEY_TEMP | CCA_ROPE;
  const int per16 = d.bf16 ? 8 : 4;
  return !(d.flags & transforms) && d.e_q % per16 == 0 && d.e_kv % per16 == 0 && d.v_half % per16 == 0;
}

__global__ void fill_f32_kernel(float *p, long long n, float val) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = val;
}

hipError_t prologue_split_norms(const Dims &d, float *rnorm, hipStream_t s) {
  if (!rnorm) return hipSuccess;
  fill_f32_kernel<<<256, 256, 0, s>>>(rnorm, d.rows() * (d.Hq + d.Hk), 1.f);
  return hipGetLastError();
}

hipError_t prologue_split_copy(const Dims &d, const void *lat, void *q, void *k, void *v, float *rnorm, hipStream_t s) {
  if (hipError_t e = prologue_split_norms(d, rnorm, s); e != hipSuccess) return e;
  const long long total = d.rows() * ((long long)d.n_lat * d.esize() / 16);
  const int grid = (int)((total + 255) / 256 < 256 * 64 ? (total + 255) / 256 : 256 * 64);
  split_copy_kernel<<<grid, 256, 0, s>>>((const unsigned char *)lat, (unsigned char *)q, (unsigned char *)k,
                                         (unsigned char *)v, d.rows(), d.T, d.e_q, d.e_kv, d.v_half, (int)d.esize(),
                                         (d.flags & CCA_V_SHIFT) ? 1 : 0);
  return hipGetLastError();
}

hipError_t prologue_split_copy_bwd(const Dims &d, const void *d_q, const void *d_k, const void *d_v, void *d_lat,
                                   hipStream_t s) {
  const long long total = d.rows() * ((long long)d.n_lat * d.esize() / 16);
  const int grid = (int)((total + 255) / 256 < 256 * 64 ? (total + 255) / 256 : 256 * 64);
  split_copy_bwd_kernel<<<grid, 256, 0, s>>>((const unsigned char *)d_q, (const unsigned char *)d_k,
                                             (const unsigned char *)d_v, (unsigned char *)d_lat, d.rows(), d.T, d.e_q,
                                             d.e_kv, d.v_half, (int)d.esize(), (d.flags & CCA_V_SHIFT) ? 1 : 0);
  return hipGetLastError();
}

bool prologue_fused_supported(const Dims &d) {
  return d.bf16 && (d.dh == 256 || d.dh == 128 || d.dh == 64) && (d.flags & CCA_CONV_CH) && !(d.flags & CCA_ROPE_INTERLEAVED) && taps(d) <= 3 &&
         d.v_half % 8 == 0;
}

size_t prologue_fused_scratch_bytes(const Dims &d) {
  if (!prologue_fused_supported(d)) return 0;
  return carve(d, nullptr, taps(d)).bytes;
}

static FusedArgs forward_args(const Dims &d) {
  return FusedArgs{d.T, d.Hq, d.Hk, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, d.rows(), d.flags, 0, 1,
                   d.rope_base, d.norm_eps, d.n_lat, d.e_q, d.e_kv, d.n_lat, d.e_kv, 0.5f, 0.5f / (float)d.R};
}

hipError_t prologue_fused_prepare(const Dims &d, const cca_weights &w, void *scratch, hipStream_t s, const TransposePair *weights) {
  const int D = taps(d);
  return run_setup(make_setup(d, w, carve(d, scratch, D), D, false), s, weights);
}

template <int D, bool BWD>
static hipError_t launch_stream(const Dims &d, FusedArgs a, const float *temp, const void *lat, const void *vsrc,
                                const FusedScratch &fs, void *q, void *k, void *v, float *rnorm, hipStream_t s) {
  // one block of 128 or 256 tokens per workgroup for every head, key heads first (the kernels' block map)
  const bool wide = stream_takes_256(d.rows(), d.Hq + d.Hk, d.R, D, BWD);
  const int tokens = wide ? 256 : ST_WAVES * 32, threads = wide ? NT : ST_NT;
  const long long blocks = (d.rows() + tokens - 1) / tokens;
  a.tiles_per_wave = a.tiles_per_wave_k = 1;
  a.n_k_blocks = (int)(d.Hk * blocks);
  a.n_conv_blocks = (int)((d.Hq + d.Hk) * blocks);
  const long long v_chunks = d.rows() * (d.e_kv / 8);
  const int grid = a.n_conv_blocks + (int)((v_chunks + threads * 4 - 1) / (threads * 4));
  const auto launch = [&](auto kernel, size_t lds) {
    kernel<<<grid, threads, lds, s>>>(a, (const bf16_t *)lat, (const bf16_t *)vsrc, (const u32x4 *)fs.wc, fs.ropeA, fs.ropeB, temp,
                                      (bf16_t *)q, (bf16_t *)k, (bf16_t *)v, rnorm);
  };
  if (wide) {
    launch(prologue_stream_long_kernel<D, BWD>, 0);
  } else {
    if (hipError_t e = raise_lds_limit<prologue_stream_kernel<D, BWD>>(stream_lds(D)); e != hipSuccess) return e;
    launch(prologue_stream_kernel<D, BWD>, stream_lds(D));
  }
  return hipGetLastError();
}

hipError_t prologue_fused_run(const Dims &d, const cca_weights &w, const void *lat, void *q, void *k, void *v,
                              float *rnorm, const void *scratch, hipStream_t s) {
  const int D = taps(d);
  FusedArgs a = forward_args(d);
  const FusedScratch fs = carve(d, const_cast<void *>(scratch), D);
  const bf16_t *vsrc = (const bf16_t *)lat + d.e_q + d.e_kv;
  if (d.dh == 256) {
    switch (D) {
      case 1: return launch_stream<1, false>(d, a, w.temp, lat, vsrc, fs, q, k, v, rnorm, s);
      case 2: return launch_stream<2, false>(d, a, w.temp, lat, vsrc, fs, q, k, v, rnorm, s);
      default: return launch_stream<3, false>(d, a, w.temp, lat, vsrc, fs, q, k, v, rnorm, s);
    }
  }
  const bool brief = prologue_is_short(d.rows(), d.Hq + d.Hk, d.R, d.dh, false);
  const int grid = brief ? plan_short(d, a) : plan_grid(d, a);
#define LAUNCH_DH(D_, B_) (brief ? d.dh == 64 ? launch_short<64, D_, B_> : launch_short<128, D_, B_> : d.dh == 64 ? launch_main<64, D_, B_> : launch_main<128, D_, B_>)
  switch (D) {
    case 1: return LAUNCH_DH(1, false)(a, lat, vsrc, fs.wc, fs.ropeA, fs.ropeB, w.temp, q, k, v, rnorm, grid, s);
    case 2: return LAUNCH_DH(2, false)(a, lat, vsrc, fs.wc, fs.ropeA, fs.ropeB, w.temp, q, k, v, rnorm, grid, s);
    default: return LAUNCH_DH(3, false)(a, lat, vsrc, fs.wc, fs.ropeA, fs.ropeB, w.temp, q, k, v, rnorm, grid, s);
  }
}

hipError_t prologue_fused_bf16(const Dims &d, const cca_weights &w, const void *lat, void *q, void *k, void *v,
                               float *rnorm, void *scratch, hipStream_t s) {
  hipError_t e = prologue_fused_prepare(d, w, scratch, s);
  if (e != hipSuccess) return e;
  return prologue_fused_run(d, w, lat, q, k, v, rnorm, scratch, s);
}

// ---- adjoint: d3 (B*T, e_q+e_kv), d_v -> d_lat.  `scratch` as for the forward; the RoPE tables its set-up leaves there are the ones
// the pointwise backward kernel reads.
PrologueSetup prologue_fused_bwd_setup(const Dims &d, const cca_weights &w, void *scratch) {
  const int D = taps(d);
  return make_setup(d, w, carve(d, scratch, D), D, true);
}
hipError_t prologue_set_up(const PrologueSetup &setup, hipStream_t s) { return run_setup(setup, s); }

// dwc (may be NULL; d_h <= 128): the filter gradients' partial sums, formed in the same launch
hipError_t prologue_fused_bwd_dlat(const Dims &d, const void *d3, const void *d_v, void *d_lat, void *scratch, const DwcArgs *dwc,
                                   hipStream_t s) {
  const int D = taps(d);
  const int ld = d.e_q + d.e_kv;
  // only the qk-mean and value-shift flags matter to the adjoint kernel
  FusedArgs a{d.T, d.Hq, d.Hk, d.R, d.e_q, d.e_kv, d.n_lat, d.v_half, d.k_seq, d.k_ch, d.rows(),
              d.flags & (CCA_QK_MEAN | CCA_V_SHIFT), 0, 1, d.rope_base, 0.f, ld, d.n_lat, d.n_lat, d.e_kv, d.n_lat,
              0.5f / (float)d.R, 0.5f};
  const FusedScratch fs = carve(d, scratch, D);
  bf16_t *dl = (bf16_t *)d_lat;
  if (d.dh == 256) {
    switch (D) {
      case 1: return launch_stream<1, true>(d, a, nullptr, d3, d_v, fs, dl, dl + d.e_q, dl + ld, nullptr, s);
      case 2: return launch_stream<2, true>(d, a, nullptr, d3, d_v, fs, dl, dl + d.e_q, dl + ld, nullptr, s);
      default: return launch_stream<3, true>(d, a, nullptr, d3, d_v, fs, dl, dl + d.e_q, dl + ld, nullptr, s);
    }
  }
  const bool brief = prologue_is_short(d.rows(), d.Hq + d.Hk, d.R, d.dh, true);
  const int grid = brief ? plan_short(d, a) : plan_grid(d, a);
  if (dwc) {
#define PAIR(D_) (brief ? d.dh == 64 ? launch_short_pair<64, D_> : launch_short_pair<128, D_> : d.dh == 64 ? launch_adjoint_pair<64, D_> : launch_adjoint_pair<128, D_>) \
      (a, d3, d_v, fs.wc, dl, dl + d.e_q, dl + ld, *dwc, grid, s)
    return D == 1 ? PAIR(1) : D == 2 ? PAIR(2) : PAIR(3);
#undef PAIR
  }
  switch (D) {
    case 1: return LAUNCH_DH(1, true)(a, d3, d_v, fs.wc, fs.ropeA, fs.ropeB, nullptr, dl, dl + d.e_q, dl + ld, nullptr, grid, s);
    case 2: return LAUNCH_DH(2, true)(a, d3, d_v, fs.wc, fs.ropeA, fs.ropeB, nullptr, dl, dl + d.e_q, dl + ld, nullptr, grid, s);
    default: return LAUNCH_DH(3, true)(a, d3, d_v, fs.wc, fs.ropeA, fs.ropeB, nullptr, dl, dl + d.e_q, dl + ld, nullptr, grid, s);
  }
}

}  // namespace cca
