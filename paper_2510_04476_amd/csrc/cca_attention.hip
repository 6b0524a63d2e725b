// Latent-space softmax attention on the gfx950 matrix cores (Sec. 2.2, third
// line of the final equation block; KV heads shared by groups of query heads
// as in the CCGQA paragraph).  bf16 in, fp32 accumulation, online softmax.
//
// One workgroup = 8 wavefronts = 256 query rows of one (batch, query head), one
// workgroup per CU (2 wavefronts per SIMD); each wavefront owns 32 rows (one
// MFMA tile) and all of d_h, so the softmax statistics of a row never leave a
// wavefront.  Keys / values arrive in tiles of 64 through double-buffered LDS:
// a tile travels HBM -> registers during one tile step and registers -> LDS
// during the next.  Where that grid would leave CUs idle (fwd_splits_keys)
// a workgroup owns 128 rows instead and its two groups of four wavefronts
// take the even and the odd key tiles; the two partial results of a row are
// merged through LDS.
//
// The scores are produced transposed, S^T = K Q^T, with the 32x32x16 bf16
// MFMA.  Its accumulator layout then gives every lane 16 keys of ONE query
// row, so (a) the row max / sum are in-lane reductions plus a single exchange
// between the two half-waves, and (b) the exponentiated scores, packed to
// bf16 in place, are already the second operand of O^T += V^T P^T: P never
// goes through LDS.  V sits in LDS row-major like K; the PV operand (8 keys of
// one channel per lane) is fetched with the gfx950 transposing LDS read
// (ds_read_b64_tr_b16), in the key order that accumulator layout dictates.
//
// Vector-ALU work per score is pared down to exp2 + convert + one add:
//   - Q is multiplied by scale*log2(e) once, so scores are in log2 units;
//   - the MFMA accumulator starts from -m (the row's reference max, kept as a
//     16-register vector) instead of 0, so the scores come out max-subtracted;
//   - the reference max is raised only when a score exceeds it by more than
//     2^8 (always on the first tile), so rescaling the accumulator is rare;
//     with the QK L2-norm of the method the scores are bounded by d_h * beta *
//     scale, that bound is the reference max and the row max is never formed;
//   - the row sum uses plain v_add_f32 (two chains).  For inference it adds
//     the fp32 probabilities while the PV product multiplies their bf16
//     roundings, so a row's output carries a common factor 1 + delta, |delta|
//     <= 2^-8 (it averages out over the keys; a row dominated by one key sees
//     all of it).  When the caller saves lse / o_lo for a backward pass the
//     sum adds the rounded values instead (two more vector instructions per
//     pair of scores, measured 4 % of the kernel): the backward pass forms
//     dS = P (dP - <dO, o>), which cancels to rounding level on a sharp row
//     only if o is exactly the convex combination the PV product formed.  The bf16 dot instructions (v_dot2*_f32_bf16) are avoided: one
//     of them per MFMA was measured to cut the MFMA issue rate by a quarter,
//     while exp2, convert, add and fma issue in an MFMA's shadow for free.
//
// Two code paths share the kernel: the generic one (running reference max,
// one tile at a time) and, for bounded scores, a software-pipelined one
// (attn_fwd_pipelined below).
#include <type_traits>

#include "cca_internal.h"

namespace cca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

namespace {

constexpr int BQ = 256;   // query rows per workgroup (8 wavefronts x 32 rows)
constexpr int BKV = 64;   // keys per LDS tile
constexpr int NT = 512;   // threads
constexpr int PF = 3;     // operand fetches run this many MFMAs ahead
constexpr float RESCALE_LOG2 = 8.f;
constexpr float LOST_LOG2 = 4096.f;  // a reference max this far below the scores rounds them by up to 2^-12

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  bf16x2 v = {(__bf16)lo, (__bf16)hi};  // round to nearest even
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Score MFMAs of the one-wavefront-per-SIMD kernels (d_h = 256), written as inline assembly so that their accumulators live in ordinary
// vector registers: in a kernel that may use more than 256 registers the compiler keeps every MFMA accumulator
// it selects itself in the accumulation registers, which the vector ALU cannot read, and the exponentials would
// need one copy per score.  The compiler does not track matrix-core hazards through inline assembly: a chain's
// result must not be read by a vector-ALU instruction until 11 issue slots after its last MFMA (an 8-pass MFMA
// writes its result late); the steady-state schedule keeps more than that between a chain and its
// exponentials, and score_mfma_settle() pads the places where it does not.
__device__ __forceinline__ f32x16 score_mfma0(bf16x8 kf, bf16x8 qf) {
  f32x16 d;
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(kf), "v"(qf));
  return d;
}
__device__ __forceinline__ f32x16 score_mfma_from(bf16x8 kf, bf16x8 qf, const f32x16 &start) {
  f32x16 d;
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(kf), "v"(qf), "v"(start));
  return d;
}
__device__ __forceinline__ f32x16 score_mfma(bf16x8 kf, bf16x8 qf, f32x16 acc) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(kf), "v"(qf));
  return acc;
}
// 18 idle issue slots; the accumulators pass through as operands, so no read of them can be scheduled before it
__device__ __forceinline__ void score_mfma_settle(f32x16 &a, f32x16 &b) {
  asm volatile("s_nop 15\n\ts_nop 1" : "+v"(a), "+v"(b));
}

// ---- pieces shared by the three forms of the kernel below -----------------------------------------------------
// Query fragments of row `row` of head h: 8 channels per k-step for lane (l32, half), multiplied by c = scale *
// log2(e) and rounded back to bf16 (the scores then come out of the MFMA in log2 units).
template <int DH>
__device__ __forceinline__ void load_q_frags(const bf16_t *__restrict__ Q, long long row_index, int Hq, int h, int half,
                                             float c, bf16x8 *qf) {
  const bf16_t *p = Q + (row_index * Hq + h) * DH + half * 8;
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) {
    u32x4 w = *reinterpret_cast<const u32x4 *>(p + kk * 16);
    w.x = pack2(bf_lo(w.x) * c, bf_hi(w.x) * c);
    w.y = pack2(bf_lo(w.y) * c, bf_hi(w.y) * c);
    w.z = pack2(bf_lo(w.z) * c, bf_hi(w.z) * c);
    w.w = pack2(bf_lo(w.w) * c, bf_hi(w.w) * c);
    qf[kk] = __builtin_bit_cast(bf16x8, w);
  }
}

__device__ __forceinline__ float both_halves(float x) { return x + __shfl_xor(x, 32); }  // each half-wave sums half of the keys

// Epilogue of one 32-row tile: lane (l32, half) holds o[t][32 dt + 8 rg + 4 half + e] / l in oacc[dt][4 rg + e].
// Normalises by the row sum, rounds once to bf16, stores 8 bytes per (dt, rg); o_lo (optional) gets what the
// rounding dropped (the backward pass forms <dO, O> from o + o_lo); lse = ln of the row sum in the caller's
// units: (log2 l + shift) ln 2, with shift the reference max the scores were taken against.
// [DT0, DT1): the 32-channel tiles this wavefront holds.
template <int DH, int DT0 = 0, int DT1 = DH / 32>
__device__ __forceinline__ void store_rows(const f32x16 *oacc, float l, float shift, bf16_t *__restrict__ O,
                                           bf16_t *__restrict__ OLO, float *__restrict__ LSE, int b, int h, int t, int T,
                                           int Hq, int half) {
  if (t >= T) return;
  const float inv = 1.f / l;
  const long long off = (((long long)b * T + t) * Hq + h) * DH;
#pragma unroll
  for (int dt = DT0; dt < DT1; ++dt)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      u32x2 w;
      w.x = pack2(oacc[dt][rg * 4 + 0] * inv, oacc[dt][rg * 4 + 1] * inv);
      w.y = pack2(oacc[dt][rg * 4 + 2] * inv, oacc[dt][rg * 4 + 3] * inv);
      *reinterpret_cast<u32x2 *>(O + off + dt * 32 + rg * 8 + half * 4) = w;
      if (OLO) {
        u32x2 x;
        x.x = pack2(oacc[dt][rg * 4 + 0] * inv - bf_lo(w.x), oacc[dt][rg * 4 + 1] * inv - bf_hi(w.x));
        x.y = pack2(oacc[dt][rg * 4 + 2] * inv - bf_lo(w.y), oacc[dt][rg * 4 + 3] * inv - bf_hi(w.y));
        *reinterpret_cast<u32x2 *>(OLO + off + dt * 32 + rg * 8 + half * 4) = x;
      }
    }
  if (DT0 == 0 && LSE && half == 0) LSE[((long long)b * Hq + h) * T + t] = (log2f(l) + shift) * 0.69314718055994530942f;
}


// Two groups of wavefronts walked the two halves of the keys of the same rows (KS = 2): the partial results of a row,
// taken against the reference maxima m (a group that saw no score of the row above -inf has l = 0), are added through LDS.  Each group
// ends with the output tiles [kg * DT / 2, (kg + 1) * DT / 2) of its wavefront's rows; l and m are the row's afterwards.
// The K / V tiles in `smem` are no longer read by anyone when this is called.  MAY_LOSE: l = -inf in either group stays.
template <int DH, bool MAY_LOSE>
__device__ __forceinline__ void merge_key_groups(f32x16 *oacc, float &l, float &m, int kg, int wave_g, int lane,
                                                 unsigned char *smem) {
  constexpr int HT = DH / 64;  // output tiles a group keeps
  float *const buf = reinterpret_cast<float *>(smem) + lane;
  float *const mine = buf + (kg * 4 + wave_g) * (HT * 16 + 2) * 64, *const other = buf + ((1 - kg) * 4 + wave_g) * (HT * 16 + 2) * 64;
  // (values are selected, never array elements: a selected element would move the accumulators to scratch memory)
#pragma unroll
  for (int x = 0; x < HT; ++x)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float first = oacc[x][r], second = oacc[HT + x][r];
      mine[(x * 16 + r) * 64] = kg == 0 ? second : first;
    }
  mine[HT * 16 * 64] = l;
  mine[(HT * 16 + 1) * 64] = m;
  __syncthreads();
  const float lo = other[HT * 16 * 64], mo = other[(HT * 16 + 1) * 64];
  const float M = l == 0.f ? mo : lo == 0.f ? m : fmaxf(m, mo);
  const float f = l == 0.f ? 0.f : __builtin_amdgcn_exp2f(m - M), fo = lo == 0.f ? 0.f : __builtin_amdgcn_exp2f(mo - M);
  l = MAY_LOSE && fminf(l, lo) < 0.f ? -INFINITY : l * f + lo * fo;
  m = M;
#pragma unroll
  for (int x = 0; x < HT; ++x)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float first = oacc[x][r], second = oacc[HT + x][r];
      const float sum = (kg == 0 ? first : second) * f + other[(x * 16 + r) * 64] * fo;
      oacc[x][r] = kg == 0 ? sum : first;
      oacc[HT + x][r] = kg == 0 ? second : sum;
    }
  __syncthreads();  // the buffer may hold K / V tiles again
}

// Epilogue of a wavefront: the row sums over both half-waves, with KS = 2 the other group's part, then the rows.  Rows that
// either group lost (MAY_LOSE: l = -inf) are not stored; true for them.
template <int DH, int KS, bool MAY_LOSE>
__device__ __forceinline__ bool finish_rows(f32x16 *oacc, float l_part, float m, int kg, int wave_g, int lane, bool live,
                                            unsigned char *smem, bf16_t *__restrict__ O, bf16_t *__restrict__ OLO,
                                            float *__restrict__ LSE, int b, int h, int t, int T, int Hq) {
  float l = both_halves(l_part);
  const int half = lane >> 5;
  if constexpr (KS == 2) merge_key_groups<DH, MAY_LOSE>(oacc, l, m, kg, wave_g, lane, smem);
  if (!live) return false;
  if (MAY_LOSE && l < 0.f) return true;
  if constexpr (KS == 1) {
    store_rows<DH>(oacc, l, m, O, OLO, LSE, b, h, t, T, Hq, half);
  } else {
    if (kg == 0) store_rows<DH, 0, DH / 64>(oacc, l, m, O, OLO, LSE, b, h, t, T, Hq, half);
    else store_rows<DH, DH / 64, DH / 32>(oacc, l, m, O, OLO, LSE, b, h, t, T, Hq, half);
  }
  return false;
}

// One row by one wavefront, straight from memory, a key at a time against the running max itself: for rows whose scores
// attn_fwd_body could not hold against one reference max.  Lane = DH / 64 channels; same roundings of q and P as there.
template <int DH, bool RSUM>
__device__ __forceinline__ void single_row(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K, const bf16_t *__restrict__ V,
                                           bf16_t *__restrict__ O, bf16_t *__restrict__ OLO, float *__restrict__ LSE, int b, int h,
                                           int g, int t, int keys, int T, int Hq, int Hk, float c, int lane) {
  constexpr int CPL = DH / 64;
  asm volatile("" : "+v"(lane), "+s"(t));  // nothing of this may be formed ahead, it would take registers in the caller's loop
  const long long qo = (((long long)b * T + t) * Hq + h) * DH + lane * CPL;
  float q[CPL], acc[CPL], m = -INFINITY, l = 0.f;
#pragma unroll
  for (int x = 0; x < CPL; ++x) q[x] = bf_lo(pack2(bf_lo(Q[qo + x]) * c, 0.f)), acc[x] = 0.f;
  for (int key = 0; key < keys; ++key) {
    const long long ko = (((long long)b * T + key) * Hk + g) * DH + lane * CPL;
    float sc = 0.f;
#pragma unroll
    for (int x = 0; x < CPL; ++x) sc += q[x] * bf_lo(K[ko + x]);
#pragma unroll
    for (int d = 1; d < 64; d *= 2) sc += __uint_as_float(__builtin_amdgcn_ds_bpermute((lane ^ d) * 4, __float_as_uint(sc)));
    const float mn = fmaxf(m, sc), ref = mn == -INFINITY ? 0.f : mn;
    const float a = __builtin_amdgcn_exp2f(m - ref), p = __builtin_amdgcn_exp2f(sc - ref), pr = bf_lo(pack2(p, 0.f));
    l = l * a + (RSUM ? pr : p);
#pragma unroll
    for (int x = 0; x < CPL; ++x) acc[x] = acc[x] * a + pr * bf_lo(V[ko + x]);
    m = mn;
  }
  const float inv = 1.f / l;
#pragma unroll
  for (int x = 0; x < CPL; ++x) {
    const uint32_t w = pack2(acc[x] * inv, 0.f);
    O[qo + x] = (bf16_t)w;
    if (OLO) OLO[qo + x] = (bf16_t)pack2(acc[x] * inv - bf_lo(w), 0.f);
  }
  if (LSE && lane == 0) LSE[((long long)b * Hq + h) * T + t] = (log2f(l) + m) * 0.69314718055994530942f;
}

// BOUNDED: the caller guarantees |score| <= bound (log2 units) for every query / key pair, as the QK L2-norm
// of Sec. 2.2 does (|q| = sqrt(d_h), |k| = sqrt(d_h) * beta).  Then `bound` itself serves as the reference max
// of every row: no row max, no rescaling, and exp2 arguments lie in [-2*bound, 0].
// NTH threads = NTH / 64 wavefronts x 32 rows = BQ_ query rows per workgroup: 512 threads (256 rows, two wavefronts
// per SIMD) for d_h <= 128, 256 threads (128 rows, one wavefront per SIMD and twice the registers) for d_h = 256.
// KS = 2: two groups of NTH / 2 threads share the rows of one group (BQ_ = 128 at 512 threads, 64 at 256: fwd_takes_64_rows); group kg takes the key
// tiles 2 j + kg through LDS buffers of its own, and the two partial results of a row are merged at the end.
template <int DH, bool CAUSAL, bool BOUNDED, bool RSUM, int NTH = NT, int KS = 1>
__device__ __forceinline__ void attn_fwd_body(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                              const bf16_t *__restrict__ V, bf16_t *__restrict__ O,
                                              bf16_t *__restrict__ OLO, float *__restrict__ LSE, int T, int Hq, int Hk,
                                              int BH, int nqb,
                                              int paired, float scale, float bound, unsigned char *smem) {
  constexpr int KK = DH / 16;          // MFMA k-steps over the head width
  constexpr int DT = DH / 32;          // 32-wide output tiles over the head width
  constexpr int KCH = DH / 8;          // 16-byte chunks per key row
  constexpr int KROW = DH * 2 + 16;    // padded key row in LDS: conflict-free 16-byte reads down a column of rows
  constexpr int KBUF = BKV * KROW;     // bytes per K buffer
  constexpr int VROW = DH * 2 + 64;    // padded value row: the 4 rows x 32 bytes a transposing read touches per
                                       // 16 lanes fall into disjoint banks
  constexpr int VBUF = BKV * VROW;     // bytes per V buffer
  constexpr int NTG = NTH / KS;        // threads of a key group
  constexpr int K_PER_THREAD = BKV * KCH / NTG;
  constexpr int K_ROWS_PER_PASS = NTG / KCH;
  constexpr int BQ_ = NTG / 64 * 32;
  const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NTG);
  unsigned char *const sKb = smem + kg * 2 * (KBUF + VBUF);
  unsigned char *const sVb = sKb + 2 * KBUF;

  const int tid = threadIdx.x % NTG, lane = tid & 63, wave = tid >> 6;  // within the key group
  const int l32 = lane & 31, half = lane >> 5;
  const int idx = blockIdx.x;
  const int bh = idx % BH;  // head index fastest: with B*Hq a multiple of 8 an XCD keeps one head's K/V in its L2
  const int b = bh / Hq, h = bh % Hq, g = h / (Hq / Hk);
  const float c = scale * 1.44269504088896340736f;  // exp(x * scale) = exp2(x * c)
  const int row_bytes = Hk * DH * 2;                 // one token of K or V, all KV heads
  const unsigned char *const Kg = reinterpret_cast<const unsigned char *>(K + ((long long)b * T * Hk + g) * DH);
  const unsigned char *const Vg = reinterpret_cast<const unsigned char *>(V + ((long long)b * T * Hk + g) * DH);

  // ---- per-thread constants of the K/V staging
  const int k_r0 = tid / KCH, k_ch = tid % KCH;                 // K chunk i of this thread: row k_r0 + i*K_ROWS_PER_PASS
  const uint32_t k_goff = (uint32_t)k_r0 * row_bytes + k_ch * 16;
  const uint32_t k_soff = (uint32_t)k_r0 * KROW + k_ch * 16;
  const uint32_t v_soff = (uint32_t)k_r0 * VROW + k_ch * 16;    // V is staged with the same thread -> chunk map
  // ---- per-lane constants of the MFMA operand reads
  const uint32_t kr_off = (uint32_t)l32 * KROW + half * 16;  // + ks*32*KROW + kk*32
  // Transposing read: in each block of 16 lanes, lane i supplies the address of 4 channels of one key and
  // receives element (i & 3) of the vectors addressed by lanes (i >> 2) + 4*j, j = 0..3.  With lane i pointing
  // at key 4*half + (i >> 2) + ..., channels dblock*16 + 4*(i & 3)..+3, lane L of the block receives channel
  // dblock*16 + L of keys 4*half + 0..3: exactly the MFMA fragment of lane (d = l32, half).
  const uint32_t vr_off = (uint32_t)(4 * half + ((lane & 15) >> 2)) * VROW + (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2;

  u32x4 rk[K_PER_THREAD];
  u32x4 rv[K_PER_THREAD];
  auto load_tile = [&](int kv0) {
    if (kv0 + BKV <= T) {  // whole tile in range: uniform bases + one per-thread offset
      const unsigned char *kb = Kg + (long long)kv0 * row_bytes;
      const unsigned char *vb = Vg + (long long)kv0 * row_bytes;
#pragma unroll
      for (int i = 0; i < K_PER_THREAD; ++i)
        rk[i] = *reinterpret_cast<const u32x4 *>(kb + (long long)i * K_ROWS_PER_PASS * row_bytes + k_goff);
#pragma unroll
      for (int i = 0; i < K_PER_THREAD; ++i)
        rv[i] = *reinterpret_cast<const u32x4 *>(vb + (long long)i * K_ROWS_PER_PASS * row_bytes + k_goff);
    } else {  // ragged last tile: clamp the key index (clamped keys are masked out below)
#pragma unroll
      for (int i = 0; i < K_PER_THREAD; ++i) {
        const int s = min(kv0 + k_r0 + i * K_ROWS_PER_PASS, T - 1);
        rk[i] = *reinterpret_cast<const u32x4 *>(Kg + (long long)s * row_bytes + k_ch * 16);
        rv[i] = *reinterpret_cast<const u32x4 *>(Vg + (long long)s * row_bytes + k_ch * 16);
      }
    }
  };
  auto store_tile = [&](int buf) {
    unsigned char *kd = sKb + buf * KBUF + k_soff;
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4 *>(kd + i * K_ROWS_PER_PASS * KROW) = rk[i];
    unsigned char *vd = sVb + buf * VBUF + v_soff;
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4 *>(vd + i * K_ROWS_PER_PASS * VROW) = rv[i];
  };

  const int npass = paired ? 2 : 1;
  for (int pass = 0; pass < npass; ++pass) {
    // causal work per query block grows with its index: heavy blocks are issued first (unpaired),
    // or each workgroup takes one heavy and one light block (paired) so all workgroups do equal work
    const int slot = idx / BH;
    const int qb = (paired && pass == 1) ? slot : nqb - 1 - slot;
    if (pass == 1 && slot >= nqb - 1 - slot) break;  // odd count: the middle block was done in pass 0
    const int q0 = qb * BQ_, qw0 = q0 + wave * 32;
    const bool wave_live = qw0 < T;
    const int wave_last = min(qw0 + 31, T - 1);

    // ---- query fragment of row qw0 + l32, scaled to log2 units and rounded back to bf16
    bf16x8 qf[KK];
    load_q_frags<DH>(Q, (long long)b * T + min(qw0 + l32, T - 1), Hq, h, half, c, qf);

    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
    f32x16 negm;  // minus the reference max (log2 units) of this lane's query row, replicated: MFMA start value
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = BOUNDED ? -bound : 0.f;
    float l_run = 0.f, l_run2 = 0.f;  // running sums of probabilities (two chains); each half-wave keeps its own part
    bool unset = true;                // every score of this row was -inf so far: its reference max is still to come

    const int kv_end = CAUSAL ? min(q0 + BQ_, T) : T;  // keys [0, kv_end) matter to this workgroup
    const int ntiles = ((kv_end + BKV - 1) / BKV + KS - 1) / KS;  // of a key group (the last one may lie past the end)

    auto tile = [&](int j, auto buf_c) {
      constexpr int BUF = decltype(buf_c)::value;
      const int kv0 = (j * KS + kg) * BKV;
      // Tile j+1 is already in registers (loaded while tile j-1 was multiplied): put it into the other LDS
      // buffer right away, so that its stores drain under this tile's MFMAs instead of in front of the
      // barrier, then start the loads of tile j+2 into the same registers.
      if (j + 1 < ntiles) store_tile(BUF ^ 1);  // that buffer was last read before the barrier ending tile j-1
      if (j + 2 < ntiles) load_tile(kv0 + 2 * KS * BKV);
      if (wave_live && kv0 <= (CAUSAL ? wave_last : T - 1)) {
        const unsigned char *kp = sKb + BUF * KBUF + kr_off;
        // ---- S^T - m = K Q^T - m for 64 keys x 32 query rows (log2 units)
        // (one wavefront per SIMD: inline-assembly MFMAs keep the scores in ordinary vector registers, see above)
        constexpr bool INLINE_S = DH == 256;
        f32x16 sacc[2];
        // Fragments are requested PF_ products ahead, one behind each product, and the second half's exponentials stand between the
        // first half's products: left to the compiler a fragment was read, waited for and multiplied, and all exponentials came
        // before the first product of V.  One wavefront per SIMD has nothing else to hide that behind.  Causal, before -> now, us (heads,
        // sequences x tokens): d_h = 256, 8, 1 x 1024 64.2 -> 52.6, 1 x 4096 224 -> 179; 128, 16, 1 x 2048 39.7 -> 37.4, 1 x 4096 84.2
        // -> 80.4, 1 x 8192 248.0 -> 247.4; 64, 32, 2 x 6000 368 -> 359.
        constexpr int PF_ = INLINE_S ? 4 : PF;
        bf16x8 fr[2 * KK], vr[4 * DT];
        auto kfrag = [&](int i) __attribute__((always_inline)) {  // product i: half i % 2 of the keys, k-step i / 2
          fr[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kp + (i & 1) * 32 * KROW + (i >> 1) * 32));
        };
        const unsigned char *vp = sVb + BUF * VBUF + vr_off;
        auto vfrag = [&](int i) __attribute__((always_inline)) {  // product i: (half, 16 keys of it, 32 channels)
          const unsigned char *a = vp + (i / DT) * 16 * VROW + (i % DT) * 64;
          const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)a);
          const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(a + 8 * VROW));
          vr[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };
#pragma unroll
        for (int i = 0; i < PF_; ++i) kfrag(i);
        __builtin_amdgcn_sched_barrier(0);
        // (inline-assembly MFMAs: a query fragment that lives in the accumulation registers is copied out two products before its first use,
        // for the compiler does not keep the copy and an inline MFMA apart)
        bf16x8 qn[2] = {qf[0], qf[0]};
        if constexpr (INLINE_S) {
          asm volatile("" : "+v"(qn[0]));
          asm volatile("s_nop 3");
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * KK; ++i) {
          const int kk = i >> 1;
          if constexpr (INLINE_S)
            if (!(i & 1) && kk + 1 < KK) {
              qn[(kk + 1) & 1] = qf[kk + 1];
              asm volatile("" : "+v"(qn[(kk + 1) & 1]));
              __builtin_amdgcn_sched_barrier(0);
            }
          if (i + PF_ < 2 * KK) kfrag(i + PF_);
          f32x16 &sc = sacc[i & 1];
          if constexpr (INLINE_S) sc = i < 2 ? score_mfma_from(fr[i], qn[0], negm) : score_mfma(fr[i], qn[kk & 1], sc);
          else sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], qf[kk], i < 2 ? negm : sc, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (INLINE_S) score_mfma_settle(sacc[0], sacc[1]);

        // ---- lane (l32, half) holds keys kv0 + ks*32 + 8*(r/4) + 4*half + r%4 of row qw0 + l32
        if ((CAUSAL && kv0 + BKV - 1 > qw0) || (kv0 + BKV > T)) {
          const int t = qw0 + l32;
          const int lim = (CAUSAL ? min(t, T - 1) : T - 1) - kv0 - 4 * half;  // last visible key, tile-relative
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (ks * 32 + 8 * (r >> 2) + (r & 3) > lim) sacc[ks][r] = -INFINITY;
        }
        if (!BOUNDED) {
          float mx0 = max3(sacc[0][0], sacc[0][1], sacc[0][2]), mx1 = max3(sacc[1][0], sacc[1][1], sacc[1][2]);
  #pragma unroll
          for (int r = 3; r < 15; r += 2) {  // two independent chains
            mx0 = max3(mx0, sacc[0][r], sacc[0][r + 1]);
            mx1 = max3(mx1, sacc[1][r], sacc[1][r + 1]);
          }
          float mx = max3(mx0, mx1, fmaxf(sacc[0][15], sacc[1][15]));
          {  // the other half-wave holds the other 32 keys of the same row: exchange on the vector ALU, not through LDS
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
          }
          // Move the reference max only on a row's first tile with a score above -inf (to the tile's own max: -inf itself
          // would leave inf - inf; keys may be masked by scores of -inf, and a key group may hold nothing but such keys) or
          // when a score exceeds it by more than 2^RESCALE_LOG2; exp2 arguments stay <= RESCALE_LOG2.
          if (__any(unset || mx > RESCALE_LOG2)) {
            const float delta = unset ? (mx == -INFINITY ? 0.f : mx) : fmaxf(mx, 0.f);
            const float alpha = unset ? 1.f : __builtin_amdgcn_exp2f(-delta);  // nothing summed yet: 2^-delta may be inf
            // Scores rounded against a reference far below them (keys masked by a type's lowest value ahead of the live ones):
            // the row is lost, which its sum says for want of a register, and taken again by single_row.
            const bool lost = (!unset && delta > LOST_LOG2 && negm[0] > LOST_LOG2) || l_run2 == -INFINITY;
            unset = unset && mx == -INFINITY;
            l_run *= alpha;
            l_run2 = lost ? -INFINITY : l_run2 * alpha;
  #pragma unroll
            for (int r = 0; r < 16; ++r) negm[r] -= delta;
  #pragma unroll
            for (int ks = 0; ks < 2; ++ks)
  #pragma unroll
              for (int r = 0; r < 16; ++r) sacc[ks][r] -= delta;
  #pragma unroll
            for (int dt = 0; dt < DT; ++dt)
  #pragma unroll
              for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
          }
        }
        // probabilities of the first half, then those of the second between the first half's products
        u32x4 pw[2][2];
        auto unit = [&](int ks, int u) __attribute__((always_inline)) {  // scores 2u, 2u + 1
          const float x0 = __builtin_amdgcn_exp2f(sacc[ks][2 * u]), x1 = __builtin_amdgcn_exp2f(sacc[ks][2 * u + 1]);
          const uint32_t w = pack2(x0, x1);
          pw[ks][u >> 2][u & 3] = w;
          l_run += RSUM ? bf_lo(w) : x0;
          l_run2 += RSUM ? bf_hi(w) : x1;
        };
#pragma unroll
        for (int i = 0; i < PF_; ++i) vfrag(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) unit(0, u);
        __builtin_amdgcn_sched_barrier(0);
        // ---- O^T += V^T P^T
#pragma unroll
        for (int i = 0; i < 4 * DT; ++i) {
          if (i + PF_ < 4 * DT) vfrag(i + PF_);
          const int ks = i / (2 * DT), jj = i / DT & 1;
          oacc[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[i], __builtin_bit_cast(bf16x8, pw[ks][jj]), oacc[i % DT], 0, 0, 0);
          // (8 pairs of scores behind 2 DT products)
#pragma unroll
          for (int u = i * 4 / DT; u < (i + 1) * 4 / DT; ++u)
            if (u < 8) unit(1, u);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
    };

    load_tile(kg * BKV);
    store_tile(0);
    if (ntiles > 1) load_tile((KS + kg) * BKV);
    __syncthreads();
    for (int j = 0; j < ntiles; j += 2) {
      tile(j, std::integral_constant<int, 0>{});
      if (j + 1 < ntiles) tile(j + 1, std::integral_constant<int, 1>{});
    }

    // ---- epilogue: normalise, round once to bf16, store; log-sum-exp of the scaled logits
    int te = threadIdx.x;  // (anew, so that no lane or row number takes a register in the loop)
    asm volatile("" : "+v"(te));
    const int lane_e = te & 63, wave_e = te % NTG >> 6, qw_e = q0 + wave_e * 32;
    const bool lost = finish_rows<DH, KS, !BOUNDED>(oacc, l_run + l_run2, -negm[0], kg, wave_e, lane_e, qw_e < T, smem, O, OLO, LSE, b,
                                                    h, qw_e + (lane_e & 31), T, Hq);
    if (!BOUNDED && kg == 0 && __any(lost)) {
      uint32_t rows = (uint32_t)__ballot(lost);
      for (; rows; rows &= rows - 1) {
        const int t = __builtin_amdgcn_readfirstlane(qw_e) + __builtin_ctz(rows);
        if (t < T) single_row<DH, RSUM>(Q, K, V, O, OLO, LSE, b, h, g, t, CAUSAL ? t + 1 : T, T, Hq, Hk, c, lane_e);
      }
    }
  }
}


// Bounded scores (see above): no row max, no rescaling, so a tile's softmax is independent of every other
// tile's and the loop can be software-pipelined INSIDE a wavefront.  On this chip a wavefront whose next
// instruction is an MFMA waiting for the matrix core also keeps the other wavefront of its SIMD from issuing
// vector-ALU work, so two wavefronts do not hide each other's exponentials; the overlap has to come from one
// instruction stream in which every MFMA is followed by a few vector-ALU instructions that run in its shadow.
// Iteration j therefore issues, in this fixed order (PF operand fetches ahead of use):
//   S0(j+1), PV0(j) alternating  |  exp2 / pack / row-sum of S1(j)   -> P1(j)
//   S1(j+1), PV1(j) alternating  |  exp2 / pack / row-sum of S0(j+1) -> P0(j+1)
// where 0 / 1 are the two 32-key halves of a tile.  K therefore runs one tile ahead of V in LDS.
enum { IT_PRO = 0, IT_FULL = 1, IT_FINAL = 2, IT_IDLE = 3 };

template <int DH, bool CAUSAL, bool RSUM, int KS, int NTH>
__device__ __forceinline__ void attn_fwd_pipelined(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                   const bf16_t *__restrict__ V, bf16_t *__restrict__ O,
                                                   bf16_t *__restrict__ OLO, float *__restrict__ LSE, int T, int Hq,
                                                   int Hk, int BH, int nqb, int paired, float scale, float bound,
                                                   unsigned char *smem) {
  constexpr int KK = DH / 16, DT = DH / 32, KCH = DH / 8;
  constexpr int KROW = DH * 2 + 16, KBUF = BKV * KROW, VROW = DH * 2 + 64, VBUF = BKV * VROW;
  constexpr int NTG = NTH / KS, K_PER_THREAD = BKV * KCH / NTG, K_ROWS_PER_PASS = NTG / KCH, BQ_ = NTG / 64 * 32;
  constexpr int NB = KK;  // MFMAs per (half-tile score | half-tile PV) block; 2 * DT == KK
  static_assert(2 * DT == KK, "block sizes");
  const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NTG);  // key group (see attn_fwd_body)
  unsigned char *const sKb = smem + kg * 2 * (KBUF + VBUF);
  unsigned char *const sVb = sKb + 2 * KBUF;

  const int tid = threadIdx.x % NTG, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  // Wavefronts w and w + 4 share a SIMD.  Under the causal mask a row block needs more key tiles the further
  // down it lies, so the 32-row blocks are dealt such that every SIMD gets a light and a heavy one (0 and 7,
  // 1 and 6, ...): the SIMDs then carry equal work through the diagonal tiles of a query block.  (With two key groups
  // they own the same rows.)
  const int wave_r = wave < 4 ? wave : 11 - wave;
  const int idx = blockIdx.x;
  const int bh = idx % BH;
  const int b = bh / Hq, h = bh % Hq, g = h / (Hq / Hk);
  const float c = scale * 1.44269504088896340736f;
  const int row_bytes = Hk * DH * 2;
  const unsigned char *const Kg = reinterpret_cast<const unsigned char *>(K + ((long long)b * T * Hk + g) * DH);
  const unsigned char *const Vg = reinterpret_cast<const unsigned char *>(V + ((long long)b * T * Hk + g) * DH);
  const int k_r0 = tid / KCH, k_ch = tid % KCH;
  const uint32_t k_soff = (uint32_t)k_r0 * KROW + k_ch * 16;
  const uint32_t v_soff = (uint32_t)k_r0 * VROW + k_ch * 16;
  const uint32_t kr_off = (uint32_t)l32 * KROW + half * 16;
  const uint32_t vr_off = (uint32_t)(4 * half + ((lane & 15) >> 2)) * VROW + (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2;

  u32x4 rk[K_PER_THREAD];
  u32x4 rv[K_PER_THREAD];
  // K / V tiles are fetched with buffer loads.  Each tile gets its own descriptor (scalar arithmetic only): it
  // starts at the tile's first row and ends with row T-1 of this (batch item, KV head), so a thread's chunk
  // offsets are loop constants and rows past the end of the sequence (ragged last tile) fail the hardware's
  // range check and read as zeros: no address arithmetic on the vector ALU inside the loop.
  const int kv_span = (T - 1) * row_bytes + DH * 2;
  int k_goff[K_PER_THREAD];
#pragma unroll
  for (int i = 0; i < K_PER_THREAD; ++i) k_goff[i] = (k_r0 + i * K_ROWS_PER_PASS) * row_bytes + k_ch * 16;
  auto load_rows = [&](const unsigned char *base, int j, u32x4 *dst) {  // tile j of this key group
    // (a group's last tile may start past the end when the other group has one more: it is loaded from tile 0 and never used)
    const int kt = j * KS + kg, first = KS == 1 || kt * BKV < T ? kt * BKV * row_bytes : 0;
    const __amdgpu_buffer_rsrc_t res =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(base) + first, 0, kv_span - first, 0x00020000);
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) dst[i] = __builtin_amdgcn_raw_buffer_load_b128(res, k_goff[i], 0, 0);
  };
  auto store_k = [&](int buf) {
    unsigned char *kd = sKb + buf * KBUF + k_soff;
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4 *>(kd + i * K_ROWS_PER_PASS * KROW) = rk[i];
  };
  auto store_v = [&](int buf) {
    unsigned char *vd = sVb + buf * VBUF + v_soff;
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4 *>(vd + i * K_ROWS_PER_PASS * VROW) = rv[i];
  };
  // LDS traffic only: the global loads in flight (next tiles) are not waited for
  auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  const int npass = paired ? 2 : 1;
  for (int pass = 0; pass < npass; ++pass) {
    const int slot = idx / BH;
    const int qb = (paired && pass == 1) ? slot : nqb - 1 - slot;
    if (pass == 1 && slot >= nqb - 1 - slot) break;
    const int q0 = qb * BQ_, qw0 = q0 + wave_r * 32;
    const bool wave_live = qw0 < T;
    const int wave_last = min(qw0 + 31, T - 1);

    bf16x8 qf[KK];
    load_q_frags<DH>(Q, (long long)b * T + min(qw0 + l32, T - 1), Hq, h, half, c, qf);
    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
    f32x16 negm;
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = -bound;
    float l_run = 0.f, l_run2 = 0.f;

    const int kv_end = CAUSAL ? min(q0 + BQ_, T) : T;
    const int all_tiles = (kv_end + BKV - 1) / BKV, ntiles = (all_tiles + KS - 1) / KS;  // of the block, of a key group
    const int vis_tiles = CAUSAL ? min(all_tiles, wave_last / BKV + 1) : all_tiles;      // with keys this wavefront's rows see
    const int my_tiles = !wave_live ? 0 : (vis_tiles - kg + KS - 1) / KS;
    const int t_lim = (CAUSAL ? min(qw0 + l32, T - 1) : T - 1) - 4 * half;  // last visible key (minus the lane's offset)

    f32x16 sacc[2];      // scores of the two halves: [0] of tile j+1, [1] of tile j while iteration j runs
    uint32_t pw[2][8];   // probabilities (bf16 pairs) of the two halves, the second MFMA operand of PV

    // one softmax unit: scores 2u, 2u+1 of half `hs` (tile kt) -> exp2 -> one packed word + row sum
    float e0, e1;
    auto unit_exp = [&](int hs, int u, int kt, bool mask) {
      float s0 = sacc[hs][2 * u], s1 = sacc[hs][2 * u + 1];
      if (mask) {
        const int key = (kt * KS + kg) * BKV + hs * 32 + 8 * ((2 * u) >> 2) + ((2 * u) & 3);
        if (key > t_lim) s0 = -INFINITY;
        if (key + 1 > t_lim) s1 = -INFINITY;
      }
      e0 = __builtin_amdgcn_exp2f(s0);
      e1 = __builtin_amdgcn_exp2f(s1);
    };
    auto unit_pack = [&](int hs, int u) {
      const uint32_t pk = pack2(e0, e1);
      pw[hs][u] = pk;
      l_run += RSUM ? bf_lo(pk) : e0;
      l_run2 += RSUM ? bf_hi(pk) : e1;
    };
    auto pfrag = [&](int hs, int jj) {
      const u32x4 w = {pw[hs][4 * jj], pw[hs][4 * jj + 1], pw[hs][4 * jj + 2], pw[hs][4 * jj + 3]};
      return __builtin_bit_cast(bf16x8, w);
    };

    auto iter = [&](int j, auto kind_c, auto mask_c) {
      constexpr int KIND = decltype(kind_c)::value;
      constexpr bool MASK = decltype(mask_c)::value;
      const unsigned char *kp = sKb + ((j + 1) & 1) * KBUF + kr_off;  // K(j+1)
      const unsigned char *vp = sVb + (j & 1) * VBUF + vr_off;        // V(j)
      auto kfrag = [&](int ks, int kk) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kp + ks * 32 * KROW + kk * 32));
      };
      auto vfrag = [&](int ks, int p) {  // p = jj * DT + dt
        const int jj = p / DT, dt = p % DT;
        const unsigned char *a = vp + (ks * 32 + jj * 16) * VROW + dt * 64;
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)a);
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(a + 8 * VROW));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      auto mem_store = [&]() {  // K(j+2), V(j+1): their buffers were last read in iteration j-1
        store_k(j & 1);
        store_v((j + 1) & 1);
      };
      auto mem_load = [&]() {  // past the last tile the loads repeat it and the stores land in idle buffers
        load_rows(Kg, min(j + 3, ntiles - 1), rk);
        load_rows(Vg, min(j + 2, ntiles - 1), rv);
      };
      if (KIND == IT_FULL) {
        // packet i: fetch for MFMA i + PF; MFMA i; vector-ALU chunk i.  MFMA order: even i -> scores of half
        // (i >= 2 NB) of tile j+1, k-step (i mod 2NB) / 2; odd i -> PV of that half of tile j.
        constexpr int NP = 4 * NB;
        bf16x8 fr[NP];
        auto fetch = [&](int i) {
          const int hs = i / (2 * NB), q = (i % (2 * NB)) / 2;
          fr[i] = (i & 1) ? vfrag(hs, q) : kfrag(hs, q);
        };
#pragma unroll
        for (int i = 0; i < PF; ++i) fetch(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          if (i + PF < NP) fetch(i + PF);
          const int hs = i / (2 * NB), q = (i % (2 * NB)) / 2;
          if (i & 1) {
            const int jj = q / DT, dt = q % DT;
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], pfrag(hs, jj), oacc[dt], 0, 0, 0);
          } else {
            sacc[hs] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], qf[q], q == 0 ? negm : sacc[hs], 0, 0, 0);
          }
          // softmax unit u = i / 2: units 0..7 -> half 1 of tile j, units 8..15 -> half 0 of tile j+1
          // (for DH = 64 there are 16 packets and two units per pair of packets)
          constexpr int UPP = 16 / (NP / 2);  // units per pair of packets
#pragma unroll
          for (int x = 0; x < UPP; ++x) {
            const int u = (i / 2) * UPP + x, hs_u = u < 8 ? 1 : 0, uu = u & 7;
            if (UPP == 1) {
              if (!(i & 1)) unit_exp(hs_u, uu, u < 8 ? j : j + 1, MASK);
              else unit_pack(hs_u, uu);
            } else if ((i & 1) == x) {
              unit_exp(hs_u, uu, u < 8 ? j : j + 1, MASK);
              unit_pack(hs_u, uu);
            }
          }
          if (i == 3) {
            mem_store();
            mem_load();
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else if (KIND == IT_PRO) {  // j = -1: scores of tile 0 (both halves), probabilities of its half 0
        mem_store();
        mem_load();
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
          for (int hs = 0; hs < 2; ++hs)
            sacc[hs] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(hs, kk), qf[kk], kk == 0 ? negm : sacc[hs], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          unit_exp(0, u, 0, MASK);
          unit_pack(0, u);
        }
      } else if (KIND == IT_FINAL) {  // j = my_tiles - 1: no further scores
        mem_store();
        mem_load();
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          unit_exp(1, u, j, MASK);
          unit_pack(1, u);
        }
#pragma unroll
        for (int hs = 0; hs < 2; ++hs)
#pragma unroll
          for (int p = 0; p < 2 * DT; ++p)
            oacc[p % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfrag(hs, p), pfrag(hs, p / DT), oacc[p % DT], 0, 0, 0);
      } else {
        mem_store();
        mem_load();
      }
      lds_barrier();
    };
    using PRO_ = std::integral_constant<int, IT_PRO>;
    using FULL_ = std::integral_constant<int, IT_FULL>;
    using FINAL_ = std::integral_constant<int, IT_FINAL>;
    using IDLE_ = std::integral_constant<int, IT_IDLE>;
    using T_ = std::true_type;
    using F_ = std::false_type;

    load_rows(Kg, 0, rk);
    store_k(0);
    load_rows(Kg, min(1, ntiles - 1), rk);
    load_rows(Vg, 0, rv);
    lds_barrier();
    int j = -1;
    if (my_tiles > 0) {
      if (my_tiles == 1) iter(-1, PRO_{}, T_{});
      else iter(-1, PRO_{}, F_{});
      for (j = 0; j < my_tiles - 2; ++j) iter(j, FULL_{}, F_{});
      if (my_tiles >= 2) iter(my_tiles - 2, FULL_{}, T_{});
      iter(my_tiles - 1, FINAL_{}, T_{});
      j = my_tiles;
    }
    for (; j < ntiles; ++j) iter(j, IDLE_{}, F_{});

    // ---- epilogue: normalise, round once to bf16, store; log-sum-exp of the scaled logits
    finish_rows<DH, KS, false>(oacc, l_run + l_run2, bound, kg, wave, lane, wave_live, smem, O, OLO, LSE, b, h, qw0 + l32, T, Hq);
  }
}

// The same software pipeline for ONE wavefront per SIMD (4 wavefronts per workgroup, 512 registers each): the
// form for d_h = 256, whose 128 output accumulators, 64 query-fragment registers and two sets of scores do not fit
// the 256 registers two wavefronts per SIMD leave.  RB = row tiles (32 query rows each) per wavefront: 1 at
// d_h = 256 (128 rows per workgroup).  RB = 2 (64 rows per wavefront, every K / V fragment feeding two MFMAs, half
// the LDS bytes per MFMA) also works for d_h <= 128 and was measured there: no faster than two wavefronts per
// SIMD with 32 rows each (a single wavefront issues at most one instruction every ~7 cycles), so d_h <= 128 stays
// on attn_fwd_pipelined.  The output accumulators live in the accumulation registers (the compiler puts every
// MFMA accumulator it selects itself there once a kernel may use more than 256 registers); the scores are left
// un-shifted (|s| <= bound <= 60 in log2 units keeps 2^s, the row sums and the PV products inside the fp32 range),
// so the chains start from zero.
template <int DH, bool CAUSAL, bool RSUM, int RB>
__device__ __forceinline__ void attn_fwd_pipelined_wide(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                     const bf16_t *__restrict__ V, bf16_t *__restrict__ O,
                                                     bf16_t *__restrict__ OLO, float *__restrict__ LSE, int T, int Hq,
                                                     int Hk, int BH, int nqb, int paired, float scale,
                                                     unsigned char *smem) {
  constexpr int NTH = 256, WROWS = 32 * RB, BQ_ = NTH / 64 * WROWS;
  constexpr int KK = DH / 16, DT = DH / 32, KCH = DH / 8;
  constexpr int KROW = DH * 2 + 16, KBUF = BKV * KROW, VROW = DH * 2 + 64, VBUF = BKV * VROW;
  constexpr int K_PER_THREAD = BKV * KCH / NTH, K_ROWS_PER_PASS = NTH / KCH;
  constexpr int NB = KK;  // fragments per (half-tile score | half-tile PV) block; 2 * DT == KK
  static_assert(2 * DT == KK, "block sizes");
  unsigned char *const sKb = smem;
  unsigned char *const sVb = smem + 2 * KBUF;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int idx = blockIdx.x;
  const int bh = idx % BH;
  const int b = bh / Hq, h = bh % Hq, g = h / (Hq / Hk);
  const float c = scale * 1.44269504088896340736f;
  const int row_bytes = Hk * DH * 2;
  const unsigned char *const Kg = reinterpret_cast<const unsigned char *>(K + ((long long)b * T * Hk + g) * DH);
  const unsigned char *const Vg = reinterpret_cast<const unsigned char *>(V + ((long long)b * T * Hk + g) * DH);
  const int k_r0 = tid / KCH, k_ch = tid % KCH;
  const uint32_t k_soff = (uint32_t)k_r0 * KROW + k_ch * 16;
  const uint32_t v_soff = (uint32_t)k_r0 * VROW + k_ch * 16;
  const uint32_t kr_off = (uint32_t)l32 * KROW + half * 16;
  const uint32_t vr_off = (uint32_t)(4 * half + ((lane & 15) >> 2)) * VROW + (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2;

  // K / V tiles are fetched with buffer loads.  Each tile gets its own descriptor (scalar arithmetic only): it
  // starts at the tile's first row and ends with row T-1 of this (batch item, KV head), so a thread's chunk
  // offsets are loop constants and rows past the end of the sequence (ragged last tile) fail the hardware's
  // range check and read as zeros: no address arithmetic on the vector ALU inside the loop.
  const int kv_span = (T - 1) * row_bytes + DH * 2;
  int k_goff[K_PER_THREAD];
#pragma unroll
  for (int i = 0; i < K_PER_THREAD; ++i) k_goff[i] = (k_r0 + i * K_ROWS_PER_PASS) * row_bytes + k_ch * 16;
  u32x4 rk[K_PER_THREAD];
  u32x4 rv[K_PER_THREAD];
  auto load_rows = [&](const unsigned char *base, int kt, u32x4 *dst) {  // kt * BKV < T
    const int first = kt * BKV * row_bytes;
    const __amdgpu_buffer_rsrc_t res =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(base) + first, 0, kv_span - first, 0x00020000);
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) dst[i] = __builtin_amdgcn_raw_buffer_load_b128(res, k_goff[i], 0, 0);
  };
  auto store_k = [&](int buf) {
    unsigned char *kd = sKb + buf * KBUF + k_soff;
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4 *>(kd + i * K_ROWS_PER_PASS * KROW) = rk[i];
  };
  auto store_v = [&](int buf) {
    unsigned char *vd = sVb + buf * VBUF + v_soff;
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4 *>(vd + i * K_ROWS_PER_PASS * VROW) = rv[i];
  };
  auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  const int npass = paired ? 2 : 1;
  for (int pass = 0; pass < npass; ++pass) {
    const int slot = idx / BH;
    const int qb = (paired && pass == 1) ? slot : nqb - 1 - slot;
    if (pass == 1 && slot >= nqb - 1 - slot) break;
    const int q0 = qb * BQ_, qw0 = q0 + wave * WROWS;
    const bool wave_live = qw0 < T;
    const int wave_last = min(qw0 + WROWS - 1, T - 1);

    bf16x8 qf[RB][KK];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      load_q_frags<DH>(Q, (long long)b * T + min(qw0 + rb * 32 + l32, T - 1), Hq, h, half, c, qf[rb]);
    f32x16 oacc[RB][DT];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[rb][dt][r] = 0.f;
    float l_run[RB], l_run2[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) l_run[rb] = l_run2[rb] = 0.f;

    const int kv_end = CAUSAL ? min(q0 + BQ_, T) : T;
    const int ntiles = (kv_end + BKV - 1) / BKV;
    const int my_tiles = !wave_live ? 0 : CAUSAL ? min(ntiles, wave_last / BKV + 1) : ntiles;
    int t_lim[RB];  // last visible key of the lane's row in each row tile (minus the lane's key offset)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) t_lim[rb] = (CAUSAL ? min(qw0 + rb * 32 + l32, T - 1) : T - 1) - 4 * half;

    f32x16 sacc[2][RB];      // scores: [0] of tile j+1, [1] of tile j while iteration j runs
    uint32_t pw[2][RB][8];   // probabilities (bf16 pairs), the second MFMA operand of PV

    float e0, e1;
    auto unit_exp = [&](int hs, int rb, int u, int kt, bool mask) {
      float s0 = sacc[hs][rb][2 * u], s1 = sacc[hs][rb][2 * u + 1];
      if (mask) {
        const int key = kt * BKV + hs * 32 + 8 * ((2 * u) >> 2) + ((2 * u) & 3);
        if (key > t_lim[rb]) s0 = -INFINITY;
        if (key + 1 > t_lim[rb]) s1 = -INFINITY;
      }
      e0 = __builtin_amdgcn_exp2f(s0);
      e1 = __builtin_amdgcn_exp2f(s1);
    };
    auto unit_pack = [&](int hs, int rb, int u) {
      const uint32_t pk = pack2(e0, e1);
      pw[hs][rb][u] = pk;
      l_run[rb] += RSUM ? bf_lo(pk) : e0;
      l_run2[rb] += RSUM ? bf_hi(pk) : e1;
    };
    auto pfrag = [&](int hs, int rb, int jj) {
      const u32x4 w = {pw[hs][rb][4 * jj], pw[hs][rb][4 * jj + 1], pw[hs][rb][4 * jj + 2], pw[hs][rb][4 * jj + 3]};
      return __builtin_bit_cast(bf16x8, w);
    };

    auto iter = [&](int j, auto kind_c, auto mask_c) {
      constexpr int KIND = decltype(kind_c)::value;
      constexpr bool MASK = decltype(mask_c)::value;
      const unsigned char *kp = sKb + ((j + 1) & 1) * KBUF + kr_off;  // K(j+1)
      const unsigned char *vp = sVb + (j & 1) * VBUF + vr_off;        // V(j)
      auto kfrag = [&](int ks, int kk) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kp + ks * 32 * KROW + kk * 32));
      };
      auto vfrag = [&](int ks, int p) {  // p = jj * DT + dt
        const int jj = p / DT, dt = p % DT;
        const unsigned char *a = vp + (ks * 32 + jj * 16) * VROW + dt * 64;
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)a);
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(a + 8 * VROW));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      auto mem_store = [&]() {  // K(j+2), V(j+1): their buffers were last read in iteration j-1
        store_k(j & 1);
        store_v((j + 1) & 1);
      };
      auto mem_load = [&]() {  // past the last tile the loads repeat it and the stores land in idle buffers
        load_rows(Kg, min(j + 3, ntiles - 1), rk);
        load_rows(Vg, min(j + 2, ntiles - 1), rv);
      };
      if (KIND == IT_FULL) {
        // packet i: fetch fragment i + PF64; the RB MFMAs fed by fragment i, each followed by vector-ALU work.
        // Fragment order: even i -> K fragment of half (i >= 2 NB) of tile j+1, k-step (i mod 2NB) / 2 (scores);
        // odd i -> V fragment of that half of tile j (PV).
        constexpr int NP = 4 * NB;
        constexpr int PF64 = 4;
        // softmax work: 8 * RB units per half-phase spread over its 2 * NB * RB MFMA slots: a unit every SPU slots
        // (exp2 in its first slot, pack in its middle slot), or several units per slot when there are fewer slots
        constexpr int SLOTS = 2 * NB * RB;
        constexpr int UNITS = 8 * RB;
        bf16x8 fr[NP];
        auto fetch = [&](int i) {
          const int hs = i / (2 * NB), q = (i % (2 * NB)) / 2;
          fr[i] = (i & 1) ? vfrag(hs, q) : kfrag(hs, q);
        };
#pragma unroll
        for (int i = 0; i < PF64; ++i) fetch(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          if (i + PF64 < NP) fetch(i + PF64);
          const int hs = i / (2 * NB), q = (i % (2 * NB)) / 2;
          const int hs_u = i < 2 * NB ? 1 : 0, kt_u = i < 2 * NB ? j : j + 1;
          // margin before the first read of the chains that just ended (operands tie the reads behind it)
          if (i == 2 * NB) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) asm volatile("s_nop 7" : "+v"(sacc[0][rb]));
          }
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            if (i & 1) {
              const int jj = q / DT, dt = q % DT;
              oacc[rb][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], pfrag(hs, rb, jj), oacc[rb][dt], 0, 0, 0);
            } else {
              sacc[hs][rb] = q == 0 ? score_mfma0(fr[i], qf[rb][q]) : score_mfma(fr[i], qf[rb][q], sacc[hs][rb]);
            }
            const int slot = (i % (2 * NB)) * RB + rb;  // 0 .. SLOTS-1 within the half-phase
            if (SLOTS >= 2 * UNITS) {
              constexpr int SPU = SLOTS / UNITS;
              const int x = slot / SPU;
              if (slot % SPU == 0) unit_exp(hs_u, x / 8, x % 8, kt_u, MASK);
              if (slot % SPU == SPU / 2) unit_pack(hs_u, x / 8, x % 8);
            } else {
              constexpr int UPS = UNITS / SLOTS;
#pragma unroll
              for (int n = 0; n < UPS; ++n) {
                const int x = slot * UPS + n;
                unit_exp(hs_u, x / 8, x % 8, kt_u, MASK);
                unit_pack(hs_u, x / 8, x % 8);
              }
            }
            if (i == 1 && rb == RB - 1) {
              mem_store();
              mem_load();
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else if (KIND == IT_PRO) {  // j = -1: scores of tile 0 (both halves), probabilities of its half 0
        mem_store();
        mem_load();
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
          for (int hs = 0; hs < 2; ++hs) {
            const bf16x8 kf = kfrag(hs, kk);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              sacc[hs][rb] = kk == 0 ? score_mfma0(kf, qf[rb][kk]) : score_mfma(kf, qf[rb][kk], sacc[hs][rb]);
          }
        for (int rb = 0; rb < RB; ++rb) score_mfma_settle(sacc[0][rb], sacc[1][rb]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            unit_exp(0, rb, u, 0, MASK);
            unit_pack(0, rb, u);
          }
      } else if (KIND == IT_FINAL) {  // j = my_tiles - 1: no further scores
        mem_store();
        mem_load();
        for (int rb = 0; rb < RB; ++rb) score_mfma_settle(sacc[0][rb], sacc[1][rb]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            unit_exp(1, rb, u, j, MASK);
            unit_pack(1, rb, u);
          }
#pragma unroll
        for (int hs = 0; hs < 2; ++hs)
#pragma unroll
          for (int p = 0; p < 2 * DT; ++p) {
            const bf16x8 vf = vfrag(hs, p);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              oacc[rb][p % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pfrag(hs, rb, p / DT), oacc[rb][p % DT], 0, 0, 0);
          }
      } else {
        mem_store();
        mem_load();
      }
      lds_barrier();
    };
    using PRO_ = std::integral_constant<int, IT_PRO>;
    using FULL_ = std::integral_constant<int, IT_FULL>;
    using FINAL_ = std::integral_constant<int, IT_FINAL>;
    using IDLE_ = std::integral_constant<int, IT_IDLE>;
    using T_ = std::true_type;
    using F_ = std::false_type;

    load_rows(Kg, 0, rk);
    store_k(0);
    load_rows(Kg, min(1, ntiles - 1), rk);
    load_rows(Vg, 0, rv);
    lds_barrier();
    int j = -1;
    if (my_tiles > 0) {
      if (my_tiles == 1) iter(-1, PRO_{}, T_{});
      else iter(-1, PRO_{}, F_{});
      for (j = 0; j < my_tiles - 2; ++j) iter(j, FULL_{}, F_{});
      if (my_tiles >= 2) iter(my_tiles - 2, FULL_{}, T_{});
      iter(my_tiles - 1, FINAL_{}, T_{});
      j = my_tiles;
    }
    for (; j < ntiles; ++j) iter(j, IDLE_{}, F_{});

    // ---- epilogue: normalise, round once to bf16, store; log-sum-exp of the scaled logits (scores un-shifted)
    if (wave_live) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        store_rows<DH>(oacc[rb], both_halves(l_run[rb] + l_run2[rb]), 0.f, O, OLO, LSE, b, h, qw0 + rb * 32 + l32, T, Hq, half);
    }
  }
}

// d_h = 256: 256 threads, one wavefront per SIMD, 128 query rows per workgroup.
template <int DH, bool CAUSAL, bool RSUM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_fwd_wide_kernel(
    const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K, const bf16_t *__restrict__ V, bf16_t *__restrict__ O,
    bf16_t *__restrict__ OLO, float *__restrict__ LSE, const float *__restrict__ temp, int qk_normed, int T, int Hq,
    int Hk, int BH, int nqb, int paired, float scale) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BKV * (DH * 2 + 16) + 2 * BKV * (DH * 2 + 64)];
  float bound = INFINITY;
  if (qk_normed) {  // |q.k| <= d_h * beta; 2 % head-room for the bf16 rounding of the stored q and k
    const int g = ((int)blockIdx.x % BH % Hq) / (Hq / Hk);
    const float beta = temp ? expf(temp[g]) : 1.f;
    bound = 1.02f * (float)DH * beta * scale * 1.44269504088896340736f;
  }
  if (bound <= 60.f)
    attn_fwd_pipelined_wide<DH, CAUSAL, RSUM, 1>(Q, K, V, O, OLO, LSE, T, Hq, Hk, BH, nqb, paired, scale, smem);
  else
    attn_fwd_body<DH, CAUSAL, false, RSUM, 256>(Q, K, V, O, OLO, LSE, T, Hq, Hk, BH, nqb, paired, scale, 0.f, smem);
}

// RSUM: the row sum adds the bf16-rounded probabilities, so that o is the exact convex combination the PV
// product formed; chosen when the caller saves lse / o_lo for a backward pass (see the file header).
// KS: key groups per workgroup (attn_fwd_body)
template <int DH, bool CAUSAL, bool RSUM, int KS, int NTH>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(NTH / 256, NTH / 256))) void attn_fwd_kernel(
    const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K, const bf16_t *__restrict__ V, bf16_t *__restrict__ O,
    bf16_t *__restrict__ OLO, float *__restrict__ LSE, const float *__restrict__ temp, int qk_normed, int T, int Hq, int Hk, int BH, int nqb,
    int paired, float scale) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[KS * 2 * BKV * (DH * 2 + 16 + DH * 2 + 64)];
  float bound = INFINITY;
  if (qk_normed) {
    // |q.k| <= d_h * beta; 2 % head-room for the bf16 rounding of the stored q and k
    const int g = ((int)blockIdx.x % BH % Hq) / (Hq / Hk);
    const float beta = temp ? expf(temp[g]) : 1.f;
    bound = 1.02f * (float)DH * beta * scale * 1.44269504088896340736f;
  }
  // exp2 arguments reach -2*bound: keep them inside the fp32 exponent range
  if (bound <= 60.f)
    attn_fwd_pipelined<DH, CAUSAL, RSUM, KS, NTH>(Q, K, V, O, OLO, LSE, T, Hq, Hk, BH, nqb, paired, scale, bound, smem);
  else
    attn_fwd_body<DH, CAUSAL, false, RSUM, NTH, KS>(Q, K, V, O, OLO, LSE, T, Hq, Hk, BH, nqb, paired, scale, 0.f, smem);
}

template <int DH, int KS, int NTH>
hipError_t launch(const Dims &d, const void *q, const void *k, const void *v, void *o, void *o_lo, float *lse,
                  const float *temp, hipStream_t s) {
  constexpr bool WIDE = DH > 128;             // one wavefront per SIMD, 128-row query blocks
  constexpr int BQL = WIDE ? 128 : NTH / 2 / KS;
  const int nqb = row_blocks(d.T, BQL);
  const int BH = d.B * d.Hq;
  const bool causal = d.flags & CCA_CAUSAL;
  const int paired = pair_blocks(BH, causal, nqb) ? 1 : 0;
  const long long blocks = (long long)BH * (paired ? (nqb + 1) / 2 : nqb);
  const int qk_normed = (d.flags & CCA_QK_NORM) ? 1 : 0;
  if (!(d.flags & CCA_KEY_TEMP)) temp = nullptr;
  const bool rsum = lse != nullptr || o_lo != nullptr;
#define CCA_ATTN_LAUNCH(C, R)                                                                                          \
  if constexpr (WIDE)                                                                                                  \
    attn_fwd_wide_kernel<DH, C, R><<<(unsigned)blocks, 256, 0, s>>>((const bf16_t *)q, (const bf16_t *)k,               \
                                                                    (const bf16_t *)v, (bf16_t *)o, (bf16_t *)o_lo, lse, \
                                                                    temp, qk_normed, d.T, d.Hq, d.Hk, BH, nqb, paired,  \
                                                                    d.scale);                                          \
  else                                                                                                                 \
    attn_fwd_kernel<DH, C, R, KS, NTH><<<(unsigned)blocks, NTH, 0, s>>>((const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v,  \
                                                              (bf16_t *)o, (bf16_t *)o_lo, lse, temp, qk_normed, d.T,   \
                                                              d.Hq, d.Hk, BH, nqb, paired, d.scale)
  if (causal) {
    if (rsum) { CCA_ATTN_LAUNCH(true, true); }
    else { CCA_ATTN_LAUNCH(true, false); }
  } else {
    if (rsum) { CCA_ATTN_LAUNCH(false, true); }
    else { CCA_ATTN_LAUNCH(false, false); }
  }
#undef CCA_ATTN_LAUNCH
  return hipGetLastError();
}

}  // namespace

bool attention_mfma_supported(const Dims &d) {
  return d.bf16 && (d.dh == 256 || d.dh == 128 || d.dh == 64) && (long long)d.B * d.Hq * ((d.T + 127) / 128) < (1ll << 31) &&
         (long long)d.T * d.Hk * d.dh * 2 < (1ll << 31);
}

hipError_t attention_mfma_bf16(const Dims &d, const void *q, const void *k, const void *v, void *o, void *o_lo,
                               float *lse, const float *temp, hipStream_t s) {
  const long long BH = (long long)d.B * d.Hq;
  const bool causal = d.flags & CCA_CAUSAL;
#define ARGS d, q, k, v, o, o_lo, lse, temp, s
  if (d.dh == 256) return launch<256, 1, 256>(ARGS);
  if (!fwd_splits_keys(BH, d.T, causal)) return d.dh == 128 ? launch<128, 1, 512>(ARGS) : launch<64, 1, 512>(ARGS);
  if (fwd_takes_64_rows(BH, d.T, d.flags & CCA_QK_NORM)) return d.dh == 128 ? launch<128, 2, 256>(ARGS) : launch<64, 2, 256>(ARGS);
  return d.dh == 128 ? launch<128, 2, 512>(ARGS) : launch<64, 2, 512>(ARGS);
#undef ARGS
}

}  // namespace cca
