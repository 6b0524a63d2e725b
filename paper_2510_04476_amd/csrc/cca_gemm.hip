// bf16 GEMM on the gfx950 matrix cores for the down- and up-projection
// (Sec. 2.2: down-projection equation and last line of the final equation
// block):  C (M,N) = A (M,K) * Bt (N,K)^T, fp32 accumulation, bf16 output.
//
// Both operands are K-contiguous, so a lane's 8-element MFMA fragment is one
// 16-byte LDS read.  Workgroup tile TM x BN x 64 with 8 wavefronts; LDS is
// XOR-swizzled per 16-byte chunk; K-slabs travel HBM -> LDS directly
// (buffer_load ... lds, no staging registers, no ds_write), A two slabs ahead and the
// weight one, the loads and the next k-step's fragment reads dealt out between a
// slab's MFMAs.  The MFMA is issued with the weight rows as its first operand,
// which leaves every lane with 4 consecutive output columns of one row, so
// the epilogue packs them to bf16, stages the tile in LDS and writes whole
// rows with 16-byte stores.
#include <type_traits>

#include "cca_internal.h"
#include "cca_transpose.h"

namespace cca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int BM = 256, BK = 64;
constexpr int A_STAGES = 3, B_STAGES = 2;  // slabs of each operand in the LDS of the 256-row product
constexpr int PAUSE = 24;  // of 64 clocks each: 0.7 us (start_pauses)

// LDS position of the 16-byte chunk c (0..7) of row r in a [rows][64] bf16 tile
__device__ __forceinline__ int swz(int r, int c) { return r * 8 + (c ^ ((r & 7) ^ ((r >> 3) & 1))); }

// two floats -> one word of two bf16 (round to nearest even) with the hardware conversion instruction
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// The workgroups of a small tile may split the contraction over WAVES_K groups of wavefronts: the sums of groups 1, 2, ...
// are added to group 0's through LDS, in order.  The tiles are no longer read when this is called.
template <int WAVES_MN, int WAVES_K, int NI, int MI>
__device__ __forceinline__ void add_wave_parts(f32x16 (&acc)[NI][MI], unsigned char *smem, int wk, int wmn, int lane) {
  if constexpr (WAVES_K > 1) {
    constexpr int PER_LANE = MI * NI * 16, PART = WAVES_MN * PER_LANE * 64;
    float *sp = reinterpret_cast<float *>(smem) + (size_t)wmn * (PER_LANE * 64) + lane;
    if (wk > 0) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int r = 0; r < 16; ++r) sp[(wk - 1) * PART + ((ni * MI + mi) * 16 + r) * 64] = acc[ni][mi][r];
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int g = 0; g < WAVES_K - 1; ++g)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ni][mi][r] += sp[g * PART + ((ni * MI + mi) * 16 + r) * 64];
    }
    __syncthreads();
  }
}

// Tile (row tm, column tn) of workgroup wg; false: none.  Workgroups are dealt round-robin over the 8 XCDs, each with an L2 of its own, so
// every XCD gets a contiguous range of tiles; the order runs down panels of `panel` columns of tiles (tile_panel).  `pauses`: slabs behind
// which a workgroup of the large products pauses (start_pauses).
struct TileGrid {
  int tiles_n, tiles, panel, pauses;
};
__device__ __forceinline__ bool tile_of(const TileGrid &g, int wg, int &tm, int &tn) {
  const int tile = (wg % 8) * ((g.tiles + 7) / 8) + wg / 8;
  if (tile >= g.tiles) return false;
  const int full = g.panel * (g.tiles / g.tiles_n), p = tile / full, r = tile - p * full, width = min(g.panel, g.tiles_n - p * g.panel);
  tm = r / width;
  tn = p * g.panel + r - tm * width;
  return true;
}
TileGrid tile_grid(long long M, int N, long long K, int tm, int tn) {
  const int tiles_m = (int)((M + tm - 1) / tm), tiles_n = (N + tn - 1) / tn;
  const int tiles = tiles_m * tiles_n;
  return TileGrid{tiles_n, tiles, tile_panel(tiles_m, tiles_n, tm, tn, K), start_pauses(tm * tn, tiles, K / BK)};
}

// Products of F x F blocks (F = 32 or 16): acc[ni][mi][r] = C[m][n] with m = (wm*MI + mi)*F + lane%F and n = (wn*NI + ni)*F + 8*(r/4) +
// 4*(lane/F) + r%4 of the tile at (m0, n0): packed to bf16, staged in LDS and written as whole rows.  `owner`: this wavefront holds
// sums to store.
template <int TM, int TN, int NTHREADS, int NI, int MI, typename Acc>
__device__ __forceinline__ void store_tile_bf16(const Acc (&acc)[NI][MI], unsigned char *smem, bool owner, int wm, int wn,
                                                int tid, bf16_t *__restrict__ C, long long m0, long long M, int n0, int N,
                                                const ColumnSplit &split = ColumnSplit{}) {
  constexpr int ROW_BYTES = TN * 2 + 16;  // padded row: 8-byte column writes of 32 rows hit distinct banks
  constexpr int F = sizeof(Acc) == 64 ? 32 : 16;
  const int row = tid & (F - 1), group = (tid & 63) / F;
  if (owner) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        const int m = (wm * MI + mi) * F + row;
#pragma unroll
        for (int rg = 0; rg < F * F / 256; ++rg) {
          const int n = (wn * NI + ni) * F + rg * 8 + group * 4;
          u32x2 p;
          p.x = pack_bf16x2(acc[ni][mi][rg * 4 + 0], acc[ni][mi][rg * 4 + 1]);
          p.y = pack_bf16x2(acc[ni][mi][rg * 4 + 2], acc[ni][mi][rg * 4 + 3]);
          *reinterpret_cast<u32x2 *>(smem + m * ROW_BYTES + n * 2) = p;
        }
      }
  }
  __syncthreads();
  constexpr int CH_ROW = TN / 8;  // 16-byte chunks per tile row
  for (int id = tid; id < TM * CH_ROW; id += NTHREADS) {
    const int r = id / CH_ROW, c = id % CH_ROW;
    const long long gm = m0 + r;
    const int gn = n0 + c * 8;
    if (gm >= M || gn >= N) continue;
    const u32x4 val = *reinterpret_cast<const u32x4 *>(smem + r * ROW_BYTES + c * 16);
    if (C) *reinterpret_cast<u32x4 *>(C + gm * N + gn) = val;
    if (split.q) {
      const int ek = gn - split.e_q, ev = ek - split.e_kv;
      bf16_t *const to = ek < 0 ? (bf16_t *)split.q + gm * split.e_q + gn
                                : (ev < 0 ? (bf16_t *)split.k + gm * split.e_kv + ek : (bf16_t *)split.v + gm * split.e_kv + ev);
      *reinterpret_cast<u32x4 *>(to) = val;
    }
  }
}

// LDS holds three slabs of A and two of Bt: A streams from HBM, whose latency a slab's 1.1-1.5 us of MFMAs do not cover; Bt is
// a weight that stays in the caches, and a third stage of it would not fit (256 x 256: 3 x 32 + 2 x 32 KB, all of a CU's LDS).
// A slab's one barrier stands near the end of its first k-step, when the fragments of the last are in registers: from there on the
// slab's buffers are free for the next loads, and the next slab's first fragments are read under the last step's MFMAs.
// Every fragment read and every load stands between two MFMAs of its own, in the order of use, so the matrix core never waits behind a
// burst of them; scheduling barriers keep the order.  The loop has no branch and no scalar load in flight: either makes the
// compiler wait for the fragments just requested instead of those it needs.  Random operands, us, a k-step's reads in a burst, loads into
// LDS counted among them and 32x32x16 instructions -> this: 16384 x 1536 x 2048 101.4 -> 86.2, 4096 x 6144 x 2048 99.7 -> 82.7, 7996 x 2048
// x 1024 37.1 -> 30.6, 6000 x 1536 x 2048 45.5 -> 35.6, 8192 x 8192 x 8192 955 -> 732.
// What bounds it: the power the matrix cores draw (8192^3 on all-zero operands: 607 us).  16x16x32 instructions draw less than
// 32x32x16 ones on the same fragments: 8192^3 877 -> 796 us on random operands, 601 -> 607 on zeros.
// A large grid's workgroups pause between their first slabs (start_pauses): what all CUs draw at once would cost the kernels around it
// their clock.
// Not faster: s_setprio around the MFMAs, any other order of them, the barrier four MFMAs earlier, A's loads closer
// together or further apart, 4 wavefronts of 128 x 128 (half the fragment reads).  Rows and columns of the tile: what deals the tiles most
// evenly to 256 CUs (nt_tile).
template <int TM, int BN, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64) void gemm_bf16_nt_kernel(const bf16_t *__restrict__ A,
                                                               const bf16_t *__restrict__ Bt,
                                                               bf16_t *__restrict__ C, long long M, int N, int K,
                                                               TileGrid grid, ColumnSplit split) {
  // the epilogue's arguments are loaded here
  asm volatile("" : "+s"(C), "+s"(split.q), "+s"(split.k), "+s"(split.v), "+s"(split.e_q), "+s"(split.e_kv));
  constexpr int NWAVES = WAVES_M * WAVES_N, NTHREADS = NWAVES * 64;
  constexpr int WM = TM / WAVES_M, WN = BN / WAVES_N;  // wave tile
  constexpr int MI = WM / 16, NI = WN / 16;            // 16x16 MFMA tiles per wave
  static_assert(MI * 16 == WM && NI * 16 == WN, "wave tile must be a multiple of 16");
  static_assert(BK == 64, "two k-steps of 32");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int A_STAGE = TM * 8, B_STAGE = BN * 8;  // 16-byte chunks of a slab
  u32x4 *const sA = reinterpret_cast<u32x4 *>(smem), *const sB = sA + A_STAGES * A_STAGE;

  int tm, tn;
  if (!tile_of(grid, blockIdx.x, tm, tn)) return;
  const long long m0 = (long long)tm * TM;
  const int n0 = tn * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, first_wave = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int row = lane & 15, quad = lane >> 4;

  // Direct loads to LDS: wave instruction i deposits 64 x 16 bytes at LDS chunks [i*64, i*64+64) of a slab
  // (8 chunks per row), so lane L fetches the chunk that the XOR swizzle puts at that position.  Rows past the end of the
  // matrix are its last one.
  constexpr int A_LOADS = A_STAGE / 64 / NWAVES, B_LOADS = B_STAGE / 64 / NWAVES;  // instructions of a wavefront per slab
  static_assert(A_LOADS * 64 * NWAVES == A_STAGE && B_LOADS * 64 * NWAVES == B_STAGE,
                "instructions must divide evenly over the wavefronts");
  const int a_rows = (int)(M - m0 < TM ? M - m0 : TM), b_rows = N - n0 < BN ? N - n0 : BN;
  const int l_row = (wave * 64 + lane) >> 3, l_cs = lane & 7;  // row and chunk position of this thread's first chunk
  unsigned a_off[A_LOADS], b_off[B_LOADS];  // bytes from the tile's first row (256 rows of K: below 2^31, gemm_mfma_supported)
#pragma unroll
  for (int u = 0; u < A_LOADS; ++u) {
    const int r = l_row + u * (NTHREADS / 8), c = l_cs ^ ((r & 7) ^ ((r >> 3) & 1));  // inverse of swz()
    a_off[u] = (unsigned)(r < a_rows ? r : a_rows - 1) * K * 2 + c * 16;
  }
#pragma unroll
  for (int u = 0; u < B_LOADS; ++u) {
    const int r = l_row + u * (NTHREADS / 8), c = l_cs ^ ((r & 7) ^ ((r >> 3) & 1));
    b_off[u] = (unsigned)(r < b_rows ? r : b_rows - 1) * K * 2 + c * 16;
  }
  const bf16_t *const a_base = A + m0 * K, *const b_base = Bt + (long long)n0 * K;
  auto load_a = [&](int kt, int stage, int u) __attribute__((always_inline)) {
    load_to_lds(a_base, (unsigned)a_rows * K * 2, a_off[u], kt * (BK * 2), sA + stage * A_STAGE + (first_wave + u * NWAVES) * 64);
  };
  auto load_b = [&](int kt, int stage, int u) __attribute__((always_inline)) {
    load_to_lds(b_base, (unsigned)b_rows * K * 2, b_off[u], kt * (BK * 2), sB + stage * B_STAGE + (first_wave + u * NWAVES) * 64);
  };

  f32x4 acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[ni][mi][r] = 0.f;
  // two sets of fragments, one for each k-step: set s ^ 1 is read between the MFMAs of set s, in the order they need it
  bf16x8 fa[2][MI], fb[2][NI];
  constexpr int READS = MI + NI, MFMAS = MI * NI, PER_READ = MFMAS / READS;
  static_assert(PER_READ >= 1, "a read behind every PER_READ-th MFMA");
  auto read = [&](int a_stage, int b_stage, int set, int j) __attribute__((always_inline)) {
    if (j >= 1 && j <= MI)
      fa[set][j - 1] = __builtin_bit_cast(bf16x8, sA[a_stage * A_STAGE + swz(wm * WM + (j - 1) * 16 + row, set * 4 + quad)]);
    else
      fb[set][j ? j - MI : 0] = __builtin_bit_cast(bf16x8, sB[b_stage * B_STAGE + swz(wn * WN + (j ? j - MI : 0) * 16 + row, set * 4 + quad)]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int set, int i) __attribute__((always_inline)) {
    const int ni = i / MI, mi = i % MI;
    acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][ni], fa[set][mi], acc[ni][mi], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  const int nk = K / BK;
#pragma unroll
  for (int u = 0; u < B_LOADS; ++u) load_b(0, 0, u);
#pragma unroll
  for (int u = 0; u < A_LOADS; ++u) load_a(0, 0, u);
  if (nk > 1) {
#pragma unroll
    for (int u = 0; u < B_LOADS; ++u) load_b(1, 1, u);
#pragma unroll
    for (int u = 0; u < A_LOADS; ++u) load_a(1, 1, u);
    __builtin_amdgcn_s_waitcnt(wait_vm(A_LOADS + B_LOADS));
  } else {
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < READS; ++j) read(0, 0, 0, j);
  __builtin_amdgcn_s_waitcnt(WAIT_LDS);

  int as = 0;  // stage of A that holds slab kt
  // `next`: there is a slab kt + 1, `ahead`: and a slab kt + 2
  auto slab = [&](int kt, auto ahead_, auto next_) __attribute__((always_inline)) {
    constexpr bool ahead = decltype(ahead_)::value, next = decltype(next_)::value;
    constexpr int A_EVERY = 2 * A_LOADS <= MFMAS - 4 ? 2 : 1, B_EVERY = 2 * B_LOADS <= MFMAS ? 2 : 1;
    const int bs = kt & 1, as1 = as == 2 ? 0 : as + 1, as2 = as1 == 2 ? 0 : as1 + 1;
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
      multiply(0, i);
      if (i % PER_READ == 0 && i / PER_READ < READS) read(as, bs, 1, i / PER_READ);
      if (ahead && i % A_EVERY == A_EVERY - 1 && i / A_EVERY < A_LOADS) load_a(kt + 2, as2, i / A_EVERY);  // into the stage of slab kt - 1
    }
    if (next) {
      // slab kt + 1 has landed when no more than the newest loads, A of slab kt + 2, are outstanding
      __builtin_amdgcn_s_waitcnt(wait_vm(ahead ? A_LOADS : 0) & WAIT_LDS_TOO);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
      multiply(1, i);
      if (next && i % PER_READ == 0 && i / PER_READ < READS) read(as1, bs ^ 1, 0, i / PER_READ);
      if (ahead && i % B_EVERY == B_EVERY - 1 && i / B_EVERY < B_LOADS) load_b(kt + 2, bs, i / B_EVERY);  // every wavefront holds its last fragments of slab kt
    }
    as = as1;
  };
  int kt = 0;
  for (; kt < grid.pauses && kt + 2 < nk; ++kt) {
    slab(kt, std::true_type{}, std::true_type{});
    __builtin_amdgcn_s_sleep(PAUSE);
  }
  for (; kt + 2 < nk; ++kt) slab(kt, std::true_type{}, std::true_type{});
  if (kt + 1 < nk) slab(kt++, std::false_type{}, std::true_type{});
  slab(kt, std::false_type{}, std::false_type{});
  __syncthreads();
  store_tile_bf16<TM, BN, NTHREADS>(acc, smem, true, wm, wn, tid, C, m0, M, n0, N, split);
}

__global__ __launch_bounds__(256) void transpose_bf16_kernel(TransposePair p) {
  __shared__ TransposeTile tile;
  transpose_block(p, blockIdx.x, tile);
}

// ---------------------------------------------------------------------------
// Weight-gradient GEMM (adjoint of the two projections): C (Mo,No) = A (K,Mo)^T * B (K,No), contraction over
// the B*T token rows.  Both operands are row-major with the contraction index as the ROW, so the tiles are
// staged row-major in LDS and the MFMA fragments (8 values along K for one column) come from the transposing
// LDS read.  The output is small (a weight matrix) and K is long, so K is split over `gridDim.y` workgroups
// that write fp32 partial sums; a second kernel adds them in a fixed order and rounds to bf16.
// ---------------------------------------------------------------------------
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

constexpr int TN_BN = 256;  // tile width (both operands)

// MFMA fragment of 16 columns of a [64 tokens][256 columns] bf16 tile: lane (column lane & 15, quad = lane / 16) receives tokens 4*quad +
// 0..3 and 16 + 4*quad + 0..3 behind `base`, which holds the lane's address for the first 16 columns of the tile: token 4*quad +
// (lane & 15)/4, 8 bytes of the 32 that four lanes share.  Chunk c of token r lies at position c ^ ((r & 7) << 1), so that the 32 bytes
// that 8 tokens of one read touch fall in 8 different bank groups; the columns are 32 bytes apart in the same low bits.
__device__ __forceinline__ bf16x8 tr_frag_tn(const unsigned char *tile, unsigned lane_off, int column16) {
  const unsigned char *p = tile + (lane_off ^ (unsigned)(column16 * 32));
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)p);
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(p + 16 * 512));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The pipeline of gemm_bf16_nt_kernel (slabs of 64 tokens, three of A and two of B in LDS, reads and loads between the MFMAs) on operands
// whose rows are the contraction index; bound by the matrix cores' power and, with more than one split, by the partial sums (written and
// read at about 7 TB/s).  With register staging, padded rows and a k-step's fragments read in a burst -> this, reduction included, us (columns x
// columns over tokens): 2048 x 1536 over 7996 69.3 -> 57.5, over 16384 117.9 -> 94.3; 1024 x 2048 over 7996 52.7 -> 45.3, over 16384 82.6 ->
// 69.9; 2048 x 6144 over 4096 (one split) 138.7 -> 95.2.
__device__ __forceinline__ void gemm_bf16_tn_body(const bf16_t *__restrict__ A, long long lda, const bf16_t *__restrict__ Bm, long long ldb,
                                                  float *__restrict__ part, bf16_t *__restrict__ C, int Mo, int No, long long K,
                                                  int tiles_n, int tiles_total, int splits, int slabs_per_split,
                                                  unsigned char *__restrict__ smem) {
  constexpr int NWAVES = 8, WAVES_N = 4;
  constexpr int WM = BM / 2, WN = TN_BN / WAVES_N;  // 128 x 64 wave tile
  constexpr int MI = WM / 16, NI = WN / 16;
  constexpr int STAGE = BK * 256 * 2;            // bytes of a slab of either operand
  constexpr int LOADS = STAGE / 1024 / NWAVES;   // load instructions of a wavefront per operand and slab, two tokens each
  unsigned char *const sA = smem, *const sB = smem + A_STAGES * STAGE;

  // Units (split, tile) in split order, a contiguous range of them to each XCD: the tiles of a split read the same token rows,
  // so an XCD's L2 is filled with its share of A and B instead of all of both, and every XCD gets the same number of units
  // (1024 x 2048 over 16384 tokens, 8 splits: 85.4 -> 82.5 us; 36 tiles x 7 splits over 12000 tokens, five tiles to an XCD and
  // so two rounds before: 116 -> 75).
  const int units = tiles_total * splits, per_xcd = (units + 7) / 8, unit = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (unit >= units) return;
  const int split = unit / tiles_total, tile = unit % tiles_total;
  const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * TN_BN;
  const long long nk_all = (K + BK - 1) / BK;
  const long long slab0 = (long long)split * slabs_per_split;
  const int nk = (int)((slab0 + slabs_per_split <= nk_all ? slabs_per_split : nk_all - slab0));  // at least 1 (tn_splits)

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, first_wave = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  // Load instruction i deposits tokens 2i, 2i + 1 of a slab; a lane fetches the chunk that the swizzle puts at its position (its token
  // modulo 8 is the same in every load of a wavefront).  Each load has a descriptor of its own that begins with the wavefronts' first
  // token and ends with the last one there is: tokens past it read as zeros.  Columns past the matrix edge are some others' (they only feed
  // outputs that are never stored).
  const int l_row = wave * 2 + (lane >> 5), l_chunk = (lane & 31) ^ ((l_row & 7) << 1);
  const unsigned a_off = (unsigned)(l_row * lda * 2) + l_chunk * 16, b_off = (unsigned)(l_row * ldb * 2) + l_chunk * 16;
  const int tokens = (int)(K - slab0 * BK < (long long)nk * BK ? K - slab0 * BK : (long long)nk * BK);
  const bf16_t *const a_first = A + slab0 * BK * lda + m0, *const b_first = Bm + slab0 * BK * ldb + n0;
  const int a_width = min(Mo - m0, 256), b_width = min(No - n0, 256);
  auto load = [&](const bf16_t *first, int ld, int width, int kt, int u, unsigned off, unsigned char *to) __attribute__((always_inline)) {
    const int token = kt * BK + u * 2 * NWAVES, rows = min(tokens - token, 2 * NWAVES);  // (none left: no bytes, width <= ld)
    load_to_lds(first + (long long)token * ld, (unsigned)max(((rows - 1) * ld + width) * 2, 0), off, 0, to + (first_wave + u * NWAVES) * 1024);
  };
  auto load_a = [&](int kt, int stage, int u) __attribute__((always_inline)) { load(a_first, (int)lda, a_width, kt, u, a_off, sA + stage * STAGE); };
  auto load_b = [&](int kt, int stage, int u) __attribute__((always_inline)) { load(b_first, (int)ldb, b_width, kt, u, b_off, sB + stage * STAGE); };

  f32x4 acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[ni][mi][r] = 0.f;

  const int quad = lane >> 4, t_row = 4 * quad + ((lane & 15) >> 2);  // the lane's token of a transposing read
  const unsigned lane_off = t_row * 512 + (((t_row & 7) << 1) ^ ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
  const unsigned a_lane = lane_off ^ (wm * MI * 32u), b_lane = lane_off ^ (wn * NI * 32u);
  bf16x8 fa[2][MI], fb[2][NI];
  constexpr int READS = MI + NI, MFMAS = MI * NI, PER_READ = MFMAS / READS;
  auto read = [&](int a_stage, int b_stage, int set, int j) __attribute__((always_inline)) {
    if (j >= 1 && j <= MI) fa[set][j - 1] = tr_frag_tn(sA + a_stage * STAGE + set * 32 * 512, a_lane, j - 1);
    else fb[set][j ? j - MI : 0] = tr_frag_tn(sB + b_stage * STAGE + set * 32 * 512, b_lane, j ? j - MI : 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int set, int i) __attribute__((always_inline)) {
    const int ni = i / MI, mi = i % MI;
    acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][ni], fa[set][mi], acc[ni][mi], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int u = 0; u < LOADS; ++u) load_b(0, 0, u);
#pragma unroll
  for (int u = 0; u < LOADS; ++u) load_a(0, 0, u);
  if (nk > 1) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) load_b(1, 1, u);
#pragma unroll
    for (int u = 0; u < LOADS; ++u) load_a(1, 1, u);
    __builtin_amdgcn_s_waitcnt(wait_vm(2 * LOADS));
  } else {
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < READS; ++j) read(0, 0, 0, j);
  __builtin_amdgcn_s_waitcnt(WAIT_LDS);

  int as = 0;  // stage of A that holds slab kt
  auto slab = [&](int kt, auto ahead_, auto next_) __attribute__((always_inline)) {  // as in gemm_bf16_nt_kernel
    constexpr bool ahead = decltype(ahead_)::value, next = decltype(next_)::value;
    const int bs = kt & 1, as1 = as == 2 ? 0 : as + 1, as2 = as1 == 2 ? 0 : as1 + 1;
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
      multiply(0, i);
      if (i % PER_READ == 0 && i / PER_READ < READS) read(as, bs, 1, i / PER_READ);
      if (ahead && i % 2 == 1 && i / 2 < LOADS) load_a(kt + 2, as2, i / 2);
    }
    if (next) {
      __builtin_amdgcn_s_waitcnt(wait_vm(ahead ? LOADS : 0) & WAIT_LDS_TOO);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
      multiply(1, i);
      if (next && i % PER_READ == 0 && i / PER_READ < READS) read(as1, bs ^ 1, 0, i / PER_READ);
      if (ahead && i % 2 == 1 && i / 2 < LOADS) load_b(kt + 2, bs, i / 2);
    }
    as = as1;
  };
  int kt = 0;
  for (; kt + 2 < nk; ++kt) slab(kt, std::true_type{}, std::true_type{});
  if (kt + 1 < nk) slab(kt++, std::false_type{}, std::true_type{});
  slab(kt, std::false_type{}, std::false_type{});

  if (splits == 1) {  // the result itself (2048 x 6144 over 4096 tokens, written as fp32 and read again: 105.4 us, 95.2)
    __syncthreads();
    store_tile_bf16<BM, TN_BN, 512>(acc, smem, true, wm, wn, tid, C, m0, Mo, n0, No);
    return;
  }
  // Partial sums leave as the lanes hold them, in 32 x 32 blocks of four 16 x 16 ones of [lane][r] (block (i, j) of a split at i *
  // blocks_n + j): 1 KB per store instruction, where rows of the matrix would be 64 bytes of 16 cache lines.
  const int blocks_m = (Mo + 31) / 32, blocks_n = (No + 31) / 32;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int bi = m0 / 32 + (wm * MI + mi) / 2, bj = n0 / 32 + (wn * NI + ni) / 2;
      if (bi >= blocks_m || bj >= blocks_n) continue;
      *reinterpret_cast<f32x4 *>(part + (((long long)split * blocks_m + bi) * blocks_n + bj) * 1024 + ((mi & 1) * 2 + (ni & 1)) * 256 + lane * 4) =
          acc[ni][mi];
    }
}

// (a body inlined with restrict arguments: without them the compiler makes every transposing LDS read wait for the loads
// into LDS in flight)
__global__ __launch_bounds__(512) void gemm_bf16_tn_kernel(const bf16_t *__restrict__ A, long long lda,
                                                          const bf16_t *__restrict__ Bm, long long ldb,
                                                          float *__restrict__ part, bf16_t *__restrict__ C, int Mo, int No, long long K,
                                                          int tiles_n, int tiles_total, int splits, int slabs_per_split) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  gemm_bf16_tn_body(A, lda, Bm, ldb, part, C, Mo, No, K, tiles_n, tiles_total, splits, slabs_per_split, smem);
}

// The weight-gradient product on smaller tiles, for token counts whose 256 x 256 tiles would have to be split many ways
// over K to fill the chip (2 x 512 tokens, 2048 x 1536: 50 MB of partial sums written and read back for 6 MB of result).
// One workgroup walks all of K, so the result is rounded and stored directly: no partial sums, no second kernel.  Tiles
// travel global -> LDS directly, STAGES - 1 slabs ahead; LDS rows are unpadded (a direct load fills 1 KB at a time), so
// the 64-byte column group a transposing read touches in 4 consecutive rows is XOR-swizzled into 4 different bank groups
// instead.  With WAVES_K = 2 each half of the wavefronts takes 32 of a slab's 64 tokens.
template <int W>
__device__ __forceinline__ int swz_tn(int r, int c) {  // 16-byte chunk c of token row r in a [tokens][W] tile
  return r * (W / 8) + (c ^ (W == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2));
}

template <int TM, int TN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES>
__device__ __forceinline__ void gemm_bf16_tn_deep_body(
    const bf16_t *__restrict__ A, long long lda, const bf16_t *__restrict__ Bm, long long ldb, bf16_t *__restrict__ C,
    int Mo, int No, long long K, const TileGrid &grid, int wg, unsigned char *smem) {
  static_assert((TM == 64 || TM == 128) && (TN == 64 || TN == 128), "swz_tn");
  constexpr int NWAVES = WAVES_M * WAVES_N * WAVES_K, NTHREADS = NWAVES * 64;
  constexpr int MI = TM / WAVES_M / 32, NI = TN / WAVES_N / 32;
  constexpr int A_CH = BK * TM / 8, STAGE = BK * (TM + TN) / 8;  // 16-byte chunks of the A part / of a stage
  constexpr int PER_WAVE = STAGE / 64 / NWAVES;
  static_assert(PER_WAVE * 64 * NWAVES == STAGE && A_CH % 64 == 0, "instructions must divide evenly over the wavefronts");
  u32x4 *const sbase = reinterpret_cast<u32x4 *>(smem);

  int tm, tn;
  if (!tile_of(grid, wg, tm, tn)) return;
  const int m0 = tm * TM, n0 = tn * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int wk = wave / (WAVES_M * WAVES_N), wmn = wave % (WAVES_M * WAVES_N), wm = wmn / WAVES_N, wn = wmn % WAVES_N;

  // Load instruction wave + u * NWAVES fills 64 chunks of the stage.  A slab is read through descriptors that begin at its first token and
  // end with the last one there is: tokens past it read as zeros.  Columns past the matrix edge are some others' (they only feed
  // outputs that are never stored).
  const int first_wave = __builtin_amdgcn_readfirstlane(wave);
  const int a_width = min(Mo - m0, TM), b_width = min(No - n0, TN);
  unsigned off[PER_WAVE];
#pragma unroll
  for (int u = 0; u < PER_WAVE; ++u) {
    const int i = first_wave + u * NWAVES, pos = i * 64 + lane;
    if (i < A_CH / 64) {
      const int r = pos / (TM / 8), c = (pos % (TM / 8)) ^ (TM == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2);
      off[u] = (unsigned)(r * lda + c * 8) * 2;
    } else {
      const int p = pos - A_CH, r = p / (TN / 8), c = (p % (TN / 8)) ^ (TN == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2);
      off[u] = (unsigned)(r * ldb + c * 8) * 2;
    }
  }
  auto issue = [&](long long kt, int buf) __attribute__((always_inline)) {
    const long long left = K - kt * BK;
    const int tokens = left < BK ? (int)left : BK;
    const unsigned a_bytes = ((tokens - 1) * (int)lda + a_width) * 2, b_bytes = ((tokens - 1) * (int)ldb + b_width) * 2;
    const bf16_t *const a_first = A + kt * BK * lda + m0, *const b_first = Bm + kt * BK * ldb + n0;
#pragma unroll
    for (int u = 0; u < PER_WAVE; ++u) {
      const int i = first_wave + u * NWAVES;
      load_to_lds(i < A_CH / 64 ? a_first : b_first, i < A_CH / 64 ? a_bytes : b_bytes, off[u], 0, sbase + buf * STAGE + i * 64);
    }
  };
  f32x16 acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ni][mi][r] = 0.f;

  // a lane's place in a transposing read: row 4*half + (lane & 15)/4 of each group of 8, 8 bytes of a 64-byte column group
  const int tr = 4 * half + ((lane & 15) >> 2), tc = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1), tb = (lane & 1) * 8;
  const int nk = (int)((K + BK - 1) / BK);
#pragma unroll
  for (int i = 0; i < STAGES - 1; ++i)
    if (i < nk) issue(i, i);
  int buf = 0;
  auto multiply = [&]() __attribute__((always_inline)) {  // the slab in stage `buf`
    const unsigned char *pa = smem + (size_t)buf * STAGE * 16, *pb = pa + A_CH * 16;
    constexpr int STEPS = BK / 16 / WAVES_K;
    bf16x8 fa[STEPS][MI], fb[STEPS][NI];
#pragma unroll
    for (int k2 = 0; k2 < STEPS; ++k2) {
      const int r0 = (wk * STEPS + k2) * 16 + tr;
      auto frag = [&](const unsigned char *base, auto width, int c0) {
        constexpr int W = decltype(width)::value;
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(base + swz_tn<W>(r0, c0 / 8 + tc) * 16 + tb));
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(base + swz_tn<W>(r0 + 8, c0 / 8 + tc) * 16 + tb));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) fa[k2][mi] = frag(pa, std::integral_constant<int, TM>{}, (wm * MI + mi) * 32);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fb[k2][ni] = frag(pb, std::integral_constant<int, TN>{}, (wn * NI + ni) * 32);
    }
    if constexpr (WAVES_K == 1) __builtin_amdgcn_sched_barrier(0);  // every fragment is requested before the first is used (1-2 % at 128 x 128)
#pragma unroll
    for (int k2 = 0; k2 < STEPS; ++k2)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
          acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[k2][ni], fa[k2][mi], acc[ni][mi], 0, 0, 0);
  };
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + STAGES - 1 <= nk) __builtin_amdgcn_s_waitcnt(wait_vm((STAGES - 2) * PER_WAVE) & WAIT_LDS_TOO);
    else __builtin_amdgcn_s_waitcnt(wait_vm(0) & WAIT_LDS_TOO);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1, buf == 0 ? STAGES - 1 : buf - 1);
    multiply();
    buf = buf == STAGES - 1 ? 0 : buf + 1;
  }
  __syncthreads();
  add_wave_parts<WAVES_M * WAVES_N, WAVES_K>(acc, smem, wk, wmn, lane);
  store_tile_bf16<TM, TN, NTHREADS>(acc, smem, wk == 0, wm, wn, tid, C, (long long)m0, (long long)Mo, n0, No);
}

// (a body inlined with restrict arguments: without them the compiler makes every transposing LDS read wait for the loads
// into LDS in flight)
template <int TM, int TN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES>
__global__ __launch_bounds__(WAVES_M *WAVES_N *WAVES_K * 64) void gemm_bf16_tn_deep_kernel(
    const bf16_t *__restrict__ A, long long lda, const bf16_t *__restrict__ Bm, long long ldb, bf16_t *__restrict__ C,
    int Mo, int No, long long K, TileGrid grid) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  gemm_bf16_tn_deep_body<TM, TN, WAVES_M, WAVES_N, WAVES_K, STAGES>(A, lda, Bm, ldb, C, Mo, No, K, grid, blockIdx.x, smem);
}

// LDS of a small-tile workgroup: its stages (`rows` rows of 64 values), then the wavefronts' sums and the tile on its way out
constexpr size_t deep_lds(int tm, int tn, int waves_k, int rows) {
  const size_t epi = (size_t)tm * (tn * 2 + 16), sum = (size_t)(waves_k - 1) * tm * tn * 4, main = (size_t)rows * BK * 2;
  const size_t most = main > epi ? main : epi;
  return most > sum ? most : sum;
}

template <int TM, int TN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES>
hipError_t launch_tn_deep(const void *A, long long lda, const void *Bm, long long ldb, void *C, int Mo, int No, long long K,
                          hipStream_t s) {
  const TileGrid grid = tile_grid(Mo, No, K, TM, TN);
  constexpr size_t smem = deep_lds(TM, TN, WAVES_K, STAGES * (TM + TN));
  constexpr auto kernel = gemm_bf16_tn_deep_kernel<TM, TN, WAVES_M, WAVES_N, WAVES_K, STAGES>;
  if (hipError_t e = raise_lds_limit<kernel>(smem); e != hipSuccess) return e;
  kernel<<<(grid.tiles + 7) / 8 * 8, WAVES_M * WAVES_N * WAVES_K * 64, smem, s>>>((const bf16_t *)A, lda, (const bf16_t *)Bm, ldb,
                                                                            (bf16_t *)C, Mo, No, K, grid);
  return hipGetLastError();
}

// C = bf16(sum over splits, in order).  Workgroup = 32 rows x 128 columns, a wavefront per 32 x 32 block of the partial sums;
// the rounded rows go through LDS so that they leave 256 bytes at a time.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ part, int splits, int Mo, int No,
                                                           bf16_t *__restrict__ C) {
  constexpr int ROW_BYTES = 128 * 2 + 16;
  __shared__ __attribute__((aligned(16))) unsigned char tile[32 * ROW_BYTES];
  const int blocks_m = (Mo + 31) / 32, blocks_n = (No + 31) / 32, strips = (blocks_n + 3) / 4;
  const int bi = blockIdx.x / strips, j0 = (blockIdx.x % strips) * 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (j0 + wave < blocks_n) {
    const float *p = part + ((long long)bi * blocks_n + j0 + wave) * 1024 + lane * 4;
    const long long step = (long long)blocks_m * blocks_n * 1024;
    f32x4 acc[4];
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) acc[rg] = *reinterpret_cast<const f32x4 *>(p + rg * 256);
    auto add = [&](int s, auto n_) __attribute__((always_inline)) {  // n splits' loads in flight
      constexpr int N = decltype(n_)::value;
      f32x4 v[N][4];
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) v[u][rg] = *reinterpret_cast<const f32x4 *>(p + (s + u) * step + rg * 256);
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[rg][e] += v[u][rg][e];
    };
    int s = 1;
    for (; s + 4 <= splits; s += 4) add(s, std::integral_constant<int, 4>{});
    for (; s < splits; ++s) add(s, std::integral_constant<int, 1>{});
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      u32x2 w;
      w.x = pack_bf16x2(acc[rg][0], acc[rg][1]);
      w.y = pack_bf16x2(acc[rg][2], acc[rg][3]);
      // (16 x 16 block rg of the 32 x 32: rows rg / 2, columns rg % 2)
      *reinterpret_cast<u32x2 *>(tile + (rg / 2 * 16 + (lane & 15)) * ROW_BYTES + (wave * 32 + rg % 2 * 16 + lane / 16 * 4) * 2) = w;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int id = tid + i * 256, r = id / 16, c = id % 16, m = bi * 32 + r, n = j0 * 32 + c * 8;
    if (m < Mo && n < No)  // No % 8 == 0
      *reinterpret_cast<u32x4 *>(C + (long long)m * No + n) = *reinterpret_cast<const u32x4 *>(tile + r * ROW_BYTES + c * 16);
  }
}

template <int TM, int BN, int WAVES_M, int WAVES_N>
hipError_t launch_gemm(const void *A, const void *Bt, void *C, long long M, int N, int K, const ColumnSplit &split,
                       hipStream_t s) {
  const TileGrid grid = tile_grid(M, N, K, TM, BN);
  constexpr size_t epi_bytes = (size_t)TM * (BN * 2 + 16);
  constexpr size_t main_bytes = (size_t)(A_STAGES * TM + B_STAGES * BN) * BK * 2;
  constexpr size_t smem = main_bytes > epi_bytes ? main_bytes : epi_bytes;
  static_assert(smem <= 160 * 1024, "LDS");
  if (hipError_t e = raise_lds_limit<gemm_bf16_nt_kernel<TM, BN, WAVES_M, WAVES_N>>(smem); e != hipSuccess) return e;
  gemm_bf16_nt_kernel<TM, BN, WAVES_M, WAVES_N><<<(grid.tiles + 7) / 8 * 8, WAVES_M * WAVES_N * 64, smem, s>>>((const bf16_t *)A, (const bf16_t *)Bt, (bf16_t *)C, M, N,
                                                             K, grid, split);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// The same product on smaller tiles, for row counts whose 256-row tiles leave the chip idle (one 256 x 192 tile walks
// K = 2048 in 39 us however few tiles there are).  What bounds a small product is the chain of slabs each workgroup
// walks, so: the tile is small enough that every CU gets one, the loads run STAGES - 1 slabs ahead (one bare barrier per
// slab, `s_waitcnt vmcnt` counting the later slabs' loads as still in flight), and with WAVES_K = 2 a slab is 128 wide
// and each half of it belongs to one half of the wavefronts, whose sums are added through LDS at the end - half as many
// steps in the chain.  Measured (M x N x K, us, 256-row tiles -> this): 512 x 1536 x 2048 39.4 -> 10.0 (64 x 64 tiles),
// 512 x 2048 x 1024 22.2 -> 7.8, 1000 x 1536 x 2048 39.5 -> 14.1 (64 x 128), 2000 x 1536 x 2048 39.9 -> 20.4
// (128 x 128); its loads as buffer loads (load_to_lds): 1000 x 1536 x 2048 14.2 -> 13.8, 2000 x 1536 x 2048 20.9 -> 19.6; likewise the weight
// gradients' small tiles: 2048 x 1536 over 1024 tokens 14.5 -> 12.9, 2048 x 2048 over 4000 48.1 -> 41.1.
// Slower everywhere: 16x16x32 instructions (twice as many for a chain that waits for LDS), more stages, 32-wide slabs (half the work per barrier), 128 x 192 and 256 x 128 tiles at two workgroups per CU,
// WAVES_K = 4.
// ---------------------------------------------------------------------------
template <int TM, int TN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES>
__device__ __forceinline__ void gemm_bf16_nt_deep_body(
    const bf16_t *__restrict__ A, const bf16_t *__restrict__ Bt, bf16_t *__restrict__ C, long long M, int N, int K,
    const TileGrid &grid, const ColumnSplit &split, int wg, unsigned char *smem) {
  constexpr int NWAVES = WAVES_M * WAVES_N * WAVES_K, NTHREADS = NWAVES * 64;
  constexpr int WM = TM / WAVES_M, WN = TN / WAVES_N, MI = WM / 32, NI = WN / 32;
  static_assert(MI * 32 == WM && NI * 32 == WN, "wave tile must be a multiple of 32");
  constexpr int SUB = (TM + TN) * 8, STAGE = WAVES_K * SUB;  // 16-byte chunks of one 64-wide sub-slab / of a stage
  constexpr int PER_WAVE = STAGE / 64 / NWAVES;              // load instructions of a wavefront per stage
  static_assert(PER_WAVE * 64 * NWAVES == STAGE, "instructions must divide evenly over the wavefronts");
  u32x4 *const sbase = reinterpret_cast<u32x4 *>(smem);

  int tm, tn;
  if (!tile_of(grid, wg, tm, tn)) return;
  const long long m0 = (long long)tm * TM;
  const int n0 = tn * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int wk = wave / (WAVES_M * WAVES_N), wmn = wave % (WAVES_M * WAVES_N), wm = wmn / WAVES_N, wn = wmn % WAVES_N;

  const int a_rows = (int)(M - m0 < TM ? M - m0 : TM), b_rows = N - n0 < TN ? N - n0 : TN;
  const bf16_t *const a_base = A + m0 * K, *const b_base = Bt + (long long)n0 * K;
  const int first_wave = __builtin_amdgcn_readfirstlane(wave);
  constexpr int SLAB = BK * WAVES_K;
  unsigned off[PER_WAVE];  // bytes from the tile's first row of A or Bt (256 rows of K: below 2^31, gemm_mfma_supported)
#pragma unroll
  for (int u = 0; u < PER_WAVE; ++u) {
    const int i = first_wave + u * NWAVES, ks = i / (SUB / 64), p = i % (SUB / 64) * 64 + lane;  // chunk position inside the sub-slab
    const bool isb = i % (SUB / 64) >= TM / 8;
    const int r = (isb ? p - TM * 8 : p) >> 3, c = (p & 7) ^ ((r & 7) ^ ((r >> 3) & 1)), rows = isb ? b_rows : a_rows;
    off[u] = ((unsigned)(r < rows ? r : rows - 1) * K + ks * BK) * 2 + c * 16;
  }
  auto issue = [&](int kt, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < PER_WAVE; ++u) {
      const int i = first_wave + u * NWAVES;
      const bool isb = i % (SUB / 64) >= TM / 8;
      load_to_lds(isb ? b_base : a_base, (unsigned)(isb ? b_rows : a_rows) * K * 2, off[u], kt * (SLAB * 2), sbase + buf * STAGE + i * 64);
    }
  };
  f32x16 acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ni][mi][r] = 0.f;

  const int nk = K / SLAB;
#pragma unroll
  for (int i = 0; i < STAGES - 1; ++i)
    if (i < nk) issue(i, i);
  int buf = 0;
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + STAGES - 1 <= nk) __builtin_amdgcn_s_waitcnt(wait_vm((STAGES - 2) * PER_WAVE) & WAIT_LDS_TOO);
    else __builtin_amdgcn_s_waitcnt(wait_vm(0) & WAIT_LDS_TOO);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int nbuf = buf == 0 ? STAGES - 1 : buf - 1;  // read in the previous step: free since the barrier
    if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1, nbuf);
    const u32x4 *sa = sbase + buf * STAGE + wk * SUB, *sb = sa + TM * 8;
    bf16x8 fa[BK / 16][MI], fb[BK / 16][NI];
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) fa[kk][mi] = __builtin_bit_cast(bf16x8, sa[swz(wm * WM + mi * 32 + l32, kk * 2 + half)]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fb[kk][ni] = __builtin_bit_cast(bf16x8, sb[swz(wn * WN + ni * 32 + l32, kk * 2 + half)]);
    }
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
          acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk][ni], fa[kk][mi], acc[ni][mi], 0, 0, 0);
    buf = buf == STAGES - 1 ? 0 : buf + 1;
  }
  __syncthreads();
  add_wave_parts<WAVES_M * WAVES_N, WAVES_K>(acc, smem, wk, wmn, lane);
  store_tile_bf16<TM, TN, NTHREADS>(acc, smem, wk == 0, wm, wn, tid, C, m0, M, n0, N, split);
}

template <int TM, int TN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES>
__global__ __launch_bounds__(WAVES_M *WAVES_N *WAVES_K * 64) void gemm_bf16_nt_deep_kernel(
    const bf16_t *__restrict__ A, const bf16_t *__restrict__ Bt, bf16_t *__restrict__ C, long long M, int N, int K,
    TileGrid grid, ColumnSplit split) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  gemm_bf16_nt_deep_body<TM, TN, WAVES_M, WAVES_N, WAVES_K, STAGES>(A, Bt, C, M, N, K, grid, split, blockIdx.x, smem);
}

template <int TM, int TN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES>
hipError_t launch_gemm_deep(const void *A, const void *Bt, void *C, long long M, int N, int K, const ColumnSplit &split,
                            hipStream_t s) {
  const TileGrid grid = tile_grid(M, N, K, TM, TN);
  constexpr size_t smem = deep_lds(TM, TN, WAVES_K, STAGES * WAVES_K * (TM + TN));
  if (hipError_t e = raise_lds_limit<gemm_bf16_nt_deep_kernel<TM, TN, WAVES_M, WAVES_N, WAVES_K, STAGES>>(smem); e != hipSuccess) return e;
  gemm_bf16_nt_deep_kernel<TM, TN, WAVES_M, WAVES_N, WAVES_K, STAGES><<<(grid.tiles + 7) / 8 * 8, WAVES_M * WAVES_N * WAVES_K * 64, smem, s>>>(
      (const bf16_t *)A, (const bf16_t *)Bt, (bf16_t *)C, M, N, K, grid, split);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A projection's two adjoints, d_A = d_C W^T (NT) and d_W = A^T d_C (TN), in one launch on small tiles: they are independent, and for
// the row counts these tiles serve neither fills the chip.  Workgroups [0, first) work on the product with the longer tiles.
// Whole backward pass, a launch each -> one (us): 512 tokens of E = 2048, 8 query and 2 KV heads of 128: 86.0 -> 80.3; 2048: 173.0 ->
// 163.2; 1000 of E = 1024, 8 heads of 64: 78.7 -> 67.7; from about 4000 to 8000 tokens on each runs in its own best form.
// ---------------------------------------------------------------------------
struct NtDeep64x64 { static constexpr int TM = 64, TN = 64, WM = 2, WN = 2, WK = 2, ST = 3; };
struct NtDeep64x128 { static constexpr int TM = 64, TN = 128, WM = 1, WN = 4, WK = 2, ST = 3; };
struct NtDeep128x128 { static constexpr int TM = 128, TN = 128, WM = 2, WN = 4, WK = 1, ST = 4; };
struct TnDeep64x64 { static constexpr int TM = 64, TN = 64, WM = 2, WN = 2, WK = 2, ST = 4; };
struct TnDeep64x128 { static constexpr int TM = 64, TN = 128, WM = 2, WN = 2, WK = 2, ST = 4; };
struct TnDeep128x128 { static constexpr int TM = 128, TN = 128, WM = 2, WN = 4, WK = 1, ST = 4; };

struct NtArgs {
  const bf16_t *A, *Bt;
  bf16_t *C;
  long long M;
  int N, K;
  TileGrid grid;
};
struct TnArgs {
  const bf16_t *A, *B;
  bf16_t *C;
  int Mo, No;
  long long K;
  TileGrid grid;
};

template <typename NT_, typename TN_>
__global__ __launch_bounds__(512) void gemm_bf16_pair_kernel(NtArgs nt, TnArgs tn, int first, int nt_first) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wg = (int)blockIdx.x < first ? blockIdx.x : blockIdx.x - first;
  if (((int)blockIdx.x < first) == (nt_first != 0))
    gemm_bf16_nt_deep_body<NT_::TM, NT_::TN, NT_::WM, NT_::WN, NT_::WK, NT_::ST>(nt.A, nt.Bt, nt.C, nt.M, nt.N, nt.K, nt.grid,
                                                                                 ColumnSplit{}, wg, smem);
  else
    gemm_bf16_tn_deep_body<TN_::TM, TN_::TN, TN_::WM, TN_::WN, TN_::WK, TN_::ST>(tn.A, tn.Mo, tn.B, tn.No, tn.C, tn.Mo, tn.No, tn.K,
                                                                                 tn.grid, wg, smem);
}

template <typename NT_, typename TN_>
hipError_t launch_pair(NtArgs nt, TnArgs tn, bool nt_first, hipStream_t s) {
  static_assert(NT_::WM * NT_::WN * NT_::WK == 8 && TN_::WM * TN_::WN * TN_::WK == 8, "512 threads each");
  constexpr size_t a = deep_lds(NT_::TM, NT_::TN, NT_::WK, NT_::ST * NT_::WK * (NT_::TM + NT_::TN)),
                   b = deep_lds(TN_::TM, TN_::TN, TN_::WK, TN_::ST * (TN_::TM + TN_::TN)), smem = a > b ? a : b;
  static_assert(smem <= 160 * 1024, "LDS");
  nt.grid = tile_grid(nt.M, nt.N, nt.K, NT_::TM, NT_::TN);
  tn.grid = tile_grid(tn.Mo, tn.No, tn.K, TN_::TM, TN_::TN);
  const int n_nt = (nt.grid.tiles + 7) / 8 * 8, n_tn = (tn.grid.tiles + 7) / 8 * 8;
  constexpr auto kernel = gemm_bf16_pair_kernel<NT_, TN_>;
  if (hipError_t e = raise_lds_limit<kernel>(smem); e != hipSuccess) return e;
  kernel<<<n_nt + n_tn, 512, smem, s>>>(nt, tn, nt_first ? n_nt : n_tn, nt_first ? 1 : 0);
  return hipGetLastError();
}

}  // namespace

// Measurement aid: nothing but matrix-core instructions (four independent accumulator chains per wavefront, no
// memory traffic inside the loop), to read off the MFMA rate the chip sustains, i.e. the clock it holds under
// matrix-core load.  One float per thread is written so that the work cannot be removed.
__global__ __launch_bounds__(256) void mfma_probe_kernel(float *__restrict__ out, int iters) {
  bf16x8 a, b;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    a[i] = (__bf16)((float)(threadIdx.x & 7) * 0.125f);
    b[i] = (__bf16)((float)i * 0.25f);
  }
  f32x16 c0 = {0}, c1 = {0}, c2 = {0}, c3 = {0};
  for (int it = 0; it < iters; ++it) {
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c1, 0, 0, 0);
    c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c2, 0, 0, 0);
    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c3, 0, 0, 0);
  }
  out[(size_t)blockIdx.x * 256 + threadIdx.x] = c0[0] + c1[1] + c2[2] + c3[3];
}

// The same loop on varied operands: 8 register sets of pseudo-random values in (-2, 2) with random mantissas, as
// activations and weights have.  The matrix cores draw more power multiplying such values than the few small
// constants above (it is the values, not their changing: one random set used for every instruction costs the
// same), and the clock the chip holds follows the power.
__global__ __launch_bounds__(256) void mfma_probe_random_kernel(float *__restrict__ out, int iters) {
  bf16x8 a[8], b[8];
  unsigned h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h = h * 1664525u + 1013904223u;
      a[s][i] = (__bf16)((float)(int)(h >> 8) * (1.0f / 4194304.0f) - 2.0f);
      h = h * 1664525u + 1013904223u;
      b[s][i] = (__bf16)((float)(int)(h >> 8) * (1.0f / 4194304.0f) - 2.0f);
    }
  f32x16 c0 = {0}, c1 = {0}, c2 = {0}, c3 = {0};
  for (int it = 0; it < iters; it += 2) {
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], c1, 0, 0, 0);
    c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[2], c2, 0, 0, 0);
    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[3], b[3], c3, 0, 0, 0);
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[4], b[4], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[5], b[5], c1, 0, 0, 0);
    c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[6], b[6], c2, 0, 0, 0);
    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[7], b[7], c3, 0, 0, 0);
  }
  out[(size_t)blockIdx.x * 256 + threadIdx.x] = c0[0] + c1[1] + c2[2] + c3[3];
}

hipError_t mfma_probe(float *out, int blocks, int iters, bool random_operands, hipStream_t s) {
  if (random_operands) mfma_probe_random_kernel<<<blocks, 256, 0, s>>>(out, iters);
  else mfma_probe_kernel<<<blocks, 256, 0, s>>>(out, iters);
  return hipGetLastError();
}

// (a tile's 256 rows are addressed with 32 bits)
bool gemm_mfma_supported(long long M, int N, int K) { return M >= 1 && K % BK == 0 && K >= BK && K < 1 << 22 && N % 8 == 0 && N >= 8; }

hipError_t gemm_mfma_bf16(const void *A, const void *Bt, void *C, long long M, int N, int K, hipStream_t s,
                          const ColumnSplit &split) {
  switch (nt_tile(M, N, K)) {
    case NT_256x256: return launch_gemm<256, 256, 2, 4>(A, Bt, C, M, N, K, split, s);
    case NT_256x192: return launch_gemm<256, 192, 2, 4>(A, Bt, C, M, N, K, split, s);
    case NT_192x256: return launch_gemm<192, 256, 2, 4>(A, Bt, C, M, N, K, split, s);
    case NT_256x128: return launch_gemm<256, 128, 4, 2>(A, Bt, C, M, N, K, split, s);
    case NT_192x192: return launch_gemm<192, 192, 2, 4>(A, Bt, C, M, N, K, split, s);
    case NT_64x64: return launch_gemm_deep<64, 64, 2, 2, 2, 3>(A, Bt, C, M, N, K, split, s);
    case NT_64x128: return launch_gemm_deep<64, 128, 1, 4, 2, 3>(A, Bt, C, M, N, K, split, s);
    case NT_128x128: return launch_gemm_deep<128, 128, 2, 4, 1, 4>(A, Bt, C, M, N, K, split, s);
  }
  return hipErrorInvalidValue;
}

// (64 tokens are addressed with 32 bits)
bool gemm_tn_mfma_supported(int Mo, int No, long long K) {
  return Mo % 8 == 0 && No % 8 == 0 && Mo >= 8 && No >= 8 && Mo < 1 << 23 && No < 1 << 23 && K >= 1;
}

size_t gemm_tn_scratch_bytes(int Mo, int No, long long K) { return (size_t)tn_part_blocks(Mo, No, K) * 1024 * sizeof(float); }

hipError_t gemm_tn_mfma_bf16(const void *A, long long lda, const void *Bm, long long ldb, void *C, int Mo, int No,
                             long long K, float *part, hipStream_t s) {
  switch (tn_tile(Mo, No, K)) {
    case TN_64x64: return launch_tn_deep<64, 64, 2, 2, 2, 4>(A, lda, Bm, ldb, C, Mo, No, K, s);
    case TN_64x128: return launch_tn_deep<64, 128, 2, 2, 2, 4>(A, lda, Bm, ldb, C, Mo, No, K, s);
    case TN_128x128: return launch_tn_deep<128, 128, 2, 4, 1, 4>(A, lda, Bm, ldb, C, Mo, No, K, s);
    case TN_SPLIT: break;
  }
  const int splits = tn_splits(Mo, No, K);
  const int tiles_m = (Mo + BM - 1) / BM, tiles_n = (No + TN_BN - 1) / TN_BN;
  const int total = tiles_m * tiles_n;
  const long long nk = (K + BK - 1) / BK;
  const int per = (int)((nk + splits - 1) / splits);
  constexpr size_t smem = (size_t)(A_STAGES + B_STAGES) * BK * 256 * 2;
  if (hipError_t e = raise_lds_limit<gemm_bf16_tn_kernel>(smem); e != hipSuccess) return e;
  gemm_bf16_tn_kernel<<<(total * splits + 7) / 8 * 8, 512, smem, s>>>((const bf16_t *)A, lda, (const bf16_t *)Bm, ldb, part, (bf16_t *)C,
                                                                       Mo, No, K, tiles_n, total, splits, per);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits == 1) return e;
  const int blocks = ((Mo + 31) / 32) * ((No + 127) / 128);
  splitk_reduce_kernel<<<blocks, 256, 0, s>>>(part, splits, Mo, No, (bf16_t *)C);
  return hipGetLastError();
}

hipError_t gemm_adjoint_pair(const void *d_C, const void *W, void *d_A, const void *A, void *d_W, long long rows, int n_in, int n_out,
                             float *part, hipStream_t s) {
  const PairForm f = gemm_pair(rows, n_in, n_out);
  if (!f.one_launch) {
    if (hipError_t e = gemm_tn_mfma_bf16(A, n_in, d_C, n_out, d_W, n_in, n_out, rows, part, s); e != hipSuccess) return e;
    return gemm_mfma_bf16(d_C, W, d_A, rows, n_in, n_out, s);
  }
  const NtArgs nt{(const bf16_t *)d_C, (const bf16_t *)W, (bf16_t *)d_A, rows, n_in, n_out, {}};
  const TnArgs tn{(const bf16_t *)A, (const bf16_t *)d_C, (bf16_t *)d_W, n_in, n_out, rows, {}};
#define PAIR(NT_)                                                                               \
  switch (f.tn) {                                                                               \
    case TN_64x64: return launch_pair<NT_, TnDeep64x64>(nt, tn, f.nt_first, s);                 \
    case TN_64x128: return launch_pair<NT_, TnDeep64x128>(nt, tn, f.nt_first, s);               \
    default: return launch_pair<NT_, TnDeep128x128>(nt, tn, f.nt_first, s);                     \
  }
  switch (f.nt) {
    case NT_64x64: PAIR(NtDeep64x64)
    case NT_64x128: PAIR(NtDeep64x128)
    default: PAIR(NtDeep128x128)
  }
#undef PAIR
}

hipError_t transpose_bf16(const void *src, void *dst, int rows, int cols, hipStream_t s) {
  TransposePair p;
  if (hipError_t e = make_transposes(src, dst, rows, cols, nullptr, nullptr, 0, 0, &p); e != hipSuccess) return e;
  return transpose2_bf16(p, s);
}

hipError_t make_transposes(const void *src1, void *dst1, int rows1, int cols1, const void *src2, void *dst2, int rows2, int cols2,
                           TransposePair *pair) {
  if (rows1 % 8 || cols1 % 8 || (src2 && (rows2 % 8 || cols2 % 8))) return hipErrorInvalidValue;
  *pair = TransposePair{(const bf16_t *)src1, (const bf16_t *)src2, (bf16_t *)dst1, (bf16_t *)dst2, rows1, cols1,
                        ((cols1 + 63) / 64) * ((rows1 + 63) / 64), rows2, cols2,
                        src2 ? ((cols2 + 63) / 64) * ((rows2 + 63) / 64) : 0};
  return hipSuccess;
}

hipError_t transpose2_bf16(const TransposePair &pair, hipStream_t s) {
  transpose_bf16_kernel<<<pair.n1 + pair.n2, 256, 0, s>>>(pair);
  return hipGetLastError();
}

}  // namespace cca
