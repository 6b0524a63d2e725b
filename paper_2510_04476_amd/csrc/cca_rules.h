// Which form of a kernel serves a call: rules on sizes alone, in plain host arithmetic (no HIP), so that the launchers and the
// tests ask the same functions.  Every rule compares estimated times; the constants are fits to measurements, quoted beside
// them in microseconds.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>

namespace cca {

// ---- projections: C (M,N) = A (M,K) * Bt (N,K)^T, bf16 -------------------------------------------------------------------
enum NtTile { NT_256x256, NT_256x192, NT_64x64, NT_64x128, NT_128x128, NT_256x128, NT_192x256, NT_192x192 };  // rows x columns

// A tile shape costs (rounds of the grid over the chip) x (64-wide slabs x time per slab + fill and epilogue).  The two
// numbers of each large shape (us) are fits (11 % rms) to back-to-back timings of every shape at K = 256 ... 4096,
// N = 512 ... 6144, M = 1500 ... 16384; over these the choice costs 0.5 % on average against the best shape.  They rank the shapes of one
// product: the chip's clock falls under a long one, which takes up to 1.3 times the estimate (16384 x 1536 x 2048: 67.7, measured 85).  The small shapes' (128 x 128
// and below) are fits over M = 64 ... 16384.
//   256 x 256 (1.06, 7.5)  192 x 256 (0.90, 6.1)  256 x 192 (0.87, 6.0)  192 x 192 (0.715, 5.1)  256 x 128 (0.66, 4.9)
//   128 x 128 (0.528, 3)  64 x 128 (0.354, 3)  64 x 64 (0.232, 2.2)
// e.g. N = 1536, M = 16384: 384 tiles of 256 (2 rounds, half empty, 102 us) or 512 tiles of 256 x 192 (2 full rounds, 86); N = 2048,
// K = 1024, M = 6000: 192 tiles of 256 x 256 (29.5) or 256 of 192 x 256 (24.7); N = 1536, K = 2048, M = 6000: 192 tiles of 256 x 192 (38.2)
// or 256 of 192 x 192 (35.6); M = 12000: 376 of 256 x 192 or 504 of 192 x 192, K = 2048 76.1 and 64.4, K = 4096 139.0 and 124.8, K = 8192
// 264.3 and 230.5.
inline NtTile nt_tile(long long M, int N, int K, double *us = nullptr) {
  const double slabs = (double)(K / 64);
  const bool halves = K % 128 == 0;  // the shapes that split a slab over two halves of the wavefronts
  const struct { NtTile t; int tm, tn; double per_slab, fixed; bool ok; } shapes[] = {
      {NT_256x192, 256, 192, 0.87, 6.0, true}, {NT_256x256, 256, 256, 1.06, 7.5, true}, {NT_192x256, 192, 256, 0.90, 6.1, true},
      {NT_192x192, 192, 192, 0.715, 5.1, true}, {NT_256x128, 256, 128, 0.66, 4.9, true}, {NT_128x128, 128, 128, 0.528, 3.0, true}, {NT_64x128, 64, 128, 0.354, 3.0, halves},
      {NT_64x64, 64, 64, 0.232, 2.2, halves}};
  NtTile best = NT_128x128;
  double least = 1e300;
  for (const auto &f : shapes) {
    const long long tiles = ((M + f.tm - 1) / f.tm) * ((N + f.tn - 1) / f.tn);
    const double cost = (double)((tiles + 255) / 256) * (slabs * f.per_slab + f.fixed);
    if (f.ok && cost < least) least = cost, best = f.t;
  }
  if (us) *us = least;
  return best;
}

// ---- start of a large product ----------------------------------------------------------------------------------------------
// How many of its first slabs a workgroup of the large products (tile of `area` elements) follows with a pause of 0.7 us.  Without any, all CUs
// come to full load within a slab's time, in every round of the grid; the chip answers with a lower clock, for as long as a loop over
// a layer lasts (it recovers within milliseconds: the next pass is there before), and kernels that draw less than the product run up
// to 14 % slower.  Attention adjoint over 12000 tokens, 12 / 4 heads of 64, 937 us by itself, behind three products; us, and the product's own,
// without pauses, with two, with four: 12288 x 1536 x 1280 on 192 x 192 1070, 990, 936 (46.9, 46.8, 46.3); 16384 x 1536 x 2048 on 256 x 192 1069, 937, 938
// (83.2, 78.5, 79.5); 6144 x 2048 x 2048 on 192 x 256, one round, 984, 936, 936 (42.0, 41.0, 41.6).  Whole calls: training, 12000 tokens, E =
// 1536, 12 / 4 heads of 64 1779, 1699, 1630; 16384, 8 / 2 of 128 2851, 2756, 2761; prefill 16384 635.3, 629.1, 631.2; 2 x 3000, 4 / 1 of 256, not
// causal 181.7, 176.8, 178.0; 4096, plain heads 198.9, 193.5, 200.3; 6000, 16 / 2 plain heads 244.3, 245.8, 246.9.  On a machine with power to spare calls take
// up to 1 % longer with two (4096, plain heads 191.4, 192.7; prefill 16384 629.9, 631.9).
// So two, and four for several rounds of the smaller ones of these tiles, whose slabs are shorter.  None on less than 7/8 of the CUs, where
// they cost short calls more than they give (4593 x 1536 x 2048, 216 workgroups: 975 -> 935, 27.7 -> 28.5; 4593 x 2048 x 512 1.5 us of a
// pass of 75).  Not better: fewer and longer pauses, starts spread over 8 us by CU or XCD (as good behind the product, 2-4
// us longer on one round), the first round's workgroups alone (no effect on two); in the weight gradients (no effect on whole calls).
inline int start_pauses(int area, long long tiles, long long slabs) {
  if (tiles < 224 || slabs < 8) return 0;
  return area < 192 * 256 && tiles > 256 ? 4 : 2;
}

// ---- order of the tiles of a product ---------------------------------------------------------------------------------------
// Each XCD gets a contiguous range of tiles, taken down panels of `panel` columns of tiles.  Its L2 has to bring in the rows of both
// operands that its range touches (the first 32 tiles of it, one per CU): the panel width that makes the fewest of them, unless row by row they
// fit its 4 MB anyway.  There a panel saves nothing, and the next kernel finds its rows in other L2s than their reader's: whole prefill, us, row
// by row -> in panels (tokens, E, H_q + 2 H_k, d_h; MB row by row of the two products): 1024, 1024, 20, 64 (2.8, 2.2): 26.9 -> 28.2 and 31.1
// -> 32.4; 1024, 1536, 12, 64 (2.6, 1.2): 32.9 -> 33.9; above it 512, 2048, 48, 64 (12.2, 4.1): 41.2 -> 37.2; 200, 2048, 96, 64 (12.2, 4.2):
// 35.3 -> 31.8; 1024, 2048, 32, 64 (8.5, 4.2): 46.7 -> 45.0.  The same with the weights of twelve layers in turn (0.94-0.98, 1.02-1.08x).
// Row by row -> in panels, us (rows x columns x contraction): 300 x 1536 x 2048 18.0 -> 15.0, 300 x 3072
// x 4096 32.8 -> 27.4 (64 x 64 tiles), 1000 x 2048 x 1024 16.7 -> 15.1 (64 x 128), 1000 x 4096 x 2048 34.8 -> 33.7, 12000 x 4096 x 2048
// 209 -> 200 (256 x 256).  Tiles 128 columns wide and as high lost 1 ... 4 % where the panels save less than half of the rows (1531 x 1536
// x 2048 27.1 -> 27.8) and keep the row order there.
// The choice is made on the host for every launch, so it looks at few widths: whole rows, whole columns, and between those that put a
// range into one or two panels and are no wider than 16, where the rows an XCD's 32 tiles touch are fewest; of these only such
// that could beat the best so far.  The cost is that of a search over every width (up to 300 x 1024 tiles of every shape), in 0.2 ... 0.6 us
// a launch; the search took 3.1 at 512 x 1536 x 2048, 31 at 128 x 12288 x 8192, 380 at 1024 columns of tiles.
struct TilePanel {
  unsigned tiles_m, tiles_n, tm, tn, tiles, range, at_once;  // range: tiles of an XCD; at_once: those that run first
  TilePanel(int tiles_m_, int tiles_n_, int tm_, int tn_)
      : tiles_m(tiles_m_), tiles_n(tiles_n_), tm(tm_), tn(tn_), tiles(tiles_m * tiles_n), range((tiles + 7) / 8), at_once(range < 32 ? range : 32) {}
  // rows of both operands that the ranges touch with panels of w columns
  unsigned touched(unsigned w) const {
    const unsigned full = w * tiles_m;
    unsigned sum = 0;
    for (unsigned a = 0; a < tiles; a += range) {
      const unsigned b = a + at_once < tiles ? a + at_once : tiles;
      if (w == 1) {  // whole columns one after the other
        sum += (b - a < tiles_m ? b - a : tiles_m) * tm + ((b - 1) / tiles_m - a / tiles_m + 1) * tn;
        continue;
      }
      unsigned rows = 0, cols = 0;
      for (unsigned p = a / full, start = p * full; start < b; ++p, start += full) {
        const unsigned lo = a > start ? a - start : 0, hi = b - start < full ? b - start : full, left = tiles_n - p * w, width = w < left ? w : left;
        rows += (hi - 1) / width - lo / width + 1;
        cols += hi - lo < width ? hi - lo : width;
      }
      sum += (rows < tiles_m ? rows : tiles_m) * tm + cols * tn;
    }
    return sum;
  }
  // the widths of ceil(tiles_n / w) panels as even as can be
  unsigned even(unsigned w) const {
    const unsigned panels = (tiles_n + w - 1) / w;
    return (tiles_n + panels - 1) / panels;
  }
  unsigned best() const {
    const unsigned row_major = touched(tiles_n), ranges = (tiles - at_once) / range + 1;  // ranges of at_once tiles
    unsigned width = tiles_n, least = row_major;
    auto look_at = [&](unsigned w) {
      const unsigned cost = touched(w);
      if (cost < least || (cost == least && w > width)) least = cost, width = w;
    };
    const unsigned square = even((unsigned)fmin(sqrt((double)at_once * tm / tn) + 0.5, (double)tiles_n));
    if (square < tiles_n) look_at(square);
    const unsigned narrow = at_once / tiles_m > 2 ? at_once / tiles_m : 2;  // (narrower, a range takes several panels whole: no fewer columns)
    for (unsigned w = tiles_n - 1 < 16 ? tiles_n - 1 : 16; w >= narrow; --w) {
      w = even(w);
      const unsigned rows = (at_once + w - 1) / w, cols = w < at_once ? w : at_once;
      if (w != square && w > 1 && ranges * ((rows < tiles_m ? rows : tiles_m) * tm + cols * tn) <= least + least / 16) look_at(w);  // (a narrower last panel touches a little less)
    }
    if (tiles_n > 1) look_at(1);
    return tn == 128 && tm >= 128 && 2 * least > row_major ? tiles_n : width;
  }
};
// Columns of a panel; `K`: terms of the contraction, two bytes each
inline int tile_panel(int tiles_m, int tiles_n, int tm, int tn, long long K) {
  const TilePanel p(tiles_m, tiles_n, tm, tn);
  return (long long)p.touched((unsigned)tiles_n) * K * 2 <= 8 * (4ll << 20) ? tiles_n : (int)p.best();
}

// ---- weight gradients: C (Mo,No) = A (K,Mo)^T * B (K,No), bf16, K tokens -------------------------------------------------
enum TnTile { TN_SPLIT, TN_64x64, TN_64x128, TN_128x128 };

// Number of K splits: minimise (rounds on 256 CUs) x (slabs per split) x (time of a 256 x 256 x 64 slab) + the two launches
// and the fp32 partial sums, written and read once (one split stores the result itself).  Fits (8 % rms) to back-to-back timings of 1 ...
// 32 splits at K = 256 ... 16384, 2 ... 192 tiles: a slab takes 0.92 us on a few CUs and 1.13 with all of them at work, the rest 9.6 us +
// the bytes at 7.2 TB/s, 4.6 without partial sums.  `us`: that minimum.  1024 x 2048 over 7996 tokens: 5 splits 47.2, 7 splits 45.3, 10
// splits 62.4 us; 2048 x 2048 over 8192: 5 splits 98.0, 4 splits 69.9; 512 x 512 over 12000: 16 splits 28.3, 32 splits 26.7.
inline int tn_splits(int Mo, int No, long long K, double *us = nullptr) {
  const long long tiles = (long long)((Mo + 255) / 256) * ((No + 255) / 256);
  const long long nk = (K + 63) / 64;
  int best = 1;
  double best_t = -1.0;
  for (int sp = 1; sp <= 32; ++sp) {
    const long long per = (nk + sp - 1) / sp;
    if (sp > 1 && per < 4) break;
    if ((per * (sp - 1)) >= nk) continue;  // an empty last split
    const double busy = tiles * sp < 256 ? (double)(tiles * sp) / 256.0 : 1.0;
    const double t = (double)((tiles * sp + 255) / 256) * (double)per * (0.92 + 0.21 * busy * busy * busy) +
                     (sp == 1 ? 4.6 : 9.6 + (double)sp * Mo * No * 8.0 / 7.2e6);
    if (best_t < 0 || t < best_t) best_t = t, best = sp;
  }
  if (us) *us = best_t;
  return best;
}

// Small tiles without partial sums or 256 x 256 tiles split over K, by estimated time (us).  Fits (8 % rms) to back-to-back
// timings over K = 256 ... 16384 tokens and 8 ... 768 tiles of (rounds) x (slabs x time per slab + fill and epilogue), b the share of
// the CUs at work: 128 x 128 (0.509 + 0.051 b^4, 4.1), 64 x 128 (0.336 + 0.023 b^2, 3.6), 64 x 64 (0.209, 3.7) up to one workgroup per CU
// and (0.488, 3.2) at two; the split form as in tn_splits.  Over these the choice costs 0.5 % on average, 13 % at most.  2048 x 1536 over
// 1024 tokens 128 x 128 12.9 us, 64 x 64 15.5, over 4000 38.1 and split 39.4, over 7996 split 57.5; 2048 x 2048 over 4000 128 x 128 41.1,
// over 8192 split 69.9.
inline TnTile tn_tile(int Mo, int No, long long K, double *us = nullptr) {
  const double slabs = (double)((K + 63) / 64);
  auto tiles = [&](int tm, int tn) { return (long long)((Mo + tm - 1) / tm) * ((No + tn - 1) / tn); };
  auto busy = [](long long t) { return t < 256 ? (double)t / 256.0 : 1.0; };
  double split_us;
  tn_splits(Mo, No, K, &split_us);
  const long long t128 = tiles(128, 128), t64x128 = tiles(64, 128), t64 = tiles(64, 64);
  const double c128 = (double)((t128 + 255) / 256) * (slabs * (0.509 + 0.051 * pow(busy(t128), 4.0)) + 4.1),
               c64x128 = (double)((t64x128 + 255) / 256) * (slabs * (0.336 + 0.023 * pow(busy(t64x128), 2.0)) + 3.6),
               c64 = t64 <= 256 ? slabs * 0.209 + 3.7 : (double)((t64 + 511) / 512) * (slabs * 0.488 + 3.2);
  const double small = fmin(c128, fmin(c64x128, c64));
  if (us) *us = fmin(small, split_us);
  if (small >= split_us) return TN_SPLIT;
  return c64 == small ? TN_64x64 : c64x128 == small ? TN_64x128 : TN_128x128;
}

// 32 x 32 blocks of fp32 partial sums that the product leaves: none where one workgroup walks all of K or one split stores its result
inline long long tn_part_blocks(int Mo, int No, long long K) {
  const int splits = tn_splits(Mo, No, K);
  return tn_tile(Mo, No, K) == TN_SPLIT && splits > 1 ? (long long)splits * ((Mo + 31) / 32) * ((No + 31) / 32) : 0;
}

// ---- launches that share ------------------------------------------------------------------------------------------------
// Whether two buffers have bytes in common.  Products that were a launch each ran in stream order, so that one's output could lie over
// the other's input; where it does they still get a launch each.
inline bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes) {
  const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
  return a0 < b0 + b_bytes && b0 < a0 + a_bytes;
}

// ---- the two adjoints of a projection, d_A (rows, n_in) = d_C (rows, n_out) W^T and d_W (n_in, n_out) = A^T d_C -----------------
// One launch on small tiles of both, one workgroup per CU, the product with the longer tiles first, or a launch each in its own best
// form.  The time of the one launch is that of its busiest CU: workgroups go round the 8 XCDs, there round the 4 groups of 8 CUs, and in a
// group to the CU that is free first.  Both sides are fits (3 % and 5 % rms) to the same sweep of whole adjoints, all nine pairs of tiles in
// either order and two launches, 64 ... 8192 rows, 24 products of E = 1024 ... 2048 and 256 ... 6144 columns: a tile takes (slabs x time per
// slab + fill and epilogue), us, NT 64 x 64 (0.185, 2.0), 64 x 128 (0.275, 2.7), 128 x 128 (0.45, 2.4), TN 0.23, 1.9, 0.32, 2.55 and 0.51, 2.6, the
// slabs a tenth slower with all CUs at work, the launch 1.4; two launches the sum of what ranks their own tiles, which their
// length at a falling clock makes 1.05 and 1.15 of it.  Beyond 55 us the one launch is held to a tenth more: from there on it takes 3 ... 8 %
// more than its estimate (8192 x 1024 x 2048: 75.6, measured 82.1, two launches 78.4), where the large tiles of two launches gain.  Above 10000
// rows a tile's walk along all of them takes longer than two launches (10974 x 512 x 1024: 46.3 and 43.7; 11810: 49.1 and 44.8).  Over the
// sweep the choice costs 0.5 % on average, 9 % at most (E = 2048, 2048 columns, 1400 rows: 38.7 and 35.6); with the busiest CU of an even
// deal over all 256 and the single products' numbers 2.4 % and 38 %.  One launch and two, us: 2100 x 1536 x 640 16.5 and 27.6, 4096 x 768 x
// 1536 30.3 and 44.7, 4096 x 1536 x 1280 42.5 and 46.8, 8000 x 1536 x 1536 105.9 and 82.4.
struct PairForm {
  bool one_launch;
  NtTile nt;
  TnTile tn;
  bool nt_first;
};
// 8 CUs, n_long tiles and then n_short, each to the CU that is free first
inline double dealt_to_8(int n_long, double t_long, int n_short, double t_short) {
  const int more = n_long % 8, others = 8 - more;  // `more` CUs take one long tile more
  const double low = (double)(n_long / 8) * t_long, high = low + t_long;
  if (!more) return low + (double)((n_short + 7) / 8) * t_short;
  const int beside = (int)(t_long / t_short);  // short tiles of another CU beside the last long one
  if (n_short <= others * beside) return fmax(high, low + (double)((n_short + others - 1) / others) * t_short);
  const int left = n_short - others * beside, rounds = left / 8, last = left % 8;
  if (!last) return high + (double)rounds * t_short;
  return last <= others ? low + (double)(beside + rounds + 1) * t_short : high + (double)(rounds + 1) * t_short;
}
inline double dealt(long long n_long, double t_long, long long n_short, double t_short) {
  const int l = (int)((n_long + 7) / 8), s = (int)((n_short + 7) / 8);  // of an XCD
  double most = 0.0;
  for (int g = 0; g < 4; ++g) {
    const int lg = (l - g + 3) / 4;
    most = fmax(most, dealt_to_8(lg, t_long, (l + s - g + 3) / 4 - lg, t_short));
  }
  return most;
}
inline PairForm gemm_pair(long long rows, int n_in, int n_out) {
  PairForm best{false, NT_256x256, TN_SPLIT, true};
  double nt_us, tn_us;
  nt_tile(rows, n_in, n_out, &nt_us);
  tn_tile(n_in, n_out, rows, &tn_us);
  if (rows > 10000) return best;
  double least = 1.05 * nt_us + 1.15 * tn_us;
  const double s_nt = (double)(n_out / 64), s_tn = (double)((rows + 63) / 64);
  auto tiles = [](long long m, long long n, int tm, int tn) { return ((m + tm - 1) / tm) * ((n + tn - 1) / tn); };
  const bool halves = n_out % 128 == 0;
  const struct { NtTile t; int tm, tn; double slab, fixed; bool ok; } nts[3] = {
      {NT_64x64, 64, 64, 0.185, 2.0, halves}, {NT_64x128, 64, 128, 0.275, 2.7, halves}, {NT_128x128, 128, 128, 0.45, 2.4, true}};
  const struct { TnTile t; int tm, tn; double slab, fixed; } tns[3] = {
      {TN_64x64, 64, 64, 0.23, 1.9}, {TN_64x128, 64, 128, 0.32, 2.55}, {TN_128x128, 128, 128, 0.51, 2.6}};
  for (const auto &a : nts)
    for (const auto &b : tns) {
      if (!a.ok) continue;
      const long long na = tiles(rows, n_in, a.tm, a.tn), nb = tiles(n_in, n_out, b.tm, b.tn);
      if ((na > nb ? na : nb) > 1 << 24) continue;  // (counted in ints; far from where one launch pays)
      const double busy = na + nb < 256 ? (double)(na + nb) / 256.0 : 1.0, slower = 1.0 + 0.1 * busy * busy;
      const double ta = s_nt * a.slab * slower + a.fixed, tb = s_tn * b.slab * slower + b.fixed;
      double us = 1.4 + (ta >= tb ? dealt(na, ta, nb, tb) : dealt(nb, tb, na, ta));
      if (us > 55.0) us *= 1.1;
      if (us < least) least = us, best = PairForm{true, a.t, b.t, ta >= tb};
    }
  return best;
}

// ---- grids of the attention kernels (forward and backward, d_h <= 128), one 8-wavefront workgroup per CU -----------------
// BH = batch x query heads.  Blocks of `rows` query rows (or keys); whether each workgroup takes two of them.  Causal work per
// block grows (keys: falls) with its index.  Giving every workgroup one heavy and one light block (equal work for all)
// measured ~20 % faster in the forward kernel at BH = 8 than issuing the heavy blocks first; only worth it while it still
// leaves a workgroup for each of the 256 CUs.
inline int row_blocks(int T, int rows) { return (T + rows - 1) / rows; }
inline bool pair_blocks(long long BH, bool causal, int blocks) { return causal && BH * ((blocks + 1) / 2) >= 256; }
// A grid takes as long as its busiest CU: steps of 64 rows of the other kind per group of wavefronts, with 256 rows per
// workgroup (one group) or 128 (two groups, each with half of the steps); a block's steps end with the sequence.  Workgroups
// are issued longest first: up to 256 the longest counts, up to 512 the CU that takes the 256th and the 257th, beyond that an even share.
// Every block pays `start` steps (its resident rows and first tile); the split form's steps cost `step` each (a tile is staged
// for half as many rows), its blocks `merge` steps more, and with all CUs at work everything a share `busy` more.  `pairs`: the
// kernel takes paired blocks.
struct SplitCost {
  double start, step, merge, busy;
};
inline double busiest_cu(long long BH, int T, bool causal, int rows, bool pairs, const SplitCost &c) {
  const long long n = row_blocks(T, rows), steps = (T + 63) / 64;
  const double tile = c.step * rows / 256.0;
  auto block = [&](long long i) {  // the i-th in the order of its work
    const long long s = (i + 1) * (rows / 64);
    return (double)(causal && s < steps ? s : steps) * tile + c.start + c.merge;
  };
  const bool paired = pairs && pair_blocks(BH, causal, (int)n);
  const long long units = paired ? (n + 1) / 2 : n, jobs = BH * units;
  auto unit = [&](long long i) { return block(n - 1 - i) + (paired && 2 * i < n - 1 ? block(i) : 0.0); };  // as issued
  const double longest = fmax(unit(0), units > 1 ? unit(1) : 0.0);
  const double all = causal ? (double)((rows / 64) * (n * (n - 1) / 2) + steps) : (double)(n * steps);
  const double even = (double)BH * (all * tile + (double)n * (c.start + c.merge)) / 256.0;
  double t = longest;
  if (jobs > 512) t = fmax(longest, even + 0.5 * unit(units - 1));
  else if (jobs > 256) t = fmax(longest, unit(255 / BH) + unit(256 / BH));
  return t * (1.0 + c.busy * fmin(1.0, even / longest));
}
inline bool split_pays(long long BH, int T, bool causal, bool pairs, const SplitCost &split) {
  return busiest_cu(BH, T, causal, 128, pairs, split) < busiest_cu(BH, T, causal, 256, pairs, SplitCost{split.start, 1.0, 0.0, 0.0});
}
// Forward: two key groups per workgroup (128 query rows, half the key tiles for each group) or one (256 rows)?  256-row blocks
// leave most CUs idle until B * H_q * T reaches about 32 k rows, and each walks all keys of its rows.  The costs are the
// best of a grid against timings of both forms at d_h = 64 and 128, B * H_q = 1 ... 128, T = 40 ... 12288, causal with and without
// a bound on the scores and not causal: over these the choice costs 0.4 % on average against the faster form.
// Measured (T, B * H_q, d_h: one group -> two, us, causal): split 512, 8, 128: 19.1 -> 16.2; 2048, 8, 128: 47.6 -> 33.6;
// 8192, 8, 128: 171.6 -> 134.2; 4096, 16, 128 without bound: 101.8 -> 81.8; 1531, 24, 64: 26.6 -> 19.4; kept on one group
// 64, 8, 64: 4.4 -> 5.4; 128, 8, 128: 8.2 -> 9.4; 400, 96, 64: 10.8 -> 15.6; 640, 64, 64: 12.7 -> 14.1; 16384, 8, 128: 446 ->
// 501; 1999, 64, 64: 44.7 -> 54.7; the line is soft (777, 48, 128 is split: 24.7 -> 26.0).  256 threads and 128 rows without the split: 2048, 8: 38.1.
inline bool fwd_splits_keys(long long BH, int T, bool causal) {
  return split_pays(BH, T, causal, true, SplitCost{3.0, 1.04, 1.0, 0.2});
}
// Two key groups: blocks of 64 rows (256 threads, one wavefront per SIMD) where they still are one round of the grid, or of 128?  A
// step over a key tile is then shorter by what two wavefronts of a SIMD cost each other (us, 128 rows -> 64; B * H_q, d_h): T = 400, 8,
// 128: 13.4 -> 12.0; 512, 8, 128: 15.0 -> 13.5; 512, 24, 64: 10.1 -> 9.0; 777, 8, 128: 17.7 -> 16.7; 1024, 16, 64: 13.5 -> 12.5; 1280,
// 4, 64: 15.2 -> 14.1; 1531, 8, 128: 25.8 -> 25.6; 2048, 8: 31.5 -> 31.6; beyond a round 777, 24, 64: 12.1 -> 12.7, not causal 13.0 ->
// 22.9; without a bound on the scores 512, 16, 64: 9.9 -> 9.8, 777: 12.1 -> 13.0.
inline bool fwd_takes_64_rows(long long BH, int T, bool normed) { return normed && T <= 1536 && BH * ((T + 63) / 64) <= 256; }
// Backward, likewise (B * H_q = 4 ... 400, T = 64 ... 16384, causal and not, one and four query heads per KV head): neither kernel
// is split where that measured more than 2 % slower, and the choice costs 0.1 % on average.  Attention backward, us, neither -> dQ
// -> dK / dV -> both split, causal, d_h = 128: T = 512, B * H_q = 16: 71 -> 64 -> 59 -> 53; 2048, 8: 180 -> 156 -> 139 -> 115;
// 8192, 8: 658 -> 590 -> 546 -> 478; 4096, 16 MHA: 343 -> 312 -> 290 -> 258; d_h = 64, 1531, 24: 95 -> 83 -> 78 -> 65; kept whole:
// 1999, 64: 174 -> 181 -> 185 -> 194; dK / dV alone 1531, 64: 104.5 -> 115.3; dQ alone 300, 128: 36.8 -> 38.8, and not causal
// 6000, 64, d_h = 64: 2084 -> 2246.
constexpr SplitCost BWD_SPLIT{2.0, 1.0, 1.0, 0.1};
inline bool dq_splits_keys(long long BH, int T, bool causal) { return split_pays(BH, T, causal, true, BWD_SPLIT); }
inline bool dkdv_splits_rows(long long BH, int T, bool causal) { return split_pays(BH, T, causal, false, BWD_SPLIT); }

// ---- prologue at d_h = 64, 128: 64 tokens of one head per workgroup, everything requested at once, or 256 and more ------------
// The short form reads the whole filter for every 64 tokens (d_h = 128: one workgroup per CU, 64: three), the long one's workgroups
// are a chain of ten memory latencies, longer where a key head adds the rows of several query heads.  Its lead ends with the first
// round of the grid, at R > 1 with the second.  Prologue with its set-up, short and long, us (heads, rows): d_h = 128: 8 + 2, 512:
// 12.4, 18.8; 3000: 19.1, 20.0; 4593: 25.5, 21.2; 4 + 4, 2048: 13.3, 16.7; 3000: 19.0, 16.9; 32 + 8, 512: 20.1, 22.7; 1024: 26.5,
// 23.3; d_h = 64: 16 + 4, 1024: 10.2, 12.0; 2048: 12.1, 12.6; 3000: 14.9, 14.1; 8 + 8, 3000: 13.2, 12.1.  The adjoint shares its
// launch with the filter gradients: d_h = 128: 8 + 2, 1024: 35.7, 38.5; 2048: 48.6, 47.2; 4 + 4, 2048: 41.5, 39.1; d_h = 64: 16 + 4,
// 3000: 36.0, 37.8; 4593: 43.2, 43.8; 8000: 56.6, 56.0.
inline bool prologue_is_short(long long rows, int heads, int R, int dh, bool adjoint) {
  const long long blocks = (rows + 63) / 64 * heads;
  if (dh == 64) return blocks <= (adjoint ? 1536 : 640);
  return blocks <= (adjoint ? 240 : R > 1 ? 512 : 256);
}

// ---- filter gradients of the prologue's adjoint -------------------------------------------------------------------------------
// Tokens per chunk of the filter-gradient kernel: the largest of 512..64 (or more, below) that still gives 80 workgroups.  They run beside the
// adjoint's (at d_h = 256 in a launch of their own), and every chunk's sums (196 KB a head at d_h = 128) are written and read once more: with 256 workgroups and a unit's
// last few chunks added one after the other the backward pass took (us, then now) 2 x 512 tokens, 8 query and 2 KV heads of 128:
// 105.7, 99.5; 2 x 2048: 266.0, 251.6; 1 x 2048, 6 + 6 heads: 179.7, 165.3; 1 x 4096, 4 + 1 heads of 256: 638, 631; 40 workgroups:
// 98.1, 256.6, 165.7, 628.  The prologue's adjoint alone at d_h = 256 (heads, tokens; before this chunk and other changes of its adjoint, and
// after): 4 + 1, 1024: 70.5, 59.7; 2048: 76.2, 67.0; 6000: 101.0, 85.7; 16384: 197.7, 195.7; 8 + 8, 2048: 110.2, 106.0; 9000: 357.5, 360.3; 2 + 2,
// 3000: 75.8, 63.6.
// Beside an adjoint of several rounds a chain of 1024 or 2048 tokens still ends in time, and half or a quarter of the sums are written
// and read (both launches, us, 512, 1024 and 2048 tokens; heads of 128, then of 64): 11500 tokens, 8 + 2: 63.0, 62.5; 13200: 78.9, 70.0, 71.2;
// 16384: 86.2, 75.5, 90.0; 32768: 152.0, 138.3, 130.3; 49152: 219.1, 190.2, 176.6; 9000, 8 + 8: 83.6, 71.1, 87.9; 16384, 8 + 8: 143.7,
// 124.4, 134.5; 16 x 1000, 8 + 2: 88.9, 79.0; but 10000, 8 + 2: 54.8, 58.6; 4 x 6000, 16 + 4: 99.4, 89.7, 99.6; 2 x 16384, 16 + 4:
// 129.5, 124.6, 120.9; 10000, 16 + 4: 47.2, 50.7.
// `slices`: workgroups that share a head's output channels.
inline int filter_gradient_chunk(long long B, int T, int heads, int slices, int dh) {
  const long long channels = B * T * heads * dh;
  const int longest = dh == 256 || channels < 16000000 ? 512 : channels < 40000000 ? 1024 : 2048;
  for (int c = longest; c > 64; c >>= 1)
    if (B * ((T + c - 1) / c) * heads * slices >= 80) return c;
  return 64;
}

// ---- prologue at d_h = 256: one head x 128 tokens per workgroup (one wavefront per SIMD) or 256 (two) -------------------
// One workgroup per CU either way.  A lone round of the 128-token form takes half of the other's time, a full one 0.55 of it, so it
// wins while one round is enough and, by how little a nearly empty last round costs, between 2 and 2.75 of its rounds, where the
// other begins a second one (8000, 8 / 2 heads: 63.7 and 82).  Full rounds of both are within 3 % of each other: us with 128 and 256
// tokens, 3000, 8 / 8: 42.7 and 43.5; 6000, 8 / 8: 86.8 and 88.8 (adjoint 81.5 and 82.7); 8000, 8 / 8: 111 and 113 (108 and 105);
// 16384, 8 / 2: 132 and 129 (119 and 119).  With many query heads to a group the small form also wins in its second round: the other
// fetches all their rows for the key head's mean straight from memory (three taps together, 5000, 6 / 1: 39.5 and 57.3; 8000, 4 / 1: 40.3
// and 51.3; 6000, 8 / 2: 48.5 and 55.5; one tap 36.3 and 43.5; the adjoint, where it did so before as well, 35.0, 36.0 and 46.2).
inline bool stream_takes_256(long long rows, int heads, int R, int taps, bool adjoint) {
  const long long wgs = (rows + 127) / 128 * heads;
  if (wgs <= 256) return false;
  if (wgs <= 512) return !(R > 3 || (adjoint && R > 2 && wgs <= 448));
  return wgs > 704 || (taps == 1 && !adjoint);
}

// ---- generic attention (fp32, other widths): rows and wavefronts of a workgroup ------------------------------------------
// 16 query rows (or keys) with up to 16 wavefronts walk a chain half as long as 32 rows with 8, but load every row of the other
// kind for half as many products: the better form while its workgroups fit one round of the chip.  Forward, 32 -> 16 rows, us
// (fp32, T, batch x query heads, d_h): 1000, 2, 32: 20.5 -> 16.8; 1000, 4, 128: 58.1 -> 48.4; 2000, 1, 32: 36.0 -> 25.4; 1000, 4, 256:
// 127 -> 98 and 700, 4, 256: 90 -> 74 (but 1500, 2, 256: 184 -> 192); two rounds lose: 700, 8, 64 not causal 0.65 of the speed, 4096, 4, 128: 366 -> 420; causal with one or two heads, where
// the second round's blocks are short, goes on to 200 blocks of 32 rows (6000, 1, 64: 1.57x; 3000, 2, 128: 1.10x; 1500, 4, 64: 0.94).
// Up to 320 keys 8 wavefronts do (64, 2, 32: 8.6 -> 6.2; beyond d_h = 64 there are never more).
// The adjoint's 16-row form is also one launch where the other is two: not causal it wins up to 128 blocks of 32 keys (d_h = 128, 128
// blocks: 1.09-1.40x, 188: 0.88-1.00), at d_h <= 64 up to 200 (1.13-1.31x, 252: 0.96-1.03), and wider than 128 up to 128, or 96 where
// several query heads share the keys (fp32, 256, 4096 keys, R = 4: 5775 -> 6294); causal, where the 32-key form's blocks are uneven, much
// further: at d_h <= 32 always, at 64 up to 6000 keys (16 heads, 4096: 1.06x, 6000: 0.97; 4 x 8192: 0.96, 4 x 16384: 0.93), in bf16 up
// to 128 always (96, 12288 keys: 1.33x, 16384: 1.13x), in fp32, where a row is read at twice the bytes, up to 4096 keys (128, 8 heads x 2048: 1.16x, x 8192:
// 0.89; 2 / R = 4 x 8192: 0.87) and not on a chip full of them (16 heads x 96 x 4096: 0.95), in any case up to 400 blocks (128, 1 x
// 12288: 1.03x; 112, 2 x 6000: 0.95-0.97), but not on one full round of many short blocks (16 heads x 512: 0.79-0.95); at 256 up to
// 200 (188: 1.12-1.19x, 252: 0.97).  Over 2092 measured sizes the choice costs 0.8 % against the better form, 5 % at most against the 32-key one.
enum GenericRows { GR_16, GR_16_WIDE, GR_32 };
inline GenericRows generic_attention_rows(long long BH, int T, int dh, bool causal) {
  const long long blocks = BH * ((T + 31) / 32);
  if (dh > 128 && T > 1000) return GR_32;
  if (blocks > 128 && !(causal && BH <= 2 && blocks <= 200)) return GR_32;
  return T > 320 && dh <= 64 ? GR_16_WIDE : GR_16;
}
inline bool generic_attention_bwd_16(long long BHk, int R, int T, int dh, bool causal, bool bf16) {
  const long long blocks = BHk * ((T + 31) / 32);
  if (!causal) return blocks <= (dh <= 64 ? 200 : dh <= 128 || R == 1 ? 128 : 96);
  if (dh > 128) return blocks <= 200;
  if (blocks > 200 && blocks <= 256 && BHk > 8) return false;
  if (dh <= 32 || blocks <= 400) return true;
  return dh <= 64 ? T <= 6000 : bf16 || (T <= 4096 && blocks <= 1504);
}

// ---- generic product: blocks of terms that a wavefront has in flight, one or four ------------------------------------------
// Its eight wavefronts take 64 terms a round, so four need 256 of them.  A small grid waits for the chain of a wavefront; a large one hides its
// loads behind more wavefronts, which four blocks' registers do not leave.  One -> four, us or the gain (tiles of 32 x 32, terms): a weight
// gradient of 48, 1000: 12.9 -> 12.4; 8 ... 256 tiles, 256 ... 2048 terms 1.03-1.10x, 384 and 512 tiles 0.99-1.10x; 1024 0.96-1.01x, 4096 0.91-0.96x;
// 64 terms 0.87-0.99x, the fewer the more tiles; 192 terms, 256 tiles 4.31 -> 4.42.
inline bool generic_product_looks_ahead(long long tiles, long long K) { return K >= 256 && tiles <= 512; }

// The two products of a projection's adjoint share a launch while four workgroups to a CU hold the tiles of both; the filter gradients
// share theirs with d_lat, a thread per element, up to twelve to a CU.  Backward pass, fp32, a launch each -> shared, us (E, H_q, H_k, d_h x tokens; number
// of workgroups of the second kind): 256, 2, 2, 32 x 64 39.1 -> 30.7, x 1000 (413) 77.3 -> 66.7, x 8192 (3134) 749 -> 741; 512, 4, 4, 32 x 4096 (3100)
// 450 -> 445; beyond it the gradients hold up d_lat: x 8192 (6200) 1337 -> 1346; 256, 4, 2, 64 x 4096 (4200) 707.9 -> 714.0.
inline bool generic_products_share(long long tiles) { return tiles <= 1024; }
inline bool generic_gradients_share(long long workgroups) { return workgroups <= 3328; }

// ---- generic prologue: tokens of a workgroup, 32 or 8 ---------------------------------------------------------------------
// The chain of a workgroup's loads before and after the convolution is four times shorter with 8 tokens, the convolution itself (32
// columns of a matrix instruction either way) takes as long: the better form while its query and key heads are one round of the grid.
// 32 -> 8 tokens, us (T, H_q + H_k, d_h, k_ch): 300, 6, 40, 1: 10.5 -> 8.7; 128, 10, 128, 2: 19.1 -> 15.8; 64, 32, 64, 2: 10.4 -> 8.9;
// beyond a round 300, 10, 128, 2: 19.2 -> 21.3; 64, 40, 128, 2: 19.1 -> 21.9.
inline bool generic_prologue_takes_8(long long B, int T, int heads) { return B * ((T + 7) / 8) * heads <= 256; }

// ---- generic filter gradients: workgroups over the rows of each unit of outputs ------------------------------------------
// About one workgroup per CU, none with fewer than 64 rows (a round of its wavefronts); the sums of the splits are added by a
// second launch, so a grid that fills the chip by itself is not split.
inline int grad_splits(long long units, long long rows) {
  const long long by_rows = (rows + 63) / 64, by_cus = 256 / (units > 0 ? units : 1);
  const long long s = by_rows < by_cus ? by_rows : by_cus;
  return s < 2 ? 1 : s > 32 ? 32 : (int)s;
}

// ---- decode attention: keys of a split -----------------------------------------------------------------------------------
// Every split but a sequence's last holds this many keys: one or two rounds of the kernel's four wavefronts, as few splits as
// leave about 1024 workgroups on the chip, at most `max_splits`.  groups = sequences x KV heads.  A wavefront of the row kernel
// (bf16, d_h 64, 128, 256) takes 8 load instructions of keys per round (4 for three and more heads to a group); one of the general
// kernel 64 keys, so fewer than 256 leave it wavefronts without any.  That pays only while most CUs are idle (4 sequences x
// 300 keys, 2 KV heads of 200, fp32, whole steps: 64 keys 58 us, 256 60); else 256 is the least (100 x 300: 197 and 154; 40 x
// 1000, 2 x 128: 86 and 73; 13 x 4000, 1 x 200: 101 and 72) and it goes on in half rounds (40 x 4000, 2 x 128: 384 keys 146, 320
// 155, 512 157).
inline int decode_keys_per_split(long long groups, int len, int dh, bool rows_kernel, int max_splits) {
  const bool whole = !rows_kernel && groups * ((len + 255) / 256) >= 64;
  const int unit = dh <= 64 ? 256 : dh <= 128 || whole ? 128 : 64, least = whole ? 256 : unit;
  const long long want = (1024 + groups - 1) / groups, most = want < max_splits ? want : max_splits;
  const int even = (int)(((len + most - 1) / most + unit - 1) / unit) * unit;
  return even > least ? even : least;
}

// Decode: the up-projection combines the splits of the attention itself?  Every one of its workgroups then reads all of them, a thread
// per four channels (2048 channels at most), which by 16 splits costs what the launch did.  Step with the launch, without, us (sequences x
// tokens): E = 2048, 8 / 2 heads of 128: 1 x 200 22.1, 21.4; 1 x 1000 (8 splits) 22.5, 22.2; 2 x 500 22.5, 21.8; 1 x 2000 (16) 23.1, 22.9;
// 2 x 2000 24.0, 24.0; 4 / 4 of 64, 8 x 1000 18.8, 18.1; 8 x 4000 (16) 22.4, 22.8; 4 / 1 of 256, 1 x 4000 29.8, 30.2.
constexpr int UP_CHANNELS = 2048;
inline bool decode_up_combines(long long B, int e_q, int nsplit, int max_splits) { return B * e_q <= UP_CHANNELS && nsplit <= max_splits; }
// Dynamic LDS of that up-projection: 32 columns of W and the B rows that multiply them, bf16, all channels in whole lines of 128; the most
// that any step asks for is that of one sequence (the lines' padding is at most 64 channels a row)
constexpr size_t decode_up_lds(long long B, int e_q) { return (size_t)((e_q + 127) / 128 * 128) * (size_t)(64 + 2 * B); }
constexpr size_t DECODE_UP_LDS = decode_up_lds(1, UP_CHANNELS);

}  // namespace cca
