"""The library's dispatch rules (csrc/cca_rules.h), compiled for the host, so that a test can ask which form of a kernel serves
a size instead of keeping a copy of the rule."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <chrono>

#include "cca_rules.h"
using namespace cca;
extern "C" {
int r_nt_tile(long long M, int N, int K) { return nt_tile(M, N, K); }
int r_tn_tile(int Mo, int No, long long K) { return tn_tile(Mo, No, K); }
int r_tn_splits(int Mo, int No, long long K) { return tn_splits(Mo, No, K); }
int r_tn_part_blocks(int Mo, int No, long long K) { return (int)tn_part_blocks(Mo, No, K); }
int r_prologue_is_short(long long rows, int heads, int R, int dh, int adjoint) { return prologue_is_short(rows, heads, R, dh, adjoint); }
int r_tile_panel(int tiles_m, int tiles_n, int tm, int tn, long long K) { return tile_panel(tiles_m, tiles_n, tm, tn, K); }
int r_panel_touches(int tiles_m, int tiles_n, int tm, int tn, int w) { return TilePanel(tiles_m, tiles_n, tm, tn).touched(w); }
double r_tile_panel_us(int tiles_m, int tiles_n, int tm, int tn) {  // of one choice: the fastest of ten batches
  double least = 1e9;
  for (int batch = 0; batch < 10; ++batch) {
    volatile int sum = 0;
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 20; ++i) sum = sum + tile_panel(tiles_m, tiles_n, tm, tn, 1 << 20);
    const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() * 1e6 / 20;
    least = us < least ? us : least;
  }
  return least;
}
int r_decode_up_combines(long long B, int e_q, int nsplit) { return decode_up_combines(B, e_q, nsplit, 8); }
int r_decode_up_lds(long long B, int e_q) { return (int)decode_up_lds(B, e_q); }
int r_decode_up_lds_limit() { return (int)DECODE_UP_LDS; }
int r_fwd_takes_64_rows(long long BH, int T, int normed) { return fwd_takes_64_rows(BH, T, normed); }
int r_fwd_splits_keys(long long BH, int T, int causal) { return fwd_splits_keys(BH, T, causal); }
int r_dq_splits_keys(long long BH, int T, int causal) { return dq_splits_keys(BH, T, causal); }
int r_dkdv_splits_rows(long long BH, int T, int causal) { return dkdv_splits_rows(BH, T, causal); }
int r_decode_keys_per_split(long long groups, int len, int dh, int rows_kernel) { return decode_keys_per_split(groups, len, dh, rows_kernel, 32); }
int r_stream_takes_256(long long rows, int heads, int R, int taps, int adjoint) { return stream_takes_256(rows, heads, R, taps, adjoint); }
int r_generic_attention_rows(long long BH, int T, int dh, int causal) { return generic_attention_rows(BH, T, dh, causal); }
int r_generic_product_looks_ahead(long long tiles, long long K) { return generic_product_looks_ahead(tiles, K); }
int r_generic_products_share(long long tiles) { return generic_products_share(tiles); }
int r_generic_gradients_share(long long workgroups) { return generic_gradients_share(workgroups); }
int r_generic_prologue_takes_8(long long B, int T, int heads) { return generic_prologue_takes_8(B, T, heads); }
int r_generic_attention_bwd_16(long long BHk, int R, int T, int dh, int causal, int bf16) { return generic_attention_bwd_16(BHk, R, T, dh, causal, bf16); }
int r_grad_splits(long long units, long long rows) { return grad_splits(units, rows); }
int r_gemm_pair(long long rows, int n_in, int n_out) {
  const PairForm f = gemm_pair(rows, n_in, n_out);
  return f.one_launch ? 1 + f.nt_first + 2 * f.nt + 32 * f.tn : 0;
}
int r_filter_gradient_chunk(long long B, int T, int heads, int slices, int dh) { return filter_gradient_chunk(B, T, heads, slices, dh); }
int r_start_pauses(int area, long long tiles, long long slabs) { return start_pauses(area, tiles, slabs); }
int r_overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes) { return overlap(a, a_bytes, b, b_bytes); }
int r_pair_blocks(long long BH, int causal, int blocks) { return pair_blocks(BH, causal, blocks); }
}
"""
NT_TILES = ("256x256", "256x192", "64x64", "64x128", "128x128", "256x128", "192x256", "192x192")
GENERIC_ROWS = ("16 rows", "16 rows, 16 wavefronts", "32 rows")
TN_TILES = ("split", "64x64", "64x128", "128x128")


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                        os.path.join(ROOT, "paper_2510_04476_amd", "csrc"), src, "-o", so], check=True)
        lib = C.CDLL(so)
    L, I = C.c_longlong, C.c_int
    for name, args in dict(r_nt_tile=[L, I, I], r_tn_tile=[I, I, L], r_tn_splits=[I, I, L], r_tn_part_blocks=[I, I, L], r_fwd_splits_keys=[L, I, I], r_fwd_takes_64_rows=[L, I, I], r_decode_up_combines=[L, I, I], r_decode_up_lds=[L, I], r_decode_up_lds_limit=[], r_tile_panel=[I, I, I, I, L], r_panel_touches=[I, I, I, I, I], r_tile_panel_us=[I, I, I, I], r_prologue_is_short=[L, I, I, I, I],
                           r_filter_gradient_chunk=[L, I, I, I, I], r_start_pauses=[I, L, L], r_overlap=[C.c_void_p, C.c_size_t, C.c_void_p, C.c_size_t], r_dq_splits_keys=[L, I, I], r_dkdv_splits_rows=[L, I, I], r_pair_blocks=[L, I, I],
                           r_stream_takes_256=[L, I, I, I, I], r_generic_attention_rows=[L, I, I, I],
                           r_generic_attention_bwd_16=[L, I, I, I, I, I], r_generic_prologue_takes_8=[L, I, I], r_generic_products_share=[L], r_generic_gradients_share=[L], r_generic_product_looks_ahead=[L, L], r_grad_splits=[L, L], r_gemm_pair=[L, I, I],
                           r_decode_keys_per_split=[L, I, I, I]).items():
        getattr(lib, name).argtypes = args
    lib.r_tile_panel_us.restype = C.c_double
    return lib


def nt_tile(M, N, K):
    return NT_TILES[_lib().r_nt_tile(M, N, K)]


def tn_tile(Mo, No, K):
    return TN_TILES[_lib().r_tn_tile(Mo, No, K)]


def tn_part_blocks(Mo, No, K):
    return _lib().r_tn_part_blocks(Mo, No, K)


def tn_splits(Mo, No, K):
    return _lib().r_tn_splits(Mo, No, K)


def prologue_is_short(rows, heads, R, dh, adjoint):
    return bool(_lib().r_prologue_is_short(rows, heads, R, dh, adjoint))


def tile_panel(tiles_m, tiles_n, tm, tn, K):
    return _lib().r_tile_panel(tiles_m, tiles_n, tm, tn, K)


def panel_touches(tiles_m, tiles_n, tm, tn, width):
    return _lib().r_panel_touches(tiles_m, tiles_n, tm, tn, width)


def tile_panel_us(tiles_m, tiles_n, tm, tn):
    return _lib().r_tile_panel_us(tiles_m, tiles_n, tm, tn)


def decode_up_combines(B, e_q, nsplit):
    return bool(_lib().r_decode_up_combines(B, e_q, nsplit))


def decode_up_lds(B, e_q):
    return _lib().r_decode_up_lds(B, e_q)


def decode_up_lds_limit():
    return _lib().r_decode_up_lds_limit()


def fwd_takes_64_rows(BH, T, normed):
    return bool(_lib().r_fwd_takes_64_rows(BH, T, normed))


def fwd_splits_keys(BH, T, causal):
    return bool(_lib().r_fwd_splits_keys(BH, T, causal))


def dq_splits_keys(BH, T, causal):
    return bool(_lib().r_dq_splits_keys(BH, T, causal))


def dkdv_splits_rows(BH, T, causal):
    return bool(_lib().r_dkdv_splits_rows(BH, T, causal))


def pair_blocks(BH, causal, blocks):
    return bool(_lib().r_pair_blocks(BH, causal, blocks))


def stream_takes_256(rows, heads, R, taps, adjoint):
    return bool(_lib().r_stream_takes_256(rows, heads, R, taps, adjoint))


def decode_keys_per_split(groups, keys, dh, rows_kernel):
    return _lib().r_decode_keys_per_split(groups, keys, dh, rows_kernel)


def generic_product_looks_ahead(tiles, K):
    return bool(_lib().r_generic_product_looks_ahead(tiles, K))


def generic_products_share(tiles):
    return bool(_lib().r_generic_products_share(tiles))


def generic_gradients_share(workgroups):
    return bool(_lib().r_generic_gradients_share(workgroups))


def filter_gradient_chunk(B, T, heads, slices, dh):
    return _lib().r_filter_gradient_chunk(B, T, heads, slices, dh)


def start_pauses(area, tiles, slabs):
    return _lib().r_start_pauses(area, tiles, slabs)


def overlap(a, a_bytes, b, b_bytes):
    return bool(_lib().r_overlap(a, a_bytes, b, b_bytes))


def generic_prologue_takes_8(B, T, heads):
    return bool(_lib().r_generic_prologue_takes_8(B, T, heads))


def generic_attention_rows(BH, T, dh, causal):
    return GENERIC_ROWS[_lib().r_generic_attention_rows(BH, T, dh, causal)]


def generic_attention_bwd_16(BHk, R, T, dh, causal, bf16):
    return bool(_lib().r_generic_attention_bwd_16(BHk, R, T, dh, causal, bf16))


def grad_splits(units, rows):
    return _lib().r_grad_splits(units, rows)


def gemm_pair(rows, n_in, n_out):
    """None (a launch each) or (tile of the first adjoint, tile of the second, the first one's tiles come first)"""
    f = _lib().r_gemm_pair(rows, n_in, n_out)
    return (NT_TILES[(f - 1) // 2 % 16], TN_TILES[(f - 1) // 32], bool((f - 1) % 2)) if f else None
