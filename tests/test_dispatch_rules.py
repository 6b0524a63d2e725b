"""The dispatch rules of csrc/cca_rules.h on the CPU: the GPU tests' case lists reach every form of a kernel that the rules can
choose, and at sizes where every form was timed the chosen one is not the slower."""
import pytest

import paper_2510_04476_amd as P
import rules
import test_gpu_small_shapes as small


def test_projection_cases_reach_every_tile():
    reached = set()
    for M, Hq, Hk, dh, E in small.GEMM_CASES:
        reached |= {rules.nt_tile(M, (Hq + 2 * Hk) * dh, E), rules.nt_tile(M, E, Hq * dh)}
    assert reached == set(rules.NT_TILES)


def test_projection_cases_reach_every_order_of_tiles():
    orders = set()
    for M, Hq, Hk, dh, E in small.GEMM_CASES:
        for N, K in (((Hq + 2 * Hk) * dh, E), (E, Hq * dh)):
            tm, tn = (int(x) for x in rules.nt_tile(M, N, K).split("x"))
            tiles_n = -(-N // tn)
            panel = rules.tile_panel(-(-M // tm), tiles_n, tm, tn, K)
            assert 1 <= panel <= tiles_n
            orders.add((tm <= 64, "rows" if panel == tiles_n else "whole panels" if tiles_n % panel == 0 else "a narrower one"))
    assert {(False, "rows")} | {(small_tile, o) for small_tile in (True, False) for o in ("whole panels", "a narrower one")} <= orders


TILE_SHAPES = [(256, 256), (192, 256), (256, 192), (256, 128), (128, 128), (64, 128), (64, 64)]


def touched(tiles_m, tiles_n, tm, tn, w):
    """Rows of both operands that the first 32 tiles of each XCD's range touch, tile by tile"""
    tiles = tiles_m * tiles_n
    n = -(-tiles // 8)
    total = 0
    for a in range(0, tiles, n):
        rows, cols = 0, set()
        panels = {}
        for t in range(a, min(a + min(n, 32), tiles)):
            p, r = divmod(t, w * tiles_m)
            width = min(w, tiles_n - p * w)
            panels.setdefault(p, set()).add(r // width)
            cols.add(p * w + r % width)
        rows = sum(len(v) for v in panels.values())
        total += min(rows, tiles_m) * tm + len(cols) * tn
    return total


@pytest.mark.parametrize("tiles_m,tiles_n", [(1, 1), (1, 40), (2, 17), (3, 5), (5, 24), (7, 9), (8, 44), (19, 6), (40, 8), (64, 13)])
def test_rows_touched_by_a_panel_are_counted(tiles_m, tiles_n):
    for tm, tn in TILE_SHAPES[:4]:
        for w in range(1, tiles_n + 1):
            assert rules.panel_touches(tiles_m, tiles_n, tm, tn, w) == touched(tiles_m, tiles_n, tm, tn, w), w


def test_panels_touch_as_few_rows_as_any_width():
    for tm, tn in TILE_SHAPES:
        for tiles_m in [*range(1, 41), 63, 100, 171, 255]:
            for tiles_n in [*range(1, 34), 48, 64, 96, 177, 300]:
                cost = {w: rules.panel_touches(tiles_m, tiles_n, tm, tn, w) for w in {-(-tiles_n // p) for p in range(1, tiles_n + 1)}}
                kept = tn == 128 and tm >= 128 and 2 * min(cost.values()) > cost[tiles_n]  # the row order, by its own rule
                panel = rules.tile_panel(tiles_m, tiles_n, tm, tn, 1 << 20)
                assert panel == tiles_n if kept else cost[panel] <= 1.02 * min(cost.values()), (tiles_m, tiles_n, tm, tn, panel)


# rows, columns and terms of a product and whether it is taken row by row: what an XCD then brings in fits its 4 MB, or not
@pytest.mark.parametrize("M,N,K,by_rows", [(1024, 1280, 1024, True), (1024, 1024, 1024, True), (1024, 768, 1536, True), (512, 3072, 2048, False),
                                           (200, 6144, 2048, False), (1024, 2048, 2048, False), (300, 1536, 2048, False)])
def test_products_that_fit_an_l2_keep_their_rows(M, N, K, by_rows):
    tm, tn = (int(x) for x in rules.nt_tile(M, N, K).split("x"))
    tiles_n = -(-N // tn)
    assert (rules.tile_panel(-(-M // tm), tiles_n, tm, tn, K) == tiles_n) == by_rows


# 512 x 1536 x 2048, 512 x 2048 x 1024, 128 x 12288 x 8192, 64 x 24576 x 16384, 64 x 16384 x 8192, 1 x 65536 x 65536, and long and wide
@pytest.mark.parametrize("tiles_m,tiles_n,tm,tn", [(8, 24, 64, 64), (8, 32, 64, 64), (2, 96, 64, 128), (1, 192, 64, 128), (1, 256, 64, 64), (2, 1024, 64, 64),
                                                   (3, 1000, 64, 64), (64, 8, 256, 192), (4096, 256, 256, 256)])
def test_order_of_tiles_is_chosen_in_no_time(tiles_m, tiles_n, tm, tn):
    """It runs on the host at every launch of a product, which itself takes about 5 us."""
    assert rules.tile_panel_us(tiles_m, tiles_n, tm, tn) <= 2.0


def test_weight_gradient_cases_reach_every_tile():
    alone = [(E, 3 * Hq * dh, r) for r, Hq, dh, E in small.WGRAD_CASES]  # d W_down: no d_x is wanted
    # d W_out, where d_o is not on the matrix cores (widths that 64 does not divide) or the rule gives both a launch each
    alone += [(Hq * dh, E, r) for r, Hq, dh, E in small.WGRAD_CASES if E % 64 or not rules.gemm_pair(r, Hq * dh, E)]
    assert {rules.tn_tile(*a) for a in alone} == set(rules.TN_TILES)
    splits = {a: rules.tn_splits(*a) for a in alone if rules.tn_tile(*a) == "split"}
    assert len(set(splits.values())) >= 3 and max(splits.values()) > 16  # few and many parts to add
    assert {1, 2, 3} < {-(-a[2] // 64) for a, n in splits.items() if n == 1}  # stored directly: slabs fewer than the kernel's stages, and more


@pytest.mark.parametrize("Mo,No,K,parts", [(1536, 2048, 16384, True), (1024, 2048, 7996, True), (2048, 6144, 4096, False), (1536, 2048, 1024, False)])
def test_weight_gradients_reserve_the_parts_that_they_write(Mo, No, K, parts):
    """Sums of several splits; none where one split stores the result, or on small tiles.  The backward's workspace holds them."""
    blocks = rules.tn_part_blocks(Mo, No, K)
    assert blocks == (rules.tn_splits(Mo, No, K) * -(-Mo // 32) * -(-No // 32) if parts else 0)
    cfg = lambda B: P.CCAConfig(B=B, T=K, d_model=No, n_q_heads=Mo // 64, n_kv_heads=1, head_dim=64, flags=P.CCA_FLAGS_MHA)
    c = cfg(1)
    taken = max(blocks, rules.tn_part_blocks(No, c.n_lat, K)) * 4096
    # without the parts, every region grows with the rows alone (each rounded up to 256 bytes)
    two = [P.cca_backward_workspace_size(cfg(B)) - max(rules.tn_part_blocks(Mo, No, B * K), rules.tn_part_blocks(No, c.n_lat, B * K)) * 4096 for B in (1, 2)]
    assert P.cca_backward_workspace_size(c) >= taken and abs(two[1] - 2 * two[0]) <= 16 * 256


def test_projection_adjoint_cases_reach_every_form():
    reached = set()
    for rows, Hq, Hk, dh, E in small.PAIR_CASES:
        reached |= {rules.gemm_pair(rows, Hq * dh, E), rules.gemm_pair(rows, E, (Hq + 2 * Hk) * dh)}
    assert None in reached and {True, False} == {f[2] for f in reached if f}
    # over rows, widths and heads of the repository's layouts: no pair of forms is left out
    chosen = set()
    for rows in list(range(64, 2048, 97)) + [2048, 3000, 4096, 6000]:
        for E in (256, 512, 1024, 1536, 2048):
            for n in (128, 256, 512, 768, 1024, 1536, 2048, 3072):
                chosen |= {rules.gemm_pair(rows, n, E), rules.gemm_pair(rows, E, n)}
    forms = lambda s: {f[:2] for f in s if f}
    print(sorted(forms(chosen)), sorted(forms(reached)))
    assert forms(chosen) == forms(reached)


# rows, n_in, n_out and us of both adjoints of a projection in a launch each, and of the fastest forms of the one launch (tile of the
# first adjoint, of the second, the first one's tiles come first)
PAIR_MEASURED = [
    (4096, 768, 1536, 43.0, {("128x128", "64x128", False): 30.4, ("64x128", "64x128", False): 36.2, ("128x128", "64x64", False): 37.7}),
    (4096, 1536, 1280, 46.7, {("128x128", "128x128", False): 43.1, ("64x128", "128x128", False): 49.3, ("64x128", "64x128", False): 52.0}),
    (1999, 384, 1536, 19.0, {("64x128", "64x64", False): 12.1, ("64x128", "64x64", True): 12.2, ("64x128", "64x128", True): 14.7}),
    (1999, 1536, 640, 21.2, {("128x128", "64x128", False): 16.5, ("64x128", "64x128", False): 18.4, ("128x128", "64x64", True): 18.8}),
    (2600, 2048, 768, 32.4, {("128x128", "64x128", False): 27.8, ("128x128", "128x128", False): 29.0, ("64x128", "64x128", False): 32.1}),
    (8192, 384, 1536, 42.9, {("128x128", "64x64", False): 36.1, ("64x128", "64x64", False): 43.5, ("64x64", "64x128", False): 47.3}),
    (5000, 512, 1024, 34.9, {("128x128", "64x64", False): 23.4, ("64x128", "64x64", False): 24.4, ("64x64", "64x64", False): 26.9}),
    (6000, 512, 2048, 48.1, {("128x128", "64x128", False): 37.7, ("64x128", "64x128", False): 38.0, ("128x128", "64x64", False): 44.8}),
    (512, 2048, 3072, 29.5, {("64x128", "128x128", True): 22.8, ("64x128", "128x128", False): 26.6, ("64x64", "128x128", True): 26.9}),
    (8192, 1536, 1536, 86.3, {("128x128", "128x128", False): 108.5, ("64x128", "128x128", False): 110.7, ("128x128", "64x128", False): 112.0}),
    (8192, 1024, 2048, 78.4, {("128x128", "128x128", False): 82.1, ("128x128", "64x128", False): 91.6, ("64x128", "128x128", False): 92.3}),
    (2600, 1536, 1280, 35.7, {("128x128", "128x128", False): 29.4, ("128x128", "64x128", True): 32.8, ("128x128", "64x128", False): 33.3}),
    (1024, 2048, 1536, 24.9, {("64x128", "128x128", False): 22.6, ("64x128", "128x128", True): 23.5, ("128x128", "64x128", False): 23.8, ("128x128", "64x128", True): 24.0, ("128x128", "128x128", True): 24.3}),
    (512, 1024, 2048, 16.2, {("64x64", "128x128", True): 10.3, ("64x64", "128x128", False): 10.4, ("64x64", "64x128", True): 12.0}),
    (3000, 1024, 1024, 28.2, {("128x128", "64x128", False): 22.0, ("64x128", "64x128", False): 23.7, ("128x128", "64x64", True): 25.3}),
    (300, 768, 1536, 13.3, {("64x64", "128x128", False): 8.2, ("64x64", "128x128", True): 8.2, ("64x64", "64x128", True): 8.3, ("64x64", "64x128", False): 8.3, ("64x64", "64x64", True): 8.3}),
]


@pytest.mark.parametrize("rows,n_in,n_out,two_us,one_us", PAIR_MEASURED)
def test_projection_adjoints_form_is_the_fastest(rows, n_in, n_out, two_us, one_us):
    """Within 6 %: the fits' own errors (3 % and 5 % rms) decide between forms that are closer than that."""
    form = rules.gemm_pair(rows, n_in, n_out)
    assert (one_us.get(form, 1e9) if form else two_us) <= 1.06 * min(two_us, *one_us.values()), form


def test_combining_up_projection_fits_the_lds_it_declares():
    for dh in (64, 128, 256):  # the widths whose attention leaves splits to combine
        for e_q in range(dh, 4097, dh):
            for B in range(1, 80):
                if rules.decode_up_combines(B, e_q, 8):
                    # 64 bytes of W and 2 of each row for every channel, in lines of 128
                    assert rules.decode_up_lds(B, e_q) == -(-e_q // 128) * 128 * (64 + 2 * B) <= rules.decode_up_lds_limit(), (B, e_q)
    assert rules.decode_up_combines(1, 2048, 8) and rules.decode_up_lds_limit() + 1024 <= 160 * 1024


def test_attention_cases_reach_both_block_orders():
    paired = {(causal, rules.pair_blocks(B * Hq, causal, -(-T // 128))) for B, T, Hq, Hk, dh, causal, normed in small.SPLIT_CASES}
    assert paired == {(True, True), (True, False), (False, False)}


def test_attention_cases_reach_both_block_heights():
    assert {rules.fwd_takes_64_rows(B * Hq, T, normed) for B, T, Hq, Hk, dh, causal, normed in small.SPLIT_CASES} == {True, False}


def test_wide_head_prologue_cases_reach_both_forms():
    reached = set()
    for B, T, Hq, Hk, k_seq, k_ch in small.STREAM_CASES:
        for adjoint in (False, True):
            taps = k_seq + k_ch - 1
            reached.add((taps, adjoint, rules.stream_takes_256(B * T, Hq + Hk, Hq // Hk, taps, adjoint)))
    assert reached == {(taps, adjoint, wide) for taps in (1, 2, 3) for adjoint in (False, True) for wide in (False, True)}


def test_prologue_cases_reach_both_forms():
    reached = set()
    for B, T, Hq, Hk, k_seq, k_ch, dh in small.PROLOGUE_CASES:
        for adjoint in (False, True):
            reached.add((dh, k_seq + k_ch - 1, adjoint, rules.prologue_is_short(B * T, Hq + Hk, Hq // Hk, dh, adjoint)))
    assert reached == {(dh, taps, adjoint, short) for dh in (64, 128) for taps in (1, 2, 3) for adjoint in (False, True) for short in (False, True)}


# rows, query and KV heads, d_h, adjoint and us of the short and of the long form
PROLOGUE_MEASURED = [(512, 8, 2, 128, False, 12.4, 18.8), (3000, 8, 2, 128, False, 19.1, 20.0), (4593, 8, 2, 128, False, 25.5, 21.2),
                     (3000, 4, 4, 128, False, 19.0, 16.9), (2048, 4, 4, 128, False, 13.3, 16.7), (1024, 32, 8, 128, False, 26.5, 23.3),
                     (2048, 16, 4, 64, False, 12.1, 12.6), (3000, 16, 4, 64, False, 14.9, 14.1), (3000, 8, 8, 64, False, 13.2, 12.1),
                     (1024, 8, 2, 128, True, 35.7, 38.5), (2048, 8, 2, 128, True, 48.6, 47.2), (2048, 4, 4, 128, True, 41.5, 39.1),
                     (3000, 16, 4, 64, True, 36.0, 37.8), (7996, 16, 4, 64, True, 56.6, 56.0)]


@pytest.mark.parametrize("rows,Hq,Hk,dh,adjoint,short_us,long_us", PROLOGUE_MEASURED)
def test_prologue_form_is_the_faster(rows, Hq, Hk, dh, adjoint, short_us, long_us):
    assert rules.prologue_is_short(rows, Hq + Hk, Hq // Hk, dh, adjoint) == (short_us < long_us)


def test_generic_cases_reach_every_form():
    rows, bwd, splits = set(), set(), set()
    for c in small.GENERIC_CASES:
        for causal in (False, True):
            rows.add(rules.generic_attention_rows(c["B"] * c["Hq"], c["T"], c["dh"], causal))
            bwd.add(rules.generic_attention_bwd_16(c["B"] * c["Hk"], c["Hq"] // c["Hk"], c["T"], c["dh"], causal, False))
        tiles = -(-c["dh"] // 32)
        splits.add(rules.grad_splits(tiles * tiles * (c["Hq"] + c["Hk"]) * c["k_ch"], c["B"] * c["T"]))
    assert rows == set(rules.GENERIC_ROWS) and bwd == {True, False}
    assert {(rules.generic_prologue_takes_8(c["B"], c["T"], c["Hq"] + c["Hk"]), c["dh"] <= 16, c["dh"] <= 32) for c in small.GENERIC_CASES} == {
        (few, *narrow) for few in (True, False) for narrow in ((True, True), (False, True), (False, False))}
    assert 1 in splits and 2 in splits and max(splits) >= 16


# tiles, terms and us of the generic product with one block of terms in flight, with four
@pytest.mark.parametrize("tiles,K,one,four", [(48, 1000, 12.9, 12.4), (192, 1024, 11.1, 10.6), (256, 512, 6.8, 6.5), (256, 192, 4.31, 4.42), (1024, 64, 5.1, 5.7),
                                              (1536, 256, 15.6, 16.8), (2048, 1024, 62.1, 63.2), (3072, 512, 47.8, 50.6)])
def test_generic_product_form_is_the_faster(tiles, K, one, four):
    assert rules.generic_product_looks_ahead(tiles, K) == (four < one)


def test_generic_cases_reach_both_products():
    tiles = lambda m, n: -(-m // 32) * -(-n // 32)
    ahead = set()
    for c in small.GENERIC_CASES:
        rows, n_lat = c["B"] * c["T"], (c["Hq"] + 2 * c["Hk"]) * c["dh"]
        ahead |= {(False, rules.generic_product_looks_ahead(tiles(rows, n_lat), c["E"])), (True, rules.generic_product_looks_ahead(tiles(c["E"], n_lat), rows))}
    assert ahead == {(transposed, four) for transposed in (False, True) for four in (False, True)}


def test_generic_cases_share_launches_and_do_not():
    tiles = lambda m, n: -(-m // 32) * -(-n // 32)
    products, gradients = set(), set()
    for c in small.GENERIC_CASES:
        rows, e_q, n_lat = c["B"] * c["T"], c["Hq"] * c["dh"], (c["Hq"] + 2 * c["Hk"]) * c["dh"]
        products |= {rules.generic_products_share(tiles(n_in, n_out) + tiles(rows, n_in)) for n_in, n_out in ((e_q, c["E"]), (c["E"], n_lat))}
        gradients.add(rules.generic_gradients_share(-(-rows * n_lat // 512)))
    assert products == {True, False} and gradients == {True, False}


@pytest.mark.parametrize("a,b,shared", [(4096, 4096, True), (4096, 4096 + 16, True), (4096 + 16, 4096, True), (4096, 4096 + 64, False), (4096 + 64, 4096, False),
                                        (4096, 4096 + 48, True), (4096 + 48, 4096, True), (0x7F0000000000, 4096, False)])
def test_overlapping_buffers_are_found(a, b, shared):
    assert rules.overlap(a, 64, b, 64) == shared


def test_filter_gradient_cases_reach_every_long_chunk():
    chunk = lambda B, T, Hq, Hk, k_seq, k_ch, dh: rules.filter_gradient_chunk(B, T, Hq + Hk, 1, dh)
    got = [(chunk(*c), c[1]) for c in small.FILTER_GRADIENT_CASES]
    assert {c for c, T in got} == {512, 1024, 2048}
    assert {c for c, T in got if T % c} == {512, 1024, 2048} and any(T < c for c, T in got)  # short last chunks, sequences shorter than one


# sequences, T, heads, d_h and us of the prologue's adjoint with chunks of 512, 1024 and (where timed) 2048 tokens
@pytest.mark.parametrize("B,T,heads,dh,us", [(1, 10000, 10, 128, (54.8, 58.6)), (1, 13200, 10, 128, (78.9, 70.0, 71.2)), (1, 16384, 10, 128, (86.2, 75.5, 90.0)),
                                             (1, 32768, 10, 128, (152.0, 138.3, 130.3)), (1, 49152, 10, 128, (219.1, 190.2, 176.6)), (1, 9000, 16, 128, (83.6, 71.1, 87.9)),
                                             (1, 16384, 16, 128, (143.7, 124.4, 134.5)), (16, 1000, 10, 128, (88.9, 79.0)), (1, 10000, 20, 64, (47.2, 50.7)),
                                             (4, 6000, 20, 64, (99.4, 89.7, 99.6)), (2, 16384, 20, 64, (129.5, 124.6, 120.9))])
def test_filter_gradient_chunk_is_the_fastest(B, T, heads, dh, us):
    assert us[(512, 1024, 2048).index(rules.filter_gradient_chunk(B, T, heads, 1, dh))] == min(us)


# T, query and key heads and us of the prologue with 32 tokens a workgroup, with 8
@pytest.mark.parametrize("T,heads,us32,us8", [(300, 6, 10.5, 8.7), (128, 10, 19.1, 15.8), (64, 32, 10.4, 8.9), (300, 10, 19.2, 21.3), (64, 40, 19.1, 21.9)])
def test_generic_prologue_form_is_the_faster(T, heads, us32, us8):
    assert rules.generic_prologue_takes_8(1, T, heads) == (us8 < us32)


# T, batch x query heads, d_h, causal and us of 32 rows, of 16
GENERIC_MEASURED = [(1000, 2, 32, True, 20.5, 16.8), (1000, 4, 128, True, 58.1, 48.4), (2000, 1, 32, True, 36.0, 25.4),
                    (4096, 4, 128, True, 366.0, 420.0), (4096, 4, 64, False, 246.0, 257.2), (4096, 4, 256, False, 854.1, 1286.9)]


@pytest.mark.parametrize("T,BH,dh,causal,us32,us16", GENERIC_MEASURED)
def test_generic_attention_form_is_the_faster(T, BH, dh, causal, us32, us16):
    assert (rules.generic_attention_rows(BH, T, dh, causal) == "32 rows") == (us32 < us16)


# T, batch x KV heads, query heads to each, d_h, causal, bf16 and us of the adjoint in 32-row blocks, in 16-row ones
GENERIC_BWD_MEASURED = [(4096, 1, 4, 256, False, False, 5774.8, 6294.3), (4096, 1, 1, 256, False, False, 1762.1, 1447.6), (4096, 1, 4, 200, False, False, 5869.0, 6616.1),
                        (1536, 2, 4, 256, False, False, 2267.7, 1803.5), (3000, 2, 1, 256, False, False, 1381.6, 1763.2), (512, 16, 1, 128, True, False, 152.5, 189.1),
                        (512, 16, 2, 64, True, False, 136.6, 145.4), (1000, 8, 4, 128, True, False, 978.9, 879.1), (16384, 1, 1, 128, True, False, 4061.8, 4675.9),
                        (8192, 2, 4, 128, True, False, 8840.6, 10151.7), (8192, 2, 4, 112, True, False, 8888.3, 10566.8), (2048, 8, 1, 128, True, False, 954.6, 823.2),
                        (12288, 1, 1, 128, True, False, 2778.1, 2688.7), (16384, 4, 1, 64, True, False, 7206.6, 7713.1), (16384, 4, 1, 40, True, True, 7368.2, 7715.2),
                        (4096, 16, 1, 64, True, False, 2360.3, 2228.6), (6000, 4, 1, 64, True, False, 1181.4, 1097.6), (16384, 8, 1, 32, True, False, 8064.0, 7959.1),
                        (4096, 16, 1, 96, True, False, 5075.3, 5328.5), (6000, 1, 4, 256, True, False, 9957.3, 8961.6), (4096, 2, 4, 256, True, False, 7607.7, 8631.8)]


@pytest.mark.parametrize("T,BHk,R,dh,causal,bf16,us32,us16", GENERIC_BWD_MEASURED)
def test_generic_attention_adjoint_form_is_the_faster(T, BHk, R, dh, causal, bf16, us32, us16):
    assert rules.generic_attention_bwd_16(BHk, R, T, dh, causal, bf16) == (us16 < us32)


# M, N, K and us of each tile shape in the order of rules.NT_TILES
NT_MEASURED = [
    (4593, 4096, 4096, (156.4, 130.7, 327.7, 247.6, 197.6, 157.0, 135.0, 155.3)),
    (6000, 2048, 4096, (81.5, 122.1, 190.0, 147.8, 120.0, 104.1, 74.2, 101.0)),
    (12000, 2048, 4096, (169.4, 194.0, 448.8, 338.2, 253.9, 177.7, 155.8, 179.1)),
    (12000, 1536, 4096, (159.9, 136.9, 308.0, 232.4, 196.6, 144.0, 139.9, 122.6)),
    (2048, 4096, 4096, (76.7, 62.9, 125.4, 97.3, 78.3, 53.2, 66.8, 59.2)),
    (6000, 3072, 3072, (120.3, 105.7, 227.9, 174.4, 147.0, 110.0, 106.1, 92.0)),
    (512, 2048, 128, (8.2, 6.8, 3.6, 4.3, 4.5, 5.3, 6.8, 5.8)),
    (512, 1536, 2048, (36.3, 29.0, 9.8, 13.7, 19.1, 21.5, 29.7, 23.8)),
    (16384, 1536, 2048, (95.8, 85.0, 238.3, 173.8, 137.3, 97.0, 110.0, 97.8)),
    (4096, 2048, 4096, (76.6, 63.1, 125.6, 97.8, 79.6, 54.2, 68.2, 58.9)),
    (6000, 2048, 1024, (27.8, 39.0, 63.4, 48.0, 36.8, 31.7, 24.8, 32.3)),
    (4593, 1536, 2048, (39.9, 32.2, 58.8, 51.9, 40.4, 27.6, 34.7, 28.2)),
    (4096, 2048, 2048, (40.7, 34.6, 68.5, 53.8, 43.0, 29.8, 37.1, 32.6)),
    (1000, 1536, 2048, (36.5, 28.9, 18.0, 14.2, 19.4, 21.7, 29.9, 23.8)),
    (2000, 1536, 2048, (36.8, 29.5, 26.4, 26.7, 20.4, 22.5, 30.3, 24.3)),
    (12000, 1536, 2048, (85.6, 76.1, 159.2, 121.3, 103.8, 74.5, 76.5, 64.4)),
    (12000, 1536, 3072, (122.7, 109.7, 246.3, 182.6, 158.8, 110.5, 109.0, 95.0)),
    (16384, 3072, 4096, (277.7, 300.6, 825.6, 625.7, 489.4, 335.0, 358.9, 335.6)),
    (8192, 1536, 4096, (83.3, 76.3, 222.9, 154.6, 125.5, 107.9, 125.0, 109.8)),
    (9000, 3072, 3072, (137.3, 164.5, 366.3, 280.5, 220.3, 164.4, 159.0, 139.4)),
    (16384, 4096, 4096, (378.8, 429.5, 1183.5, 895.6, 653.1, 457.7, 440.8, 456.5)),
    (8192, 8192, 8192, (714.9, 816.5, 2035.7, 1574.5, 1207.5, 832.8, 819.0, 880.5)),
    (7000, 1920, 4096, (87.7, 123.7, 216.0, 173.8, 153.2, 106.8, 129.0, 108.0)),
    (10000, 3840, 3072, (197.3, 207.1, 492.9, 407.4, 304.0, 210.3, 217.8, 213.6)),
]


@pytest.mark.parametrize("M,N,K,us", NT_MEASURED)
def test_projection_tile_is_the_fastest(M, N, K, us):
    """Within 6 %: the fit's own error (11 % rms) decides between shapes that are closer than that."""
    assert len(us) == len(rules.NT_TILES)
    assert us[rules.NT_TILES.index(rules.nt_tile(M, N, K))] <= 1.06 * min(us)


# M, N, K, tile and us of an attention adjoint with three products behind it, whose workgroups start without a pause, with two, with four
@pytest.mark.parametrize("M,N,K,tile,us", [(12288, 1536, 1280, "192x192", (1210.9, 1130.3, 1075.1)), (16384, 1536, 2048, "256x192", (1318.6, 1172.6, 1176.9)),
                                           (6144, 2048, 2048, "192x256", (1109.9, 1059.0, 1060.8)), (10000, 1536, 1280, "192x256", (1129.7, 1080.5, 1085.6))])
def test_products_start_with_the_pauses_that_keep_the_clock(M, N, K, tile, us):
    tm, tn = (int(x) for x in tile.split("x"))
    assert us[(0, 2, 4).index(rules.start_pauses(tm * tn, -(-M // tm) * -(-N // tn), K // 64))] == min(us)


def test_projection_cases_start_with_every_number_of_pauses():
    reached = set()
    for M, Hq, Hk, dh, E in small.GEMM_CASES:
        for N, K in (((Hq + 2 * Hk) * dh, E), (E, Hq * dh)):
            tm, tn = (int(x) for x in rules.nt_tile(M, N, K).split("x"))
            if tm * tn >= 256 * 128:
                reached.add(rules.start_pauses(tm * tn, -(-M // tm) * -(-N // tn), K // 64))
    assert reached == {0, 2, 4}


# Mo, No, tokens and us of the small tiles (in the order of rules.TN_TILES[1:]) and of the best split
TN_MEASURED = [(2048, 2048, 8000, (116.7, 105.6, 82.3), 69.8), (2048, 2048, 4000, (58.6, 55.1, 42.5), 46.7), (2048, 1536, 8000, (89.9, 98.4, 72.8), 57.9),
               (1024, 2048, 8000, (57.3, 52.7, 70.3), 45.1), (2048, 6144, 4000, (173.2, 165.6, 122.2), 90.8), (1024, 2048, 1024, (11.0, 10.2, 12.4), 23.7),
               (1536, 1280, 4096, (30.2, 27.6, 37.7), 32.2), (768, 1536, 4096, (29.3, 26.3, 37.0), 27.2), (1536, 640, 2100, (12.0, 15.6, 21.4), 23.2),
               (384, 1536, 2100, (11.7, 15.4, 21.8), 20.1), (2048, 1536, 1024, (15.5, 17.9, 13.0), 24.0), (2048, 1536, 16384, (210.1, 213.2, 149.9), 97.6)]


@pytest.mark.parametrize("Mo,No,K,small_us,split_us", TN_MEASURED)
def test_weight_gradient_form_is_the_fastest(Mo, No, K, small_us, split_us):
    us = dict(zip(rules.TN_TILES[1:], small_us), split=split_us)
    assert us[rules.tn_tile(Mo, No, K)] <= 1.06 * min(us.values())


# B * H_q, T, causal and us on one and on two groups of wavefronts (d_h = 64 or 128)
FWD_MEASURED = [(8, 64, True, 4.4, 5.4), (8, 128, True, 8.2, 9.4), (96, 400, True, 10.8, 15.6), (128, 400, True, 17.9, 25.2),
                (64, 640, True, 12.7, 14.1), (64, 777, True, 16.2, 18.5), (128, 640, False, 40.6, 57.6), (96, 1280, True, 54.5, 72.3),
                (8, 200, True, 12.3, 10.1), (8, 2048, True, 47.6, 33.6), (24, 1531, True, 26.6, 19.4), (16, 4096, True, 101.8, 81.8),
                (16, 512, False, 19.4, 15.5), (64, 1999, True, 44.7, 54.7), (8, 16384, True, 446.0, 501.0)]
DQ_MEASURED = [(128, 300, True, 36.8, 38.8), (128, 777, True, 147.8, 155.3), (8, 2048, True, 180.0, 156.0), (24, 1531, True, 95.0, 83.0),
               (64, 1999, True, 174.0, 181.0), (64, 6000, False, 2083.6, 2246.0), (24, 8192, False, 1417.0, 1528.6)]
DKDV_MEASURED = [(64, 1531, True, 104.5, 115.3), (4, 64, True, 13.0, 13.9), (8, 2048, True, 180.0, 139.0), (24, 1531, True, 95.0, 78.0),
                 (64, 1999, True, 174.0, 185.0)]


@pytest.mark.parametrize("rule,cases", [(rules.fwd_splits_keys, FWD_MEASURED), (rules.dq_splits_keys, DQ_MEASURED),
                                        (rules.dkdv_splits_rows, DKDV_MEASURED)])
def test_attention_split_is_the_faster_form(rule, cases):
    wrong = [(BH, T, causal) for BH, T, causal, one, two in cases if rule(BH, T, causal) != (two < one)]
    assert not wrong, wrong


# rows, query heads, KV heads, taps, adjoint and us with 128 and 256 tokens per workgroup
STREAM_MEASURED = [(4096, 6, 2, 3, False, 31.3, 46.7), (6000, 4, 1, 3, False, 29.5, 49.0), (8192, 6, 2, 3, False, 57.4, 50.1),
                   (9000, 6, 2, 3, False, 70.5, 79.5), (12288, 6, 2, 3, False, 85.1, 81.1), (16384, 6, 2, 3, False, 113.8, 92.1),
                   (32768, 6, 2, 3, False, 233.0, 200.5), (3000, 8, 8, 3, False, 47.9, 41.2), (16384, 8, 8, 3, False, 261.2, 222.7),
                   (32768, 1, 1, 3, False, 62.0, 49.5), (12288, 2, 2, 3, False, 47.6, 41.9), (16384, 4, 1, 1, False, 54.6, 51.0),
                   (12288, 6, 2, 1, False, 65.1, 54.2), (7000, 6, 2, 3, True, 43.6, 46.0), (8192, 6, 2, 3, True, 50.3, 47.4),
                   (12288, 4, 1, 3, True, 45.7, 50.5), (14000, 2, 2, 3, True, 48.6, 42.3), (16384, 6, 2, 3, True, 98.2, 86.9)]


def test_wide_head_prologue_takes_the_faster_form():
    wrong = [c for c in STREAM_MEASURED if rules.stream_takes_256(c[0], c[1] + c[2], c[1] // c[2], c[3], c[4]) != (c[6] < c[5])]
    assert not wrong, wrong


@pytest.mark.parametrize("groups,keys,dh,faster", [(80, 1000, 128, 256), (200, 300, 200, 256), (13, 4000, 200, 256), (80, 4000, 128, 384),
                                                   (8, 300, 200, 64), (200, 300, 96, 256)])
def test_general_decode_kernel_has_keys_for_its_wavefronts(groups, keys, dh, faster):
    """The general kernel's four wavefronts take 64 keys each; sizes of splits that measured faster than half or double."""
    assert rules.decode_keys_per_split(groups, keys, dh, False) == faster


def test_decode_splits_cover_the_keys():
    for groups in (1, 2, 13, 80, 1000):
        for keys in (1, 63, 64, 65, 255, 256, 257, 1000, 4097, 16384, 1 << 20):
            for dh in (8, 64, 96, 128, 200, 256):
                for rows_kernel in (False, True):
                    per = rules.decode_keys_per_split(groups, keys, dh, rows_kernel)
                    assert per > 0 and -(-keys // per) <= 32 and (-(-keys // per) - 1) * per < keys
