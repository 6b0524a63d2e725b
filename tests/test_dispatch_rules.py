"""The dispatch rules of csrc/cca_rules.h on the CPU: the GPU tests' case lists reach every form of a kernel that the rules can
choose, and at sizes where every form was timed the chosen one is not the slower."""
import pytest

import rules
import test_gpu_small_shapes as small


def test_projection_cases_reach_every_tile():
    reached = set()
    for M, Hq, Hk, dh, E in small.GEMM_CASES:
        reached |= {rules.nt_tile(M, (Hq + 2 * Hk) * dh, E), rules.nt_tile(M, E, Hq * dh)}
    assert reached == set(rules.NT_TILES)


def test_weight_gradient_cases_reach_every_tile():
    forms = {(r, Hq, dh, E): rules.tn_tile(Hq * dh, E, r) for r, Hq, dh, E in small.WGRAD_CASES}
    assert set(forms.values()) == set(rules.TN_TILES)
    splits = {rules.tn_splits(Hq * dh, E, r) for (r, Hq, dh, E), f in forms.items() if f == "split"}
    assert len(splits) >= 3 and max(splits) > 16  # few and many parts to add


def test_attention_cases_reach_both_block_orders():
    paired = {(causal, rules.pair_blocks(B * Hq, causal, -(-T // 128))) for B, T, Hq, Hk, dh, causal, normed in small.SPLIT_CASES}
    assert paired == {(True, True), (True, False), (False, False)}


# M, N, K and us of each tile shape in the order of rules.NT_TILES
NT_MEASURED = [
    (4593, 4096, 4096, (207.5, 171.1, 352.7, 360.1, 215.9, 196.5)), (6000, 2048, 4096, (104.3, 160.1, 237.3, 166.6, 127.7, 119.5)),
    (12000, 2048, 4096, (216.4, 249.5, 493.9, 349.5, 248.6, 222.4)), (12000, 1536, 4096, (207.9, 177.2, 326.8, 268.3, 200.6, 188.6)),
    (2048, 4096, 4096, (97.5, 79.7, 152.8, 153.2, 91.0, 75.7)), (6000, 3072, 3072, (157.1, 137.9, 259.2, 215.1, 152.6, 138.9)),
    (512, 2048, 128, (7.8, 6.9, 4.9, 5.0, 5.0, 6.7)), (512, 1536, 2048, (49.4, 39.5, 10.1, 14.3, 19.3, 22.6)),
    (16384, 1536, 2048, (121.1, 101.8, 231.5, 185.9, 135.8, 119.9)), (4096, 2048, 4096, (96.6, 78.5, 153.2, 104.7, 82.0, 70.6)),
]


@pytest.mark.parametrize("M,N,K,us", NT_MEASURED)
def test_projection_tile_is_the_fastest(M, N, K, us):
    """Within 6 %: the fit's own error (10 % rms) decides between shapes that are closer than that."""
    assert us[rules.NT_TILES.index(rules.nt_tile(M, N, K))] <= 1.06 * min(us)
