"""The dispatch rules of csrc/cca_rules.h on the CPU: the GPU tests' case lists reach every form of a kernel that the rules can
choose."""
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
