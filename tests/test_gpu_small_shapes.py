"""GPU checks of the kernels chosen for small and odd sizes, at the edges of their tiles, against plain fp32 / fp64
products of the same bf16 inputs."""
import sys

import numpy as np
import pytest
import torch

import paper_2510_04476_amd as P
import rules
from oracle import cca_oracle as O
from synth_inputs import make_inputs, make_upstream_grad
from util import check_out, check_tap, oracle_forward, to_np

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rnd(*shape, seed, scale=1.0, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(*shape, generator=g, device="cuda") * scale).to(dtype)


def check_product(got, ref, K):
    """One bf16 rounding (2^-9 relative to the value) on top of an fp32 sum of K terms, whose rounding errors add up to at
    most K * 2^-24 of the sum of magnitudes and typically to sqrt(K) * 2^-24 of their norm."""
    got, ref = got.double(), ref.double()
    scale = float(ref.square().mean().sqrt())
    bound = 2.0 ** -8 * ref.abs() + 4 * K ** 0.5 * 2.0 ** -24 * scale
    worst = float(((got - ref).abs() / bound).max())
    assert worst <= 1.0, worst


# rows x (query heads, KV heads, head width, E): every tile shape of the projection GEMM, a row or column past and short
# of a tile's edge, contraction lengths of one slab, an odd number of slabs (no split over halves) and many; tiles in rows, in whole
# panels and with a narrower last panel
GEMM_CASES = [(1, 1, 1, 64, 64), (65, 1, 1, 64, 192), (127, 3, 1, 64, 320), (512, 8, 2, 128, 2048), (511, 4, 4, 64, 1024),
              (1000, 8, 2, 128, 2048), (1999, 16, 4, 64, 2048), (2050, 5, 5, 64, 1024), (4593, 8, 8, 64, 2048),
              (3001, 8, 2, 128, 2048), (4097, 16, 16, 128, 2048), (4097, 5, 5, 64, 320), (9001, 5, 5, 64, 448), (5953, 5, 5, 64, 2048), (65, 3, 1, 64, 256), (581, 24, 1, 64, 1536), (5999, 8, 2, 128, 2048),
              (11999, 8, 1, 64, 1536)]  # (the shortest contraction whose workgroups pause, behind four of its eight slabs)


@pytest.mark.parametrize("M,Hq,Hk,dh,E", GEMM_CASES)
def test_projection_tiles(M, Hq, Hk, dh, E):
    say("projection", M, Hq, Hk, dh, E)
    cfg = P.CCAConfig(B=1, T=M, d_model=E, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh)
    x, w_down = rnd(1, M, E, seed=1), rnd(E, cfg.n_lat, seed=2, scale=0.02)
    o, w_out = rnd(1, M, cfg.e_q, seed=3), rnd(cfg.e_q, E, seed=4, scale=0.02)
    lat, out = P.cca_down_project(cfg, x, w_down), P.cca_up_project(cfg, o, w_out)
    torch.cuda.synchronize()
    check_product(lat[0], x[0].double() @ w_down.double(), E)
    check_product(out[0], o[0].double() @ w_out.double(), cfg.e_q)


@pytest.mark.parametrize("slabs", [1, 2, 3, 4])
@pytest.mark.parametrize("M,tile,E", [(9001, "256x192", 1024), (32700, "256x256", 1024), (8001, "256x128", 1024), (12001, "192x256", 1024),
                                      (5999, "192x192", 1536)])
def test_projection_of_few_slabs_on_large_tiles(M, tile, E, slabs):
    """Contractions shorter than the three slabs of A and two of the weight that the 256-row kernel holds, and just longer."""
    say("projection", M, slabs)
    cfg = P.CCAConfig(B=1, T=M, d_model=E, n_q_heads=slabs, n_kv_heads=1, head_dim=64)
    assert rules.nt_tile(M, E, 64 * slabs) == tile
    o, w_out = rnd(1, M, cfg.e_q, seed=3), rnd(cfg.e_q, E, seed=4, scale=0.02)
    out = P.cca_up_project(cfg, o, w_out)
    torch.cuda.synchronize()
    check_product(out[0], o[0].double() @ w_out.double(), cfg.e_q)


# token rows x (query heads, head width, E): d W_out (e_q, E) = o^T d_out, beside d_o or alone as the rules have it, and d W_down (E, 3 e_q) =
# x^T d_lat, alone, on every tile shape of the weight-gradient GEMM (64 x 64, 64 x 128, 128 x 128, split 256 x 256), with no, one and a few
# tokens in the last slab of 64; some split on a number of tiles that 8 does not divide and on widths that are no multiple of
# the 32 x 32 blocks of the partial sums
WGRAD_CASES = [(1, 1, 64, 64), (63, 3, 64, 256), (1000, 8, 64, 1024), (64, 8, 128, 2048), (129, 8, 128, 2048),
               (1023, 8, 128, 2048), (512, 12, 128, 2048), (2001, 12, 128, 2048), (9001, 8, 128, 2048),
               (9001, 12, 128, 1536), (8003, 25, 40, 1160), (7001, 3, 72, 1032),
               # one split (stored directly), of one, two, three and many slabs
               (60, 32, 128, 4096), (100, 32, 128, 4096), (190, 49, 80, 4000), (1111, 49, 80, 4000),
               (60, 8, 128, 2048), (100, 8, 128, 2048), (513, 8, 128, 1024)]


@pytest.mark.parametrize("rows,Hq,dh,E", WGRAD_CASES)
def test_weight_gradient_tiles(rows, Hq, dh, E):
    say("weight gradient", rows, Hq, dh, E)
    cfg = P.CCAConfig(B=1, T=rows, d_model=E, n_q_heads=Hq, n_kv_heads=Hq, head_dim=dh, flags=P.CCA_FLAGS_MHA)
    w = P.CCAWeights(w_down=rnd(E, cfg.n_lat, seed=2, scale=0.02), w_out=rnd(cfg.e_q, E, seed=4, scale=0.02))
    x, d_out = rnd(1, rows, E, seed=1), rnd(1, rows, E, seed=5)
    saved = P.CCASaved.allocate(cfg, "cuda")
    P.cca_forward(cfg, w, x, saved=saved)
    _, g = P.cca_backward(cfg, w, x, saved, d_out, grads=P.CCAGrads(w_out=torch.full_like(w.w_out, float("nan"))))
    torch.cuda.synchronize()
    check_product(g.w_out, saved.o[0].double().t().contiguous() @ d_out[0].double(), rows)
    # d_lat stays inside and does not depend on x: with rows of the identity for x, d W_down is d_lat, E rows at a time (sums of one term)
    down = lambda x_: P.cca_backward(cfg, w, x_, saved, d_out, grads=P.CCAGrads(w_down=torch.full_like(w.w_down, float("nan"))), want_d_x=False)[1].w_down
    got, d_lat = down(x), []
    for r0 in range(0, rows, E):
        n = min(E, rows - r0)
        one = torch.zeros_like(x)
        one[0, torch.arange(r0, r0 + n), torch.arange(n)] = 1.0
        d_lat.append(down(one)[:n])
    torch.cuda.synchronize()
    check_product(got, x[0].double().t().contiguous() @ torch.cat(d_lat).double(), rows)


# rows x (query heads, KV heads, head width, E): the two adjoints of a projection in one launch, every pair of tile forms that the rule
# chooses, more tiles than CUs, rows short of and past a tile's edge, and products large enough for a launch each
PAIR_CASES = [(70, 4, 2, 64, 512), (70, 8, 2, 128, 2048), (130, 8, 2, 128, 2048), (400, 8, 2, 128, 2048),
              (130, 4, 4, 128, 1024), (1000, 8, 2, 128, 2048), (511, 4, 4, 64, 1024), (1025, 8, 8, 64, 1024), (1999, 8, 2, 128, 2048), (300, 12, 12, 64, 1536), (4001, 8, 2, 128, 2048), (2050, 16, 16, 64, 1024),
              (901, 4, 1, 128, 1024), (1301, 2, 2, 64, 1024), (777, 3, 1, 128, 1536)]


@pytest.mark.parametrize("rows,Hq,Hk,dh,E", PAIR_CASES)
def test_projection_adjoints_in_one_launch(rows, Hq, Hk, dh, E):
    """Every gradient against the product of its operands in fp64.  d_lat, which stays inside, does not depend on x: with rows of the
    identity for x, d W_down is d_lat, E rows at a time and exactly (sums of one term)."""
    say("projection adjoints", rows, Hq, Hk, dh, E)
    cfg = P.CCAConfig(B=1, T=rows, d_model=E, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, flags=P.CCA_FLAGS_MHA)
    w = P.CCAWeights(w_down=rnd(E, cfg.n_lat, seed=2, scale=0.02), w_out=rnd(cfg.e_q, E, seed=4, scale=0.02))
    x, d_out = rnd(1, rows, E, seed=1), rnd(1, rows, E, seed=5)
    saved = P.CCASaved.allocate(cfg, "cuda")
    P.cca_forward(cfg, w, x, saved=saved)
    nan = lambda t: torch.full_like(t, float("nan"))
    backward = lambda x_: P.cca_backward(cfg, w, x_, saved, d_out, d_x=nan(x), grads=P.CCAGrads(w_down=nan(w.w_down), w_out=nan(w.w_out)))
    d_x, g = backward(x)
    d_lat = []
    for r0 in range(0, rows, E):
        n = min(E, rows - r0)
        one = torch.zeros_like(x)
        one[0, torch.arange(r0, r0 + n), torch.arange(n)] = 1.0
        d_lat.append(backward(one)[1].w_down[:n])
    d_lat = torch.cat(d_lat).double()
    torch.cuda.synchronize()
    check_product(g.w_out, saved.o[0].double().t().contiguous() @ d_out[0].double(), rows)
    check_product(d_x[0], d_lat @ w.w_down.double().t().contiguous(), cfg.n_lat)
    check_product(g.w_down, x[0].double().t().contiguous() @ d_lat, rows)


# d_x over x, and a row further in the same buffer: the weight's gradient still comes from the x that the call was given
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
def test_input_gradient_may_lie_over_the_input(shift, dtype):
    say("d_x over x", shift, dtype)
    bf16 = dtype == "bf16"
    rows, E = 300, 256
    cfg = P.CCAConfig(B=1, T=rows, d_model=E, n_q_heads=2, n_kv_heads=1, head_dim=64, dtype=P.CCA_BF16 if bf16 else P.CCA_F32, flags=P.CCA_FLAGS_MHA)
    r = lambda *s, seed, scale=1.0: rnd(*s, seed=seed, scale=scale, dtype=cfg.torch_dtype)
    w = P.CCAWeights(w_down=r(E, cfg.n_lat, seed=2, scale=0.05), w_out=r(cfg.e_q, E, seed=4, scale=0.05))
    x, d_out = r(1, rows, E, seed=1), r(1, rows, E, seed=5)
    saved = P.CCASaved.allocate(cfg, "cuda")
    P.cca_forward(cfg, w, x, saved=saved)
    d_x, g = P.cca_backward(cfg, w, x, saved, d_out)
    both = torch.empty(rows + 1, E, dtype=cfg.torch_dtype, device="cuda")
    x2, d_x2 = both[None, :rows], both[None, shift:rows + shift]
    x2.copy_(x)
    _, g2 = P.cca_backward(cfg, w, x2, saved, d_out, d_x=d_x2)
    torch.cuda.synchronize()
    for name, a, b in (("d_x", d_x2, d_x), ("d_w_down", g2.w_down, g.w_down), ("d_w_out", g2.w_out, g.w_out)):
        say(name)
        check_product(a, b, rows) if bf16 else torch.testing.assert_close(a, b, rtol=0, atol=0)  # fp32: the same sums in the same order


def test_sequence_filter_gradient_may_lie_over_the_filter():
    """Alone it is written while nothing else reads the filter: d_lat, which does, is complete."""
    say("d_w_conv_seq over w_conv_seq")
    B, T, Hq, Hk, dh = 2, 150, 2, 1, 32
    cfg = P.CCAConfig(B=B, T=T, d_model=64, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, dtype=P.CCA_F32)
    f = lambda *s, seed: rnd(*s, seed=seed, dtype=torch.float32)
    w = P.CCAWeights(w_down=None, w_out=None, w_conv_seq=f(cfg.e_q + cfg.e_kv, 2, seed=1), w_conv_ch=f(Hq + Hk, dh, dh, 2, seed=2), temp=f(Hk, seed=3))
    lat, rnorm = f(B, T, cfg.n_lat, seed=4), torch.empty(B, T, Hq + Hk, device="cuda")
    q, k, v = P.cca_prologue(cfg, w, lat, rnorm=rnorm)
    call = lambda w0, to: P.cca_prologue_backward(cfg, P.CCAWeights(None, None, w0, w.w_conv_ch, w.temp), lat, q, k, rnorm, f(*q.shape, seed=5), f(*k.shape, seed=6),
                                                  f(*v.shape, seed=7), grads=P.CCAGrads(w_conv_seq=to))
    over = w.w_conv_seq.clone()
    d_lat, g = call(w.w_conv_seq, torch.empty_like(over))
    d_lat2, _ = call(over, over)
    torch.cuda.synchronize()
    assert torch.equal(d_lat, d_lat2) and torch.equal(g.w_conv_seq, over)



# B, T, Hq, Hk, d_h, causal, normalised: odd lengths, one tile more or less than a pair, rows whose second key group is
# empty, several query blocks, paired and unpaired grids; scores bounded and not
SPLIT_CASES = [(1, 300, 2, 1, 128, True, True), (1, 321, 3, 3, 64, True, False), (2, 385, 2, 2, 128, False, True),
               (1, 449, 4, 2, 128, False, False), (1, 1000, 4, 2, 64, True, True), (3, 1531, 8, 8, 64, True, True),
               (1, 2047, 16, 16, 128, True, False), (1, 4096, 16, 16, 64, True, False), (2, 513, 4, 1, 128, True, False),
               (1, 4097, 8, 2, 128, True, True),
               # blocks of 64 rows up to their edges: the longest sequence, one round of the grid exactly, and one block more
               (1, 1536, 8, 2, 64, True, True), (1, 513, 28, 7, 128, False, True), (1, 449, 32, 8, 64, True, True),
               (1, 513, 29, 29, 64, False, True)]


@pytest.mark.parametrize("B,T,Hq,Hk,dh,causal,normed", SPLIT_CASES)
def test_attention_with_split_keys(B, T, Hq, Hk, dh, causal, normed):
    """o against fp64 softmax attention on the same bf16 inputs.  P enters the PV product rounded to bf16 (2^-9 of each
    probability, independent) and o is rounded once: 2^-8 of the value plus, per element, the rounding noise of the sum.
    q * scale * log2 e is rounded to bf16 once more (2^-9 of each logit)."""
    say("split attention", B, T, Hq, Hk, dh, causal, normed)
    assert rules.fwd_splits_keys(B * Hq, T, causal)
    flags = (P.CCA_CAUSAL if causal else 0) | (P.CCA_QK_NORM if normed else 0)
    cfg = P.CCAConfig(B=B, T=T, d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, flags=flags)
    q, k = rnd(B, T, Hq, dh, seed=1, dtype=torch.float32), rnd(B, T, Hk, dh, seed=2, dtype=torch.float32)
    if normed:
        q, k = (t * (dh ** 0.5 / t.norm(dim=-1, keepdim=True)) for t in (q, k))
    else:
        q[:, ::7] *= 6.0  # rows whose maximum moves from tile to tile
    q, k, v = q.bfloat16(), k.bfloat16(), rnd(B, T, Hk, dh, seed=3)
    nan = lambda *s, dtype=torch.bfloat16: torch.full(s, float("nan"), dtype=dtype, device="cuda")
    o_inf, o, o_lo, lse = nan(B, T, Hq * dh), nan(B, T, Hq * dh), nan(B, T, Hq * dh), nan(B, Hq, T, dtype=torch.float32)
    P.cca_attention(cfg, q, k, v, o=o_inf)
    P.cca_attention(cfg, q, k, v, o=o, o_lo=o_lo, lse=lse)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(Hq):
            s = q[b, :, h].double() @ k[b, :, h // (Hq // Hk)].double().t().contiguous() / dh ** 0.5
            s_max = float(s.abs().max())
            if causal:
                s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
            p = torch.softmax(s, -1)
            vh = v[b, :, h // (Hq // Hk)].double()
            ref, ref_lse = p @ vh, torch.logsumexp(s, -1)
            # noise of a row: each |p v| term carries a relative error of 2^-9 (P) + 2^-9 s_max (its logit), independent
            noise = 2.0 ** -9 * (1.0 + s_max) * (p.square() @ vh.square()).sqrt()
            bound = 2.0 ** -8 * ref.abs() + 6.0 * noise + 1e-6
            for got in (o_inf, o):
                worst = float(((got[b, :, h * dh:(h + 1) * dh].double() - ref).abs() / bound).max())
                assert worst <= 1.0, (b, h, worst)
            exact = o[b, :, h * dh:(h + 1) * dh].double() + o_lo[b, :, h * dh:(h + 1) * dh].double()
            assert float(((exact - ref).abs() / (2.0 ** -15 * ref.abs() + 6.0 * noise + 1e-6)).max()) <= 1.0
            assert float((lse[b, h].double() - ref_lse).abs().max()) <= 2.0 ** -8 * (s_max + 1.0) + 1e-3


# B, T, H_q, H_k, d_h, causal: every head width, one and two key groups, short and long sequences and many of them
PLAIN_CASES = [(2, 128, 2, 1, 256, True), (1, 257, 3, 3, 256, False), (1, 2049, 2, 1, 256, True), (1, 4481, 8, 2, 128, True),
               (1, 4097, 2, 2, 128, False), (1, 4609, 16, 4, 64, True), (26, 1984, 1, 1, 64, False), (24, 4096, 1, 1, 128, False)]


def plain_layer(B, T, Hq, Hk, dh, causal):
    """A layer without transforms whose down-projection is the identity: the rows of x are those of q, k and v; |q| = |k| = 3."""
    cfg = P.CCAConfig(B=B, T=T, d_model=(Hq + 2 * Hk) * dh, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, k_seq=1, k_ch=1,
                      flags=P.CCA_FLAGS_MHA if causal else P.CCA_FLAGS_MHA & ~P.CCA_CAUSAL)
    w = P.CCAWeights(w_down=torch.eye(cfg.d_model, dtype=torch.bfloat16, device="cuda"), w_out=rnd(cfg.e_q, cfg.d_model, seed=4, scale=0.02))
    lat = rnd(B, T, Hq + 2 * Hk, dh, seed=1, dtype=torch.float32)
    lat[:, :, :Hq + Hk] *= 3.0 / lat[:, :, :Hq + Hk].norm(dim=-1, keepdim=True)
    return cfg, w, lat


@pytest.mark.parametrize("longest", [2.0, 40.0, float("inf"), float("nan")])
@pytest.mark.parametrize("B,T,Hq,Hk,dh,causal", PLAIN_CASES)
def test_plain_attention_of_a_forward(B, T, Hq, Hk, dh, causal, longest):
    """o and lse of a forward are those of the attention stage by itself, bit for bit, whatever the longest rows are; and against
    fp64: P enters the PV product rounded to bf16 (2^-9 of each term), the scaled q too (2^-9 of each logit), and o is rounded once, 2^-8."""
    say("plain attention", B, T, Hq, Hk, dh, causal, longest)
    cfg, w, lat = plain_layer(B, T, Hq, Hk, dh, causal)
    lat[:, T - 1, :Hq] *= longest  # the last query of each head, and an early key
    lat[:, min(T, 64) - 1, Hq:Hq + Hk] *= min(longest, 40.0)
    x = lat.bfloat16().view(B, T, cfg.d_model)
    saved = P.CCASaved.allocate(cfg, "cuda")
    P.cca_forward(cfg, w, x, saved=saved)
    o, lse = P.cca_attention(cfg, saved.q, saved.k, saved.v, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(saved.o.view(torch.int16), o.view(torch.int16)) and torch.equal(saved.lse.view(torch.int32), lse.view(torch.int32))
    if longest != 2.0:
        return
    for b in {0, B - 1}:
        for h in range(Hq):
            s = saved.q[b, :, h].double() @ saved.k[b, :, h // (Hq // Hk)].double().t().contiguous() / dh ** 0.5
            s_max = float(s.abs().max())
            if causal:
                s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
            p, vh = torch.softmax(s, -1), saved.v[b, :, h // (Hq // Hk)].double()
            ref, noise = p @ vh, 2.0 ** -9 * (1.0 + s_max) * (p.square() @ vh.square()).sqrt()
            got = saved.o[b, :, h * dh:(h + 1) * dh].double()
            assert float(((got - ref).abs() / (2.0 ** -8 * ref.abs() + 6.0 * noise + 1e-6)).max()) <= 1.0, (b, h)
            assert float((saved.lse[b, h].double() - torch.logsumexp(s, -1)).abs().max()) <= 2.0 ** -8 * (s_max + 1.0) + 1e-3


@pytest.mark.parametrize("power", [96, -90])
@pytest.mark.parametrize("B,T,Hq,Hk,dh,causal", PLAIN_CASES)
def test_plain_attention_keeps_the_range_of_v(B, T, Hq, Hk, dh, causal, power):
    """v times a power of two leaves o times that power, bit for bit: no probability is formed so far from 1 that its product with a
    large v overflows or with a small one is flushed.  A pair of rows makes scores of +-30 (43 in log2 units) beside the others' 1."""
    say("range of v", B, T, Hq, Hk, dh, causal, power)
    cfg, w, lat = plain_layer(B, T, Hq, Hk, dh, causal)
    longest = 30.0 * dh ** 0.5
    lat[:, T - 1, :Hq] = longest ** 0.5 * dh ** -0.5
    lat[:, min(T, 64) - 1, Hq:Hq + Hk] = longest ** 0.5 * dh ** -0.5
    lat[:, T // 2, Hq:Hq + Hk] = -longest ** 0.5 * dh ** -0.5
    plain = P.cca_forward(cfg, w, lat.bfloat16().view(B, T, cfg.d_model))
    lat[:, :, Hq + Hk:] *= 2.0 ** power
    scaled = P.cca_forward(cfg, w, lat.bfloat16().view(B, T, cfg.d_model))
    torch.cuda.synchronize()
    assert bool(scaled.isfinite().all()) and torch.equal(scaled.float() * 2.0 ** -power, plain.float())


def check_masked_keys(dh, causal, live, masked, hot=False):
    """Keys outside `live` (a mask over T) score `masked` times a positive number, through a channel of k at that value that every q
    reads with a positive weight: the rows that see a live key are those of attention over the live keys alone, with the
    roundings of the test above."""
    T, Hq = live.numel(), 2
    assert rules.fwd_splits_keys(Hq, T, causal)
    # hot: normalised heads, whose temperature leaves the scores without a usable bound
    flags = (P.CCA_CAUSAL if causal else 0) | (P.CCA_QK_NORM | P.CCA_KEY_TEMP if hot else 0)
    cfg = P.CCAConfig(B=1, T=T, d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hq, head_dim=dh, flags=flags)
    q, k, v = rnd(1, T, Hq, dh, seed=1), rnd(1, T, Hq, dh, seed=2), rnd(1, T, Hq, dh, seed=3)
    q[..., 5] = 1.0
    k[:, ~live, :, 5] = masked
    o, lse = P.cca_attention(cfg, q, k, v, want_lse=True, temp=torch.full((Hq,), 9.0, device="cuda") if hot else None)
    torch.cuda.synchronize()
    first = int(live.nonzero()[0]) if causal else 0
    for h in range(Hq):
        s = q[0, first:, h].double() @ k[0, live, h].double().t().contiguous() / dh ** 0.5
        s_max = float(s.abs().max())
        if causal:
            s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)[first:, live], float("-inf"))
        p, vh = torch.softmax(s, -1), v[0, live, h].double()
        noise = 2.0 ** -9 * (1.0 + s_max) * (p.square() @ vh.square()).sqrt()
        ref = p @ vh
        got = o[0, first:, h * dh:(h + 1) * dh].double()
        assert bool(got.isfinite().all())
        assert float(((got - ref).abs() / (2.0 ** -8 * ref.abs() + 6.0 * noise + 1e-6)).max()) <= 1.0
        assert float((lse[0, h, first:].double() - torch.logsumexp(s, -1)).abs().max()) <= 2.0 ** -8 * (s_max + 1.0) + 1e-3


@pytest.mark.parametrize("live", [(0, 40), (70, 140), (129, 300)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [64, 128, 256])
@pytest.mark.parametrize("masked", [float("-inf"), -2e4])
def test_attention_keys_masked_by_infinite_scores(dh, causal, live, masked):
    """Scores of -inf, or far below any other, in whole key tiles."""
    say("infinite scores", dh, causal, live, masked)
    t = torch.arange(300, device="cuda")
    check_masked_keys(dh, causal, (t >= live[0]) & (t < live[1]), masked)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("masked", [float("-inf"), -2e4, -1e38])
def test_attention_on_64_rows_without_a_bound(dh, causal, masked):
    """The same in blocks of 64 rows, which only normalised heads take."""
    say("64 rows", dh, causal, masked)
    assert rules.fwd_takes_64_rows(2, 300, True)
    t = torch.arange(300, device="cuda")
    check_masked_keys(dh, causal, (t >= 129) & (t < 290), masked, hot=True)


@pytest.mark.parametrize("gap", [(0, 64), (64, 128), (0, 300)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [64, 128, 256])
def test_attention_keys_masked_by_the_lowest_scores(dh, causal, gap):
    """Scores near the type's lowest value in the first tiles of one or both key groups: against a reference max taken from them all
    later scores round to one value."""
    say("lowest scores", dh, causal, gap)
    t = torch.arange(1000, device="cuda")
    check_masked_keys(dh, causal, (t < gap[0]) | (t >= gap[1]), -1e38)


@pytest.mark.parametrize("live", [(0, 40), (70, 140), (129, 300)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,dtype", [(32, P.CCA_F32), (200, P.CCA_F32), (40, P.CCA_BF16)])
def test_generic_attention_keys_masked_by_infinite_scores(dh, dtype, causal, live):
    """The same through the shape-generic kernel: fp32 sums of up to T terms each, bf16 results rounded once."""
    T, Hq, lo, hi = 300, 2, *live
    say("infinite scores, generic", dh, dtype, causal, live)
    cfg = P.CCAConfig(B=1, T=T, d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hq, head_dim=dh, dtype=dtype, flags=P.CCA_CAUSAL if causal else 0)
    q, k, v = (rnd(1, T, Hq, dh, seed=s, dtype=cfg.torch_dtype) for s in (1, 2, 3))
    q[..., 5] = 1.0
    k[:, :lo, :, 5], k[:, hi:, :, 5] = float("-inf"), float("-inf")
    o, lse = P.cca_attention(cfg, q, k, v, want_lse=True)
    torch.cuda.synchronize()
    first = lo if causal else 0
    for h in range(Hq):
        s = q[0, first:, h].double() @ k[0, lo:hi, h].double().t().contiguous() / dh ** 0.5
        if causal:
            s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)[first:, lo:hi], float("-inf"))
        ref = torch.softmax(s, -1) @ v[0, lo:hi, h].double()
        got = o[0, first:, h * dh:(h + 1) * dh].double()
        assert bool(got.isfinite().all())
        bound = (2.0 ** -8 if dtype == P.CCA_BF16 else 0.0) * ref.abs() + 1e-5 * float(ref.abs().max())
        assert float(((got - ref).abs() / bound).max()) <= 1.0
        assert float((lse[0, h, first:].double() - torch.logsumexp(s, -1)).abs().max()) <= 1e-5


@pytest.mark.parametrize("dh,Hk,dtype", [(64, 2, P.CCA_BF16), (128, 1, P.CCA_BF16), (256, 1, P.CCA_BF16), (40, 1, P.CCA_BF16), (64, 1, P.CCA_F32)])
def test_decode_keys_masked_by_infinite_scores(dh, Hk, dtype):
    """Whole blocks and splits of the cache at -inf: the step equals a step over the live keys alone (the first `live` ones and
    the new token's), whose sums run in another order."""
    T, live, Hq = 900, 37, 2
    say("infinite scores, decode", dh, Hk, dtype)
    mk = lambda cap: P.CCAConfig(B=1, T=cap, d_model=512, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, k_seq=1, k_ch=1, dtype=dtype,
                                 flags=P.CCA_FLAGS_MHA)
    cfg, few = mk(T), mk(live + 1)
    w = P.CCAWeights(w_down=rnd(512, cfg.n_lat, seed=1, scale=0.02, dtype=cfg.torch_dtype),
                     w_out=rnd(cfg.e_q, 512, seed=2, scale=0.05, dtype=cfg.torch_dtype))
    for h in range(Hq):  # every query reads channel 5 with a positive weight
        w.w_down[:, h * dh + 5] = 0.01
    x = rnd(1, 512, seed=3, dtype=cfg.torch_dtype).abs()
    k, v = rnd(1, T, Hk, dh, seed=4, dtype=cfg.torch_dtype), rnd(1, T, Hk, dh, seed=5, dtype=cfg.torch_dtype)

    def step(c, at, keep):
        st = P.CCADecodeState.allocate(c, "cuda")
        st.k_cache.copy_(k[:, :1].expand_as(st.k_cache)), st.v_cache.copy_(v[:, :1].expand_as(st.v_cache))
        st.k_cache[..., 5] = float("-inf")
        st.k_cache[:, keep], st.v_cache[:, keep] = k[:, :live], v[:, :live]
        return P.cca_decode_step(c, w, x, st, at)

    for first in (0, 300, T - 1 - live):
        out = step(cfg, T - 1, slice(first, first + live))
        ref = step(few, live, slice(0, live)).double()
        torch.cuda.synchronize()
        assert bool(ref.isfinite().all()) and bool(out.isfinite().all()), first
        tol = 2.0 ** -7 if dtype == P.CCA_BF16 else 1e-5
        assert float((out.double() - ref).norm()) <= tol * float(ref.norm()), first


def transforms(lat, w0, w1, temp, Hq, Hk, dh):
    """The block's steps between the down-projection and attention in plain torch: both convolutions, qk-mean, norm and
    temperature, RoPE, value-shift."""
    B, T, _ = lat.shape
    past = lambda u, n: torch.cat([torch.zeros_like(u[:, :n]), u[:, :T - n]], 1) if n else u
    e_q, e_kv = Hq * dh, Hk * dh
    u = lat[..., :e_q + e_kv]
    y = sum(w0[:, j] * past(u, w0.shape[1] - 1 - j) for j in range(w0.shape[1])).view(B, T, Hq + Hk, dh)
    taps = w1.shape[-1]
    y = torch.stack([sum(past(y[:, :, h], taps - 1 - j) @ w1[h, :, :, j].t() for j in range(taps)) for h in range(Hq + Hk)], 2)
    q0, k0 = u[..., :e_q].view(B, T, Hk, Hq // Hk, dh), u[..., e_q:].view(B, T, Hk, 1, dh)
    m = 0.5 * (q0 + k0)
    y = y + torch.cat([m.reshape(B, T, Hq, dh), m.mean(3)], 2)
    y = y * dh ** 0.5 / y.norm(dim=-1, keepdim=True)
    y = torch.cat([y[:, :, :Hq], y[:, :, Hq:] * temp.exp()[:, None]], 2)
    t = torch.arange(T, device=lat.device, dtype=lat.dtype)[:, None]
    ang = t * 10000.0 ** (-2.0 * torch.arange(dh // 2, device=lat.device, dtype=lat.dtype) / dh)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = y[..., :dh // 2], y[..., dh // 2:]
    y = torch.cat([a * c - b * s, b * c + a * s], -1)
    v = lat[..., e_q + e_kv:]
    v = torch.cat([v[..., :e_kv // 2], past(v[..., e_kv // 2:], 1)], -1).view(B, T, Hk, dh)
    return y[:, :, :Hq], y[:, :, Hq:], v


# d_h = 256, both forms of the prologue and of its adjoint (128 and 256 tokens per workgroup) with 1, 2 and 3 taps: rows that are no
# multiple of either block or of a wavefront's 32, several sequences in a block, one to four query heads per KV head
STREAM_CASES = [(3, 45, 1, 1, 1, 1), (2, 131, 4, 1, 2, 2), (1, 1, 2, 2, 2, 1), (1, 257, 4, 2, 3, 1), (5, 421, 8, 8, 2, 2),
                (1, 2100, 8, 8, 1, 1), (1, 2305, 8, 8, 1, 2), (7, 1801, 4, 1, 3, 1), (2, 7003, 6, 2, 1, 1), (3, 2999, 6, 2, 2, 1),
                (1, 130, 7, 1, 2, 2)]


@pytest.mark.parametrize("B,T,Hq,Hk,k_seq,k_ch", STREAM_CASES)
def test_wide_head_prologue(B, T, Hq, Hk, k_seq, k_ch):
    say("wide head prologue", B, T, Hq, Hk, k_seq, k_ch)
    check_prologue(B, T, Hq, Hk, k_seq, k_ch, 256)


# tokens of one sequence, and the channel from which a head's own half of the qk-mean joins behind its filter's last products: a slab of 32
# input channels with 128 tokens a workgroup, one of 64 with 256
@pytest.mark.parametrize("T,edge", [(130, 224), (16401, 192)])
def test_own_half_of_the_wide_qk_mean_joins_behind_its_slab(T, edge):
    """The order of the sums is part of the results, bit for bit.  Every output is 2^30 (first input channel) - 2^30 (last one) + 1/2
    (own row) + 1/2 (the other stream); the first half is lost in fp32 where it is added before the last channel's product."""
    say("order of the qk-mean", T)
    cfg = P.CCAConfig(B=1, T=T, d_model=256, n_q_heads=1, n_kv_heads=1, head_dim=256, k_seq=1, k_ch=1, flags=P.CCA_CAUSAL | P.CCA_CONV_CH | P.CCA_QK_MEAN)
    assert {rules.stream_takes_256(T, 2, 1, 1, adjoint) for adjoint in (False, True)} == {T > 130}
    one = lambda *s: torch.ones(s, dtype=torch.bfloat16, device="cuda")
    pattern = torch.full((256,), 0.5, device="cuda")
    pattern[edge:] = 1.0
    w1 = torch.zeros(2, 256, 256, 1, dtype=torch.bfloat16, device="cuda")  # (head, output, input, tap)
    w1[:, :, 0], w1[:, :, 255] = 2.0 ** 30, -2.0 ** 30
    w = P.CCAWeights(w_down=None, w_out=None, w_conv_ch=w1)
    q, k, v, rnorm = one(1, T, 1, 256), one(1, T, 1, 256), one(1, T, 1, 256), torch.ones(1, T, 2, device="cuda")
    P.cca_prologue(cfg, w, one(1, T, cfg.n_lat), q, k, v, rnorm=rnorm)
    w = P.CCAWeights(w_down=None, w_out=None, w_conv_ch=w1.transpose(1, 2).contiguous())
    d_lat, _ = P.cca_prologue_backward(cfg, w, one(1, T, cfg.n_lat), q, k, rnorm, one(*q.shape), one(*k.shape), one(*v.shape))
    torch.cuda.synchronize()
    for name, got in (("q", q), ("k", k), ("d_lat", d_lat[..., :512].reshape(1, T, 2, 256))):
        assert torch.equal(got.float(), pattern.expand(got.shape)), name


# d_h = 64 and 128, the short and the long form, forward and adjoint, with 1, 2 and 3 taps: sequences shorter than the taps reach, many
# of them in a workgroup's 64 tokens, one token more and less than 64, one to five query heads per KV head (their mean's weight
# exact in bf16 or not, more partner rows than are requested at a time)
PROLOGUE_CASES = [(1, 1, 2, 2, 2, 1, 64), (1, 1, 1, 1, 1, 1, 128), (13, 5, 4, 2, 2, 2, 128), (70, 2, 2, 1, 2, 2, 64), (1, 63, 3, 1, 2, 2, 128),
                  (1, 64, 5, 1, 3, 1, 64), (2, 65, 10, 2, 1, 2, 128), (1, 129, 8, 8, 1, 1, 64), (3, 131, 6, 2, 1, 1, 128), (1, 3900, 5, 1, 2, 2, 128),
                  (1, 7900, 1, 1, 1, 1, 128), (1, 8300, 1, 1, 2, 1, 128), (2, 4400, 2, 2, 2, 2, 128), (1, 8300, 1, 1, 1, 1, 128),
                  (1, 20601, 1, 1, 1, 1, 64), (3, 16421, 1, 1, 1, 2, 64), (4, 6151, 4, 4, 2, 2, 64), (3, 16421, 1, 1, 1, 1, 64)]


@pytest.mark.parametrize("B,T,Hq,Hk,k_seq,k_ch,dh", PROLOGUE_CASES)
def test_prologue_forms(B, T, Hq, Hk, k_seq, k_ch, dh):
    say("prologue", B, T, Hq, Hk, k_seq, k_ch, dh)
    check_prologue(B, T, Hq, Hk, k_seq, k_ch, dh)


# chunks of 512, 1024 and 2048 tokens of the filter gradients: last ones that are short, sequences shorter than a chunk
FILTER_GRADIENT_CASES = [(3, 2503, 8, 8, 2, 2, 128), (3, 2611, 8, 8, 2, 2, 128), (131, 61, 8, 8, 2, 1, 128), (1, 19601, 8, 8, 1, 2, 128),
                         (7, 1499, 12, 12, 2, 2, 64)]


@pytest.mark.parametrize("B,T,Hq,Hk,k_seq,k_ch,dh", FILTER_GRADIENT_CASES)
def test_filter_gradient_chunks(B, T, Hq, Hk, k_seq, k_ch, dh):
    say("filter gradient chunks", B, T, Hq, Hk, k_seq, k_ch, dh)
    check_prologue(B, T, Hq, Hk, k_seq, k_ch, dh)


def check_prologue(B, T, Hq, Hk, k_seq, k_ch, dh):
    """q, k, v and, through autograd, d_lat against the steps in fp64.  The filters are folded and rounded to bf16 (2^-9 of each
    weight), q and k rounded once, the gradient entering the convolutions once: the 1e-2 of the whole-block tests."""
    cfg = P.CCAConfig(B=B, T=T, d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, k_seq=k_seq, k_ch=k_ch)
    w = P.CCAWeights(w_down=None, w_out=None, w_conv_seq=rnd(cfg.e_q + cfg.e_kv, k_seq, seed=1, scale=k_seq ** -0.5),
                     w_conv_ch=rnd(Hq + Hk, dh, dh, k_ch, seed=2, scale=(dh * k_ch) ** -0.5), temp=rnd(Hk, seed=3, scale=0.3, dtype=torch.float32))
    lat = rnd(B, T, cfg.n_lat, seed=4)
    nan = lambda *s, dtype=torch.bfloat16: torch.full(s, float("nan"), dtype=dtype, device="cuda")
    q, k, v, rnorm = nan(B, T, Hq, dh), nan(B, T, Hk, dh), nan(B, T, Hk, dh), nan(B, T, Hq + Hk, dtype=torch.float32)
    P.cca_prologue(cfg, w, lat, q, k, v, rnorm=rnorm)
    d_q, d_k, d_v = (rnd(*t.shape, seed=s) for t, s in ((q, 5), (k, 6), (v, 7)))
    d_lat, g = P.cca_prologue_backward(cfg, w, lat, q, k, rnorm, d_q, d_k, d_v, d_lat=torch.full_like(lat, float("nan")))
    torch.cuda.synchronize()
    x = lat.double().requires_grad_()
    w0, w1, temp = (t.double().requires_grad_() for t in (w.w_conv_seq, w.w_conv_ch, w.temp))
    ref = transforms(x, w0, w1, temp, Hq, Hk, dh)
    torch.autograd.backward(ref, [t.double() for t in (d_q, d_k, d_v)])
    assert torch.equal(v, ref[2].detach().bfloat16())
    d_temp, ref_temp = g.temp, temp.grad
    if dh < 256:  # one sum over <d_k, k> per head, of terms of either sign: with a pull of d_k along k, so that they do not cancel
        along = (d_k.float() + 0.25 * k.float()).bfloat16()
        d_temp = P.cca_prologue_backward(cfg, w, lat, q, k, rnorm, d_q, along, d_v)[1].temp
        ref_temp = (along.double() * ref[1].detach()).sum((0, 1, 3))  # k is exp(temp) times what does not depend on it
    for name, got, r in (("q", q, ref[0]), ("k", k, ref[1]), ("d_lat", d_lat, x.grad), ("d_w_conv_seq", g.w_conv_seq, w0.grad),
                         ("d_w_conv_ch", g.w_conv_ch, w1.grad), ("d_temp", d_temp, ref_temp)):
        rel = float((got.double() - r.detach()).norm() / r.detach().norm())
        say(name, rel)
        assert rel <= 1e-2, (name, rel)


# the decode step's projections (several passes through LDS, K slices of the down-projection, lengths that are not whole
# groups) and filter layouts: widths 256 and 64 with up to 4 + 4 taps, 5 query heads per KV head
DECODE_CASES = [dict(B=9, T=5, E=4104, Hq=4, Hk=2, dh=64, k_seq=2, k_ch=2), dict(B=2, T=9, E=2056, Hq=4, Hk=2, dh=256, k_seq=4, k_ch=4),
                dict(B=97, T=4, E=520, Hq=3, Hk=1, dh=64, k_seq=2, k_ch=2),  # four blocks of rows, the last of one
                dict(B=3, T=7, E=640, Hq=5, Hk=1, dh=64, k_seq=1, k_ch=4), dict(B=1, T=6, E=512, Hq=2, Hk=1, dh=256, k_seq=3, k_ch=3)]


@pytest.mark.parametrize("i", range(len(DECODE_CASES)))
def test_decode_projections_and_filters(i):
    """Ring slots of tokens before the sequence's start may hold anything: they start as NaN here."""
    w = dict(DECODE_CASES[i], dtype="bf16", paper_flags=True)
    say("decode", w)
    inp = make_inputs(w, seed=170 + i, conv_visible=True)
    cfg = P.config_from_workload(w)
    x, wt = P.weights_to_device(cfg, inp)
    state = P.CCADecodeState.allocate(cfg, "cuda")
    state.lat_ring.fill_(float("nan"))
    outs = [P.cca_decode_step(cfg, wt, x[:, t].contiguous(), state, t) for t in range(w["T"])]
    torch.cuda.synchronize()
    ref = oracle_forward(w, inp)
    say(check_out(to_np(torch.stack(outs, 1)), ref["out"], "bf16"))
    say(check_tap(to_np(state.k_cache), ref["k"], "bf16", "k_cache"))
    say(check_tap(to_np(state.v_cache), ref["v"], "bf16", "v_cache"))


@pytest.mark.parametrize("dtype", [P.CCA_BF16, P.CCA_F32])
@pytest.mark.parametrize("dh,k_ch", [(64, 3), (40, 2), (64, 2), (256, 4)])
def test_decode_infinite_filter_weight(dh, k_ch, dtype):
    """An infinity in the last weight of a filter row makes that output infinite (not NaN, whatever the row's length leaves
    of the lanes that share it) and no other."""
    say("infinite weight", dh, k_ch, dtype)
    cfg = P.CCAConfig(B=2, T=9, d_model=128 if dh < 256 else 512, n_q_heads=1, n_kv_heads=1, head_dim=dh, k_seq=1, k_ch=k_ch, dtype=dtype,
                      flags=P.CCA_CAUSAL | P.CCA_CONV_CH)
    dt = cfg.torch_dtype
    w = P.CCAWeights(w_down=rnd(cfg.d_model, cfg.n_lat, seed=1, scale=0.1, dtype=dt), w_out=rnd(cfg.e_q, cfg.d_model, seed=2, dtype=dt),
                     w_conv_ch=rnd(2, dh, dh, k_ch, seed=3, dtype=dt))
    x = rnd(4, 2, cfg.d_model, seed=4, dtype=dt)

    def cache():
        st = P.CCADecodeState.allocate(cfg, "cuda")
        for t in range(4):
            P.cca_decode_step(cfg, w, x[t], st, t)
        return st.k_cache[:, :4, 0].float()

    clean = cache()
    w.w_conv_ch[1, 5, dh - 1, k_ch - 1] = float("inf")
    dirty = cache()
    torch.cuda.synchronize()
    assert bool(dirty[..., 5].isinf().all())
    keep = [c for c in range(dh) if c != 5]
    assert bool(clean.isfinite().all()) and torch.equal(dirty[..., keep], clean[..., keep])


@pytest.mark.parametrize("Hq,Hk,dh", [(4, 2, 64), (4, 1, 128), (2, 2, 256)])
def test_decode_split_edges(Hq, Hk, dh):
    """Positions around the edges of the splits of the key range (units of 64, 128 and 256 keys)."""
    w = dict(B=1, T=1100, E=512, Hq=Hq, Hk=Hk, dh=dh, k_seq=2, k_ch=2, dtype="bf16", paper_flags=True)
    inp = make_inputs(w, seed=180, conv_visible=True)
    cfg = P.config_from_workload(w)
    x, wt = P.weights_to_device(cfg, inp)
    saved = P.CCASaved.allocate(cfg, "cuda")
    P.cca_forward(cfg, wt, x, saved=saved)
    ref = oracle_forward(w, inp)["out"]
    for pos in (0, 63, 64, 126, 127, 128, 255, 256, 511, 513, 1023, 1099):
        say("decode split", Hq, Hk, dh, pos)
        state = P.CCADecodeState.allocate(cfg, "cuda")
        state.k_cache.fill_(float("nan")), state.v_cache.fill_(float("nan"))
        state.load_prefill(saved, pos)
        out = P.cca_decode_step(cfg, wt, x[:, pos].contiguous(), state, pos)
        torch.cuda.synchronize()
        check_out(to_np(out), ref[:, pos], "bf16")


# shape-generic kernels: widths that are no multiple of 32, one token, a token more than a tile, group sizes 1 and 3, every
# instantiation of the head width; fp32 against the oracle at its 1e-5, forward and backward
GENERIC_CASES = [dict(B=1, T=1, E=48, Hq=2, Hk=1, dh=12, k_seq=2, k_ch=2), dict(B=2, T=33, E=120, Hq=3, Hk=1, dh=40, k_seq=4, k_ch=3),
                 dict(B=1, T=97, E=288, Hq=3, Hk=3, dh=96, k_seq=1, k_ch=2), dict(B=1, T=70, E=264, Hq=1, Hk=1, dh=200, k_seq=2, k_ch=1),
                 dict(B=3, T=300, E=64, Hq=6, Hk=2, dh=4, k_seq=3, k_ch=4),
                 # tiles of 16 rows and of 32 tokens met exactly and by one; filter gradients whole and in 2, 6 and 16 parts of the rows
                 dict(B=2, T=161, E=64, Hq=2, Hk=2, dh=32, k_seq=2, k_ch=2), dict(B=3, T=48, E=128, Hq=2, Hk=1, dh=64, k_seq=2, k_ch=2),
                 dict(B=1, T=31, E=256, Hq=1, Hk=1, dh=256, k_seq=2, k_ch=2), dict(B=1, T=1024, E=64, Hq=2, Hk=2, dh=32, k_seq=2, k_ch=2),
                 # more workgroups than one round: the attention's 32-row forms (tests/test_dispatch_rules.py)
                 dict(B=6, T=65, E=192, Hq=24, Hk=12, dh=8, k_seq=2, k_ch=2), dict(B=13, T=161, E=288, Hq=3, Hk=3, dh=96, k_seq=2, k_ch=2),
                 # a projection's adjoints in a launch each
                 dict(B=5, T=450, E=512, Hq=2, Hk=1, dh=32, k_seq=2, k_ch=2)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("i", range(len(GENERIC_CASES)))
def test_generic_kernels_fp32(i, causal):
    w = dict(GENERIC_CASES[i], dtype="f32", paper_flags=True)
    say("generic fp32", w, causal)
    inp = make_inputs(w, seed=190 + i, conv_visible=True)
    flags = P.CCA_FLAGS_PAPER if causal else P.CCA_FLAGS_PAPER & ~P.CCA_CAUSAL
    cfg = P.config_from_workload(w, flags=flags)
    x, wt = P.weights_to_device(cfg, inp)
    saved = P.CCASaved.allocate(cfg, "cuda")
    out = P.cca_forward(cfg, wt, x, saved=saved)
    d_out = make_upstream_grad(w, seed=3)
    d_x, g = P.cca_backward(cfg, wt, x, saved, torch.from_numpy(d_out).cuda())
    torch.cuda.synchronize()
    say(check_out(to_np(out), oracle_forward(w, inp, causal=causal)["out"], "f32"))
    ref = O.cca_backward(inp["x"], inp["w_down"], inp["w_conv_seq"], inp["w_conv_ch"], inp["temp"], inp["w_out"], d_out,
                         n_q_heads=w["Hq"], n_kv_heads=w["Hk"], head_dim=w["dh"], causal=causal)
    for name, got in (("d_x", d_x), ("d_w_down", g.w_down), ("d_w_conv_seq", g.w_conv_seq), ("d_w_conv_ch", g.w_conv_ch),
                      ("d_w_out", g.w_out)):
        r = ref[name]
        err = float(np.linalg.norm(to_np(got) - r))
        # one token: softmax over one key is constant, the exact gradient of q and k is zero and only rounding is left
        assert err <= 1e-5 * float(np.linalg.norm(r)) + 1e-6, (name, err, float(np.linalg.norm(r)))


def test_generic_product_beyond_2_to_33_outputs():
    """A product of more 32 x 32 tiles than one grid dimension holds threads for (2^23 tiles x 512), 17 GB of bf16: every tile
    is there, and rows from all over are the product."""
    M, K, N = (1 << 20) + 33, 8, 8200
    say("generic product", M, K, N)
    cfg = P.CCAConfig(B=1, T=M, d_model=N, n_q_heads=1, n_kv_heads=1, head_dim=K)
    o, w = rnd(1, M, K, seed=1), rnd(K, N, seed=2)
    out = torch.full((1, M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    P.cca_up_project(cfg, o, w, out)
    torch.cuda.synchronize()
    for first in range(0, M, 1 << 17):
        assert not bool(out[0, first:first + (1 << 17)].isnan().any()), first
    rows = torch.tensor([0, 31, 32, M // 2, M - 34, M - 2, M - 1] + [(i * 2654435761) % M for i in range(200)], device="cuda")
    check_product(out[0, rows], o[0, rows].double() @ w.double(), K)


def test_generic_attention_hides_masked_infinities():
    """fp32, causal: a NaN or infinity in a later token's key, value or query must not reach earlier rows or their gradients."""
    T, cut = 75, 41
    cfg = P.CCAConfig(B=1, T=T, d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=32, dtype=P.CCA_F32, flags=P.CCA_FLAGS_MHA)
    q, k, v, d_o = (rnd(1, T, h, 32, seed=20 + h + s, dtype=torch.float32) for s, h in ((0, 2), (5, 1), (9, 1), (13, 2)))
    run = lambda q, k, v, d_o: (lambda o, lse: (o, lse) + tuple(P.cca_attention_backward(cfg, q, k, v, o, lse, d_o.reshape(1, T, 64))))(
        *P.cca_attention(cfg, q, k, v, want_lse=True))
    clean = run(q, k, v, d_o)
    bad = [t.clone() for t in (q, k, v, d_o)]
    bad[0][0, cut, :, 3], bad[1][0, cut + 1, :, 4], bad[2][0, cut, :, 5] = float("nan"), float("inf"), float("-inf")
    dirty = run(*bad)
    torch.cuda.synchronize()
    say("masked infinities")

    # the sums of a tile that holds such a value run in another order: at most 2 T 2^-24 of the sum of magnitudes apart,
    # which is below T times the largest value here
    def same(a, b):
        return bool(torch.isfinite(b).all()) and float((a - b).abs().max()) <= 2 * T * 2.0 ** -24 * T * float(a.abs().max())

    assert same(clean[0][:, :cut], dirty[0][:, :cut]) and same(clean[1][:, :, :cut], dirty[1][:, :, :cut])
    assert same(clean[2][:, :cut], dirty[2][:, :cut])  # d_q of earlier rows
    assert not torch.isfinite(dirty[0][:, cut]).all()
    # a row before a key does not count in that key's gradients
    late = [t.clone() for t in (q, k, v, d_o)]
    late[0][0, cut], late[3][0, cut] = float("nan"), float("inf")
    dk, dv = run(*late)[3:]
    torch.cuda.synchronize()
    assert same(clean[3][:, cut + 1:], dk[:, cut + 1:]) and same(clean[4][:, cut + 1:], dv[:, cut + 1:])


# the same grids backward (both kernels split): d_q, d_k, d_v against fp64 on the same bf16 inputs
BWD_SPLIT_CASES = [(1, 129, 3, 3, 64, True), (1, 300, 2, 1, 128, True), (2, 385, 2, 2, 128, False), (1, 1000, 4, 2, 64, False),
                   (1, 1023, 4, 1, 128, True), (2, 1531, 8, 8, 64, True), (1, 2047, 8, 2, 128, False), (1, 2050, 16, 16, 128, True)]


@pytest.mark.parametrize("B,T,Hq,Hk,dh,causal", BWD_SPLIT_CASES)
def test_attention_backward_with_split_rows(B, T, Hq, Hk, dh, causal):
    """P and dS enter their products rounded to bf16 (2^-9 each), q and the results are rounded once more, and the row sums
    come from the forward's bf16 scores (2^-9 of each logit, |logit| <= 11 here): six roundings of 2^-9 in quadrature on
    q (6e-3 rel-L2, as the whole-block tests measure); the asserted bound is their 1e-2."""
    say("split backward", B, T, Hq, Hk, dh, causal)
    assert rules.dq_splits_keys(B * Hq, T, causal) and rules.dkdv_splits_rows(B * Hq, T, causal)
    flags = (P.CCA_CAUSAL if causal else 0) | P.CCA_QK_NORM
    cfg = P.CCAConfig(B=B, T=T, d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, flags=flags)
    q, k = rnd(B, T, Hq, dh, seed=1, dtype=torch.float32), rnd(B, T, Hk, dh, seed=2, dtype=torch.float32)
    q, k = (t * (dh ** 0.5 / t.norm(dim=-1, keepdim=True)) for t in (q, k))
    q, k, v, d_o = q.bfloat16(), k.bfloat16(), rnd(B, T, Hk, dh, seed=3), rnd(B, T, Hq * dh, seed=4)
    o_lo = torch.empty_like(d_o)
    o, lse = P.cca_attention(cfg, q, k, v, want_lse=True, o_lo=o_lo)
    got = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    P.cca_attention_backward(cfg, q, k, v, o, lse, d_o, *got, o_lo=o_lo)
    again = P.cca_attention_backward(cfg, q, k, v, o, lse, d_o, o_lo=o_lo)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    ref = [torch.zeros_like(t, dtype=torch.float64) for t in (q, k, v)]
    mask = torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1) if causal else None
    for b in range(B):
        for h in range(Hq):
            g = h // (Hq // Hk)
            qh, kh, vh, do = q[b, :, h].double(), k[b, :, g].double(), v[b, :, g].double(), d_o[b, :, h * dh:(h + 1) * dh].double()
            s = qh @ kh.t().contiguous() / dh ** 0.5
            p = torch.softmax(s if mask is None else s.masked_fill(mask, float("-inf")), -1)
            d_p = do @ vh.t().contiguous()
            d_s = p * (d_p - (p * d_p).sum(-1, keepdim=True)) / dh ** 0.5
            ref[0][b, :, h] = d_s @ kh
            ref[1][b, :, g] += d_s.t().contiguous() @ qh
            ref[2][b, :, g] += p.t().contiguous() @ do
    for name, a, r in zip(("d_q", "d_k", "d_v"), got, ref):
        rel = float((a.double() - r).norm() / r.norm())
        worst = float((a.double() - r).abs().max() / r.abs().max())
        say(name, rel, worst)
        assert rel <= 1e-2 and worst <= 2e-2, (name, rel, worst)


@pytest.mark.parametrize("T,Hq,Hk,dh,E", [(1, 1, 1, 64, 64), (67, 3, 1, 64, 320), (511, 8, 2, 128, 1024),
                                           (2050, 5, 5, 40, 2048), (4593, 8, 8, 64, 2048), (4097, 16, 16, 128, 2048)])
@pytest.mark.parametrize("shift", [0, P.CCA_V_SHIFT])
def test_projection_stores_heads_of_plain_attention(T, Hq, Hk, dh, E, shift):
    """Without transforms q, k, v are the column ranges of the latent rows, bit for bit, whether or not the rows are kept."""
    say("plain heads", T, Hq, Hk, dh, E, shift)
    cfg = P.CCAConfig(B=2, T=T, d_model=E, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh, k_seq=1, k_ch=1,
                      flags=P.CCA_FLAGS_MHA | shift)
    x, w_down = rnd(2, T, E, seed=1), rnd(E, cfg.n_lat, seed=2, scale=0.02)
    w = P.CCAWeights(w_down=w_down, w_out=rnd(cfg.e_q, E, seed=4, scale=0.02))
    saved = P.CCASaved.allocate(cfg, "cuda")
    for t in (saved.lat, saved.q, saved.k, saved.v):
        t.fill_(float("nan"))
    saved.rnorm.fill_(float("nan"))
    out = P.cca_forward(cfg, w, x, saved=saved)
    bare = P.cca_forward(cfg, w, x)
    lat = P.cca_down_project(cfg, x, w_down)
    torch.cuda.synchronize()
    check_product(lat.view(2 * T, -1), x.view(2 * T, E).double() @ w_down.double(), E)
    assert torch.equal(saved.lat, lat)
    e_q, e_k = cfg.e_q, cfg.e_q + cfg.e_kv
    assert torch.equal(saved.q.reshape(2, T, -1), lat[..., :e_q])
    assert torch.equal(saved.k.reshape(2, T, -1), lat[..., e_q:e_k])
    v = lat[..., e_k:].clone()
    if shift:
        v[:, 1:, cfg.e_kv // 2:] = lat[:, :-1, e_k + cfg.e_kv // 2:]
        v[:, 0, cfg.e_kv // 2:] = 0
    assert torch.equal(saved.v.reshape(2, T, -1), v)
    assert bool((saved.rnorm == 1).all())
    assert float((out.double() - bare.double()).norm()) <= 2.0 ** -7 * float(out.double().norm())


@pytest.mark.parametrize("Hq,Hk,dh", [(2, 2, 64), (4, 2, 64), (4, 1, 64), (8, 1, 64), (3, 1, 128), (8, 1, 128), (1, 1, 256),
                                      (4, 1, 256)])
def test_decode_ragged_leaves_empty_splits_alone(Hq, Hk, dh):
    """Sequences from one key to the whole cache in one step, over a workspace full of NaN: each row is the row of a step of
    that sequence alone.  Both are the same sums in another split, rounded to bf16 before the projection (2^-9) and after."""
    say("ragged", Hq, Hk, dh)
    T, E = 1500, 1024
    pos = [0, 1, 31, 32, 63, 64, 127, 128, 255, 256, 511, 700, T - 1]
    B = len(pos)
    cfg = P.CCAConfig(B=B, T=T, d_model=E, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh)
    one = P.CCAConfig(B=1, T=T, d_model=E, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh)
    w = P.CCAWeights(w_down=rnd(E, cfg.n_lat, seed=1, scale=0.02), w_out=rnd(cfg.e_q, E, seed=2, scale=0.05),
                     w_conv_seq=rnd(cfg.e_q + cfg.e_kv, 2, seed=3), w_conv_ch=rnd(Hq + Hk, dh, dh, 2, seed=4, scale=(2 * dh) ** -0.5),
                     temp=rnd(Hk, seed=5, dtype=torch.float32))
    x = rnd(B, E, seed=6)

    def state(c, rows):
        s = P.CCADecodeState.allocate(c, "cuda")
        s.k_cache.copy_(rnd(B, T, Hk, dh, seed=7).reshape(B, *s.k_cache.shape[1:])[rows])
        s.v_cache.copy_(rnd(B, T, Hk, dh, seed=8).reshape(B, *s.v_cache.shape[1:])[rows])
        s.lat_ring.copy_(rnd(*((B,) + tuple(s.lat_ring.shape[1:])), seed=9)[rows])
        s.workspace.view(torch.float32).fill_(float("nan")) if s.workspace.numel() % 4 == 0 else s.workspace.fill_(255)
        return s

    out = P.cca_decode_step_ragged(cfg, w, x, state(cfg, slice(0, B)), torch.tensor(pos, dtype=torch.int32, device="cuda"), T - 1)
    for b, p in enumerate(pos):
        ref = P.cca_decode_step(one, w, x[b:b + 1], state(one, slice(b, b + 1)), p).double()
        assert bool(ref.isfinite().all())
        assert float((out[b].double() - ref[0]).norm()) <= 2.0 ** -7 * float(ref.norm()), (b, p)


@pytest.mark.parametrize("B,Hq,Hk,dh,E,last", [(8, 4, 4, 64, 512, 1999), (32, 1, 1, 64, 72, 599), (8, 2, 1, 128, 256, 1023), (2, 4, 1, 256, 1032, 511),
                                                (1, 8, 2, 128, 1024, 900), (1, 16, 2, 128, 2056, 127)])
def test_up_projection_combines_the_splits(B, Hq, Hk, dh, E, last):
    """Up to 2048 channels and eight splits the up-projection adds the splits itself, over a workspace full of NaN: bit for bit the rows
    of a step with one sequence (and so a launch) more, whose keys are split the same way."""
    say("combine", B, Hq, Hk, dh, E, last)
    per = [rules.decode_keys_per_split(n * Hk, last + 1, dh, True) for n in (B, 2 * B + 1)]
    splits = -(-(last + 1) // per[0])
    assert rules.decode_up_combines(B, Hq * dh, splits) and not rules.decode_up_combines(2 * B + 1, Hq * dh, splits) and per[0] == per[1]
    T, C = last + 1, 2 * B + 1
    cfg = lambda n: P.CCAConfig(B=n, T=T, d_model=E, n_q_heads=Hq, n_kv_heads=Hk, head_dim=dh)
    c = cfg(C)
    w = P.CCAWeights(w_down=rnd(E, c.n_lat, seed=1, scale=0.02), w_out=rnd(c.e_q, E, seed=2, scale=0.05),
                     w_conv_seq=rnd(c.e_q + c.e_kv, 2, seed=3), w_conv_ch=rnd(Hq + Hk, dh, dh, 2, seed=4, scale=(2 * dh) ** -0.5),
                     temp=rnd(Hk, seed=5, dtype=torch.float32))
    x = rnd(C, E, seed=6)
    edges = [last, 0, per[0] - 1, per[0], last // 2, 1, last - 1, 2 * per[0]]
    pos = [min(edges[b % 8], last) for b in range(C)]

    def step(n):
        s = P.CCADecodeState.allocate(cfg(n), "cuda")
        s.k_cache.copy_(rnd(C, T, Hk, dh, seed=7).reshape(C, *s.k_cache.shape[1:])[:n])
        s.v_cache.copy_(rnd(C, T, Hk, dh, seed=8).reshape(C, *s.v_cache.shape[1:])[:n])
        s.lat_ring.copy_(rnd(*((C,) + tuple(s.lat_ring.shape[1:])), seed=9)[:n])
        s.workspace.fill_(255)
        return P.cca_decode_step_ragged(cfg(n), w, x[:n], s, torch.tensor(pos[:n], dtype=torch.int32, device="cuda"), last)

    few, more = step(B), step(C)
    torch.cuda.synchronize()
    assert bool(few.isfinite().all()) and torch.equal(few, more[:B])
