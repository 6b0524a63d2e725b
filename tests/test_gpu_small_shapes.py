"""GPU checks of the kernels chosen for small and odd sizes, at the edges of their tiles, against plain fp32 / fp64
products of the same bf16 inputs."""
import sys

import pytest
import torch

import paper_2510_04476_amd as P

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
# of a tile's edge, contraction lengths of one slab, an odd number of slabs (no split over halves) and many
GEMM_CASES = [(1, 1, 1, 64, 64), (65, 1, 1, 64, 192), (127, 3, 1, 64, 320), (512, 8, 2, 128, 2048), (511, 4, 4, 64, 1024),
              (1000, 8, 2, 128, 2048), (1999, 16, 4, 64, 2048), (2050, 5, 5, 64, 1024), (4593, 8, 8, 64, 2048),
              (3001, 8, 2, 128, 2048), (4097, 16, 16, 128, 2048)]


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


# token rows x (query heads, head width, E): d W_out (e_q, E) = o^T d_out on every tile shape of the weight-gradient GEMM
# (64 x 64, 64 x 128, 128 x 128, split 256 x 256), with no, one and a few tokens in the last slab of 64
WGRAD_CASES = [(1, 1, 64, 64), (63, 3, 64, 256), (1000, 8, 64, 1024), (64, 8, 128, 2048), (129, 8, 128, 2048),
               (1023, 8, 128, 2048), (512, 12, 128, 2048), (2001, 12, 128, 2048), (9001, 8, 128, 2048)]


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
