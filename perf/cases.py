"""Performance cases: the calls a user of this library makes, over the sizes it is used at.

Every case is one layer (E = d_model wide) driven through the Python binding:

  prefill   ``cca_forward`` on prepared weights: inference over whole sequences;
  train     ``cca_forward`` keeping the intermediates, then ``cca_backward``: a training step of the layer (the weights
            change between steps, so nothing is prepared);
  decode    ``cca_decode_step``: one new token for each of B sequences of the same length;
  ragged    ``cca_decode_step_ragged``: the same for a serving batch of mixed lengths.

Layouts are those of the repository's workloads and latency grids: CCGQA (more query than KV heads), CCA (equal counts),
both with every transform on, and the plain MHA / GQA baseline through the same kernels (``paper`` False).  ``T`` is the
sequence length (decode: the position of the newest token plus one), ``cap`` the capacity of a decode cache.
"""
from __future__ import annotations

import math

import torch

import paper_2510_04476_amd as P

DEV = "cuda"


def _case(kind, B, T, E, Hq, Hk, dh, paper=True, causal=True, dtype="bf16", k_seq=2, k_ch=2, cap=0, name=None):
    c = dict(kind=kind, B=B, T=T, E=E, Hq=Hq, Hk=Hk, dh=dh, paper=paper, causal=causal, dtype=dtype, k_seq=k_seq,
             k_ch=k_ch, cap=cap)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user, chat-length context: the smallest call, where launches and latency count
        _case("decode", 1, 1000, 2048, 8, 2, 128, cap=4096, name="decode_one"),
        # full serving batch over the longest cache: the decode workload of bench.py
        _case("decode", 32, 16384, 2048, 8, 2, 128, cap=16384, name="decode_batch_16k"),
        # continuous batching: an odd number of sequences of mixed lengths, narrow heads
        _case("ragged", 13, 5003, 2048, 16, 4, 64, cap=8192, name="decode_ragged"),
        # a short prompt: the smallest sequence of the latency grid
        _case("prefill", 1, 512, 2048, 8, 2, 128, name="prefill_short"),
        # a few prompts of one odd length, plain CCA heads
        _case("prefill", 3, 1531, 2048, 8, 8, 64, name="prefill_ragged"),
        # a medium prompt on the plain multi-head baseline
        _case("prefill", 1, 4096, 2048, 16, 16, 128, paper=False, name="prefill_mha"),
        # bidirectional encoder use at the widest head
        _case("prefill", 2, 3000, 2048, 4, 1, 256, causal=False, name="prefill_wide_encoder"),
        # long-context prefill: the benchmark's shape
        _case("prefill", 1, 16384, 2048, 8, 2, 128, name="prefill_16k"),
        # training on short sequences
        _case("train", 2, 512, 2048, 8, 2, 128, name="train_short"),
        # training on a batch of odd-length sequences, narrow heads
        _case("train", 4, 1999, 2048, 16, 4, 64, name="train_ragged"),
        # long-context training: the benchmark's shape, forward and backward
        _case("train", 1, 16384, 2048, 8, 2, 128, name="train_16k"),
        # 32-bit storage (reference runs, numerics work): four times the named tiny workload's length
        _case("train", 1, 1000, 256, 2, 2, 32, dtype="f32", name="train_f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "train", "train", "decode", "ragged", "f32"])
    if kind == "f32":
        dh = rng.choice([32, 64])
        Hk = rng.choice([1, 2])
        Hq = Hk * rng.choice([1, 2])
        return _case(rng.choice(["prefill", "train"]), 1, _log_int(rng, 64, 64000 // (Hq * dh)), 256, Hq, Hk, dh,
                     dtype="f32")
    paper = rng.random() < 0.8 or kind in ("decode", "ragged")
    E = rng.choice([1024, 1536, 2048])
    dh = rng.choice([64, 128, 128, 256])
    if paper:  # query compression 2 or 4, one to eight query heads per KV head
        Hq = E // (rng.choice([2, 4]) * dh)
        Hk = Hq // rng.choice([r for r in (1, 2, 3, 4, 6, 8) if Hq % r == 0])
    else:
        Hq = E // dh
        Hk = Hq // rng.choice([r for r in (1, 8) if Hq % r == 0])
    k_seq, k_ch = rng.choice([(2, 2), (2, 2), (2, 2), (3, 1)])
    if kind in ("decode", "ragged"):
        B = _log_int(rng, 1, 48)
        T = _log_int(rng, 100, min(16384, 32 * 16384 // B))
        return _case(kind, B, T, E, Hq, Hk, dh, k_seq=k_seq, k_ch=k_ch, cap=-(-T // 1024) * 1024)
    causal = rng.random() < 0.8
    # at most the work of the longest listed case: the wide heads, the baseline and the non-causal form do more per token
    most = 16384 if kind == "prefill" else 12288
    if not paper or not causal or dh == 256:
        most //= 2
    T = _log_int(rng, 64, most)
    B = max(1, min(8, most // T, _log_int(rng, 1, 8)))
    return _case(kind, B, T, E, Hq, Hk, dh, paper=paper, causal=causal, k_seq=k_seq, k_ch=k_ch)


def _config(c):
    flags = P.CCA_FLAGS_PAPER if c["paper"] else P.CCA_FLAGS_MHA
    if not c["causal"]:
        flags &= ~P.CCA_CAUSAL
    return P.CCAConfig(B=c["B"], T=c["cap"] or c["T"], d_model=c["E"], n_q_heads=c["Hq"], n_kv_heads=c["Hk"],
                       head_dim=c["dh"], k_seq=c["k_seq"] if c["paper"] else 1, k_ch=c["k_ch"] if c["paper"] else 1,
                       dtype=P.CCA_BF16 if c["dtype"] == "bf16" else P.CCA_F32, flags=flags)


def _ring(c):
    """(depth of a decode state's ring of latent rows, taps of the two convolutions together)"""
    taps = c["k_seq"] + c["k_ch"] - 1
    return max(taps - 1, 1) + 1, taps


def _inputs(c, seed):
    """Weights and activations from the seed alone.  Scales as a trained layer's: unit hidden states, projections that
    keep them there, convolution filters of gain one, temperatures spread around zero."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    B, T, E, Hq, Hk, dh = (c[k] for k in ("B", "T", "E", "Hq", "Hk", "dh"))
    e_q, e_kv, n_lat = Hq * dh, Hk * dh, (Hq + 2 * Hk) * dh

    def rnd(*shape, scale=1.0, dtype=dt):
        return (torch.randn(*shape, generator=gen, device=DEV) * scale).to(dtype)

    i = dict(w_down=rnd(E, n_lat, scale=0.02), w_out=rnd(e_q, E, scale=0.02))
    if c["paper"]:
        i.update(w_conv_seq=rnd(e_q + e_kv, c["k_seq"], scale=c["k_seq"] ** -0.5),
                 w_conv_ch=rnd(Hq + Hk, dh, dh, c["k_ch"], scale=(dh * c["k_ch"]) ** -0.5),
                 temp=rnd(Hk, scale=0.5, dtype=torch.float32))
    if c["kind"] in ("prefill", "train"):
        i["x"] = rnd(B, T, E)
    if c["kind"] == "train":
        # the upstream gradient of a loss in its course: noise, and a pull of each token's output along its own value
        v = (i["x"].float() @ i["w_down"][:, e_q + e_kv:].float()).view(B, T, Hk, 1, dh)
        own = v.expand(B, T, Hk, Hq // Hk, dh).reshape(B, T, e_q) @ i["w_out"].float()
        i["d_out"] = (own + torch.randn(own.shape, generator=gen, device=DEV)).to(dt)
    if c["kind"] in ("decode", "ragged"):
        P_, _ = _ring(c)
        beta = i["temp"].exp().view(1, 1, Hk, 1)
        k = torch.randn(B, c["cap"], Hk, dh, generator=gen, device=DEV)
        # cached keys as the prefill leaves them: length sqrt(d_h) * beta
        i["k"] = (k * (beta * math.sqrt(dh) / k.norm(dim=-1, keepdim=True))).to(dt)
        i["v"] = rnd(B, c["cap"], Hk, dh, scale=0.02 * math.sqrt(E))
        i["ring"] = rnd(B, P_, n_lat, scale=0.02 * math.sqrt(E))
        i["x"] = rnd(B, E)
        if c["kind"] == "ragged":  # one sequence at the full length, the others anywhere below
            pos = (torch.rand(B, generator=gen, device=DEV) * c["T"]).to(torch.int32)
            pos[B // 2] = c["T"] - 1
            i["pos"] = pos.clamp_(0, c["T"] - 1)
    return i


def prepare(case, seed):
    cfg, i = _config(case), _inputs(case, seed)
    w = P.CCAWeights(w_down=i["w_down"], w_out=i["w_out"], w_conv_seq=i.get("w_conv_seq"), w_conv_ch=i.get("w_conv_ch"),
                     temp=i.get("temp"))
    s = dict(kind=case["kind"], cfg=cfg, w=w, x=i["x"])
    if case["kind"] == "prefill":
        s.update(w=P.cca_prepare(cfg, w), workspace=P.new_workspace(cfg, DEV))
    elif case["kind"] == "train":
        s.update(d_out=i["d_out"], saved=P.CCASaved.allocate(cfg, DEV), workspace=P.new_workspace(cfg, DEV),
                 grads=P.CCAGrads.allocate_like(w), bwd_workspace=P.new_backward_workspace(cfg, DEV))
    else:
        nbytes, _ = P.cca_decode_workspace_size(cfg)
        s["state"] = P.CCADecodeState(i["k"], i["v"], i["ring"], torch.empty(nbytes, dtype=torch.uint8, device=DEV))
        s["pos"] = i["pos"] if case["kind"] == "ragged" else case["T"] - 1
        s["max_pos"] = case["T"] - 1
    return s


def run(s):
    cfg, w, x = s["cfg"], s["w"], s["x"]
    if s["kind"] == "prefill":
        return P.cca_forward(cfg, w, x, workspace=s["workspace"])
    if s["kind"] == "train":
        out = P.cca_forward(cfg, w, x, saved=s["saved"], workspace=s["workspace"])
        d_x, g = P.cca_backward(cfg, w, x, s["saved"], s["d_out"], grads=s["grads"], workspace=s["bwd_workspace"])
        return dict(out=out, d_x=d_x, w_down=g.w_down, w_out=g.w_out, w_conv_seq=g.w_conv_seq, w_conv_ch=g.w_conv_ch,
                    temp=g.temp)
    st = s["state"]
    if s["kind"] == "ragged":
        out = P.cca_decode_step_ragged(cfg, w, x, st, s["pos"], s["max_pos"])
    else:
        out = P.cca_decode_step(cfg, w, x, st, s["pos"])
    return dict(out=out, k=st.k_cache, v=st.v_cache, ring=st.lat_ring)  # the state as the step leaves it


def work(case):
    B, T, E, Hq, Hk, dh = (case[k] for k in ("B", "T", "E", "Hq", "Hk", "dh"))
    es = 2 if case["dtype"] == "bf16" else 4
    e_q, e_kv, n_lat = Hq * dh, Hk * dh, (Hq + 2 * Hk) * dh
    taps = case["k_seq"] + case["k_ch"] - 1
    weights = E * n_lat + e_q * E + ((e_q + e_kv) * (case["k_seq"] + dh * case["k_ch"]) if case["paper"] else 0)
    conv = 2.0 * (e_q + e_kv) * (case["k_seq"] + dh * case["k_ch"]) if case["paper"] else 0.0  # per token
    proj = 2.0 * E * (n_lat + e_q)
    if case["kind"] in ("decode", "ragged"):
        # a ragged batch: uniform lengths below T, half of it on average
        keys = B * T if case["kind"] == "decode" else T + (B - 1) * T / 2
        return dict(bytes=es * (2.0 * keys * e_kv + weights + B * (2 * E + taps * n_lat + 2 * e_kv)),
                    flops=B * (proj + conv) + 4.0 * keys * e_q)
    attn = 4.0 * B * T * T * e_q * (0.5 if case["causal"] else 1.0)
    fwd = B * T * (proj + conv) + attn
    if case["kind"] == "prefill":
        return dict(bytes=es * (2.0 * B * T * E + weights), flops=fwd)
    # training: x and d_out read, out and d_x written, each weight read and its gradient written; twice the forward's
    # products in the backward, and the scores once more
    return dict(bytes=es * (4.0 * B * T * E + 2 * weights), flops=3.0 * fwd + 0.5 * attn)


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "max": 1e-3}
    if case["kind"] == "train":
        # the filter gradients are sums over all tokens of products of bf16-stored tensors
        return {"rel": 2e-2}
    return {"rel": 1e-2}


# ---- the block in 64 bits, from its definition ---------------------------------------------------------------------


def _shift(u, s):
    return u if s == 0 else torch.nn.functional.pad(u, (0, 0) * (u.dim() - 2) + (s, 0))[:, : u.shape[1]]


def _transforms(c, i, lat, positions):
    """lat (B,T,N) -> q (B,T,Hq,dh), k, v (B,T,Hk,dh); positions (B,T) or (T,) for the rotary angles."""
    B, T, _ = lat.shape
    Hq, Hk, dh = c["Hq"], c["Hk"], c["dh"]
    e_q, e_kv = Hq * dh, Hk * dh
    q0, k0 = lat[..., :e_q].view(B, T, Hq, dh), lat[..., e_q:e_q + e_kv].view(B, T, Hk, dh)
    v = lat[..., e_q + e_kv:]
    if not c["paper"]:
        return q0, k0, v.view(B, T, Hk, dh)
    half = e_kv // 2
    v = torch.cat([v[..., :half], _shift(v[..., half:], 1)], -1).view(B, T, Hk, dh)
    u, w0, w1 = lat[..., :e_q + e_kv], i["w_conv_seq"], i["w_conv_ch"]
    y = sum(w0[:, j] * _shift(u, c["k_seq"] - 1 - j) for j in range(c["k_seq"])).view(B, T, Hq + Hk, dh)
    z = []
    for h in range(Hq + Hk):
        z.append(sum(_shift(y[:, :, h], c["k_ch"] - 1 - j) @ w1[h, :, :, j].t().contiguous() for j in range(c["k_ch"])))
    z = torch.stack(z, 2)
    m_q = 0.5 * (q0 + k0.repeat_interleave(Hq // Hk, 2))
    q, k = z[:, :, :Hq] + m_q, z[:, :, Hq:] + m_q.view(B, T, Hk, Hq // Hk, dh).mean(3)
    q = q * (math.sqrt(dh) / q.norm(dim=-1, keepdim=True))
    k = k * (math.sqrt(dh) / k.norm(dim=-1, keepdim=True)) * i["temp"].exp().view(Hk, 1)
    theta = 10000.0 ** (-2.0 * torch.arange(dh // 2, dtype=torch.float64, device=DEV) / dh)
    ang = positions.double().unsqueeze(-1) * theta
    ang = ang.view(-1, ang.shape[-2], 1, dh // 2)

    def rope(t):
        a, b = t[..., : dh // 2], t[..., dh // 2:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

    return rope(q), rope(k), v


def _rows(c, T, chunk=2048):
    for r0 in range(0, T, chunk):
        r1 = min(T, r0 + chunk)
        yield r0, r1, (r1 if c["causal"] else T)


def _probs(c, q, k, r0, r1, s1):
    s = (q @ k.t().contiguous()) / math.sqrt(c["dh"])
    if c["causal"]:
        s = s.masked_fill(torch.arange(s1, device=DEV) > torch.arange(r0, r1, device=DEV)[:, None], -math.inf)
    return torch.softmax(s, -1)


def _attend(c, q, k, v):
    B, T, Hq, dh = q.shape
    o = torch.empty_like(q)
    for b in range(B):
        for h in range(Hq):
            g = h // (Hq // c["Hk"])
            for r0, r1, s1 in _rows(c, T):
                o[b, r0:r1, h] = _probs(c, q[b, r0:r1, h], k[b, :s1, g], r0, r1, s1) @ v[b, :s1, g]
    return o.reshape(B, T, Hq * dh)


def _attend_backward(c, q, k, v, d_o):
    B, T, Hq, dh = q.shape
    d_o = d_o.view(B, T, Hq, dh)
    d_q, d_k, d_v = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for b in range(B):
        for h in range(Hq):
            g = h // (Hq // c["Hk"])
            for r0, r1, s1 in _rows(c, T):
                qh, kh, vh, do = q[b, r0:r1, h], k[b, :s1, g], v[b, :s1, g], d_o[b, r0:r1, h]
                p = _probs(c, qh, kh, r0, r1, s1)
                d_p = do @ vh.t().contiguous()
                d_s = p * (d_p - (p * d_p).sum(-1, keepdim=True)) / math.sqrt(dh)
                d_v[b, :s1, g] += p.t().contiguous() @ do
                d_q[b, r0:r1, h] = d_s @ kh
                d_k[b, :s1, g] += d_s.t().contiguous() @ qh
    return d_q, d_k, d_v


def _exact_decode(c, i):
    B, Hq, Hk, dh = c["B"], c["Hq"], c["Hk"], c["dh"]
    P_, taps = _ring(c)
    pos = i["pos"].tolist() if c["kind"] == "ragged" else [c["T"] - 1] * B
    ring, k_cache, v_cache = i["ring"].clone(), i["k"].clone(), i["v"].clone()
    o = torch.empty(B, Hq * dh, dtype=torch.float64, device=DEV)
    for b, t in enumerate(pos):
        ring[b, t % P_] = i["x"][b] @ i["w_down"]
        first = max(0, t - max(taps - 1, 1))  # tokens before the sequence's start read as zero
        lat = torch.stack([ring[b, s % P_] for s in range(first, t + 1)]).unsqueeze(0)
        q, k, v = _transforms(c, i, lat, torch.arange(first, t + 1, device=DEV))
        k_cache[b, t], v_cache[b, t] = k[0, -1], v[0, -1]
        for h in range(Hq):
            kh = k_cache[b, : t + 1, h // (Hq // Hk)]
            p = torch.softmax(kh @ q[0, -1, h] / math.sqrt(dh), 0)
            o[b, h * dh:(h + 1) * dh] = p @ v_cache[b, : t + 1, h // (Hq // Hk)]
    return dict(out=o @ i["w_out"], k=k_cache, v=v_cache, ring=ring)


def exact(case, seed):
    c, i = case, {k: v if k == "pos" else v.double() for k, v in _inputs(case, seed).items()}
    if c["kind"] in ("decode", "ragged"):
        return _exact_decode(c, i)
    train = c["kind"] == "train"
    names = [n for n in ("x", "w_down", "w_conv_seq", "w_conv_ch", "temp") if n in i]
    for n in names:
        i[n].requires_grad_(train)
    with torch.set_grad_enabled(train):
        q, k, v = _transforms(c, i, i["x"] @ i["w_down"], torch.arange(c["T"], device=DEV))
    with torch.no_grad():
        qd, kd, vd = (t.detach().contiguous() for t in (q, k, v))
        o = _attend(c, qd, kd, vd)
        out = o @ i["w_out"]
        if not train:
            return out
        d_w_out = o.flatten(0, 1).t().contiguous() @ i["d_out"].flatten(0, 1)
        d_o = i["d_out"] @ i["w_out"].t().contiguous()
        d_qkv = _attend_backward(c, qd, kd, vd, d_o)
    torch.autograd.backward((q, k, v), d_qkv)
    g = {n: i[n].grad for n in names}
    return dict(out=out, d_x=g["x"], w_down=g["w_down"], w_out=d_w_out, w_conv_seq=g.get("w_conv_seq"),
                w_conv_ch=g.get("w_conv_ch"), temp=g.get("temp"))
