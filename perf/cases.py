"""The work that is timed: what a program that serves a DBRX-shaped model asks of this library.

Three kinds of case, each through the package's public entry points:

- ``moe``: one Mixture-of-Experts layer (MoeLayer.forward), whole or one node's expert-parallel
  share of 4 of 16 experts with an fp32 partial sum, or a short stack of layers in place
  (MoeLayer.forward_stack);
- ``attn``: one self-attention block against a key/value cache (AttnLayer.forward), T new tokens
  at positions pos0 .. pos0+T-1;
- ``decoder``: whole decoder layers, attention with both norms and the MoE layer on the
  normalised input (AttnLayer.forward_norm, MoeLayer.forward_residual).

T runs from one generated token over a few tokens decoded together and short prompts up to a
2048-token prompt; positions from an empty cache to a long context.  The shapes are those of the
repository's workloads (d 6144, ffn 10752, 16 experts, top-4; 48 query heads over 8 key/value
heads of 128) and of its small test layers.

Inputs: normal activations and weights of trained-like scale (pre-activations of order one),
normal router weights, a normal per-expert router bias where the routing is skewed, cached keys
and values of earlier positions with a spread that keeps the softmax far from uniform.
"""
import math

import torch

import paper_2506_23635_amd as moe

# one DBRX-shaped layer
D, F, E, K = 6144, 10752, 16, 4
HEADS, KV, HD = 48, 8, 128
THETA, EPS = 5e5, 1e-5


def _moe(T, **kw):
    return dict(dict(kind="moe", T=T, d=D, f=F, E=E, k=K, begin=0, local=E, layers=1, f32=False,
                     skew=False), **kw)


def _attn(T, pos0, **kw):
    return dict(dict(kind="attn", T=T, pos0=pos0, d=D, heads=HEADS, kv=KV, hd=HD), **kw)


def _decoder(T, pos0, layers):
    return dict(kind="decoder", T=T, pos0=pos0, layers=layers, d=D, f=F, E=E, k=K, heads=HEADS,
                kv=KV, hd=HD)


def listed():
    return [
        # the smallest call: a small layer on a few tokens, where launches and latency count
        dict(_moe(16, d=256, f=512, E=8, k=2, local=8), name="moe_small_t16"),
        # one generated token through the whole layer
        dict(_moe(1), name="moe_t1"),
        # four tokens decoded together through consecutive layers in place
        dict(_moe(4, layers=2), name="moe_stack2_t4"),
        # one node's share at eight tokens, its partial sum in fp32 for the all-reduce
        dict(_moe(8, begin=4, local=4, f32=True), name="moe_share_t8"),
        # a short prompt (up to 128 tokens)
        dict(_moe(128), name="moe_t128"),
        # a long prompt with skewed expert loads
        dict(_moe(2048, skew=True), name="moe_t2048"),
        # one node's share of a 2000-token prompt
        dict(_moe(2000, begin=8, local=4, f32=True), name="moe_share_t2000"),
        # one generated token after a 2047-token context
        dict(_attn(1, 2047), name="attn_t1_p2047"),
        # sixteen tokens at once (the most the decode path takes) in a long context
        dict(_attn(16, 16000), name="attn_t16_p16000"),
        # a ragged piece of a prompt behind a cached prefix
        dict(_attn(300, 1000), name="attn_t300_p1000"),
        # a long prompt from an empty cache
        dict(_attn(2048, 0), name="attn_t2048_p0"),
        # one generated token through whole decoder layers
        dict(_decoder(1, 2047, 2), name="decoder2_t1_p2047"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["moe", "moe", "moe", "share", "small", "attn", "attn", "attn", "attn_small", "decoder"])
    if kind == "moe":
        T = _log_int(rng, 1, 2048)
        return _moe(T, skew=rng.random() < 0.5)
    if kind == "share":
        T = _log_int(rng, 1, 2048)
        return _moe(T, begin=4 * rng.randrange(4), local=4, f32=rng.random() < 0.5, skew=rng.random() < 0.5)
    if kind == "small":
        n = rng.choice([4, 8, 16, 32, 64])
        k = rng.randint(1, min(8, n))
        return _moe(_log_int(rng, 1, 2000), d=256 * rng.randint(1, 6), f=128 * rng.randint(1, 16), E=n,
                    k=k, local=n, skew=rng.random() < 0.5)
    if kind == "attn":
        T = _log_int(rng, 1, 2048)
        return _attn(T, _log_int(rng, 1, 18000 if T <= 512 else 4096) - 1)
    if kind == "attn_small":
        hd = rng.choice([64, 128])
        kv = rng.choice([1, 2, 8])
        heads = kv * rng.choice([2, 4, 8]) if kv > 1 else 8
        while heads * hd % 256 or (heads + 2 * kv) * hd % 256:
            heads += kv
        return _attn(_log_int(rng, 1, 1500), _log_int(rng, 1, 6000) - 1, d=256 * rng.randint(1, 8),
                     heads=heads, kv=kv, hd=hd)
    return _decoder(rng.randint(1, 16), _log_int(rng, 1, 8000), rng.randint(1, 2))


# ------------------------------------------------------------------ inputs --

_KINDS = {"x": 1, "router": 2, "bias": 3, "gate": 4, "up": 5, "down": 6, "gamma": 7, "gamma2": 8,
          "wqkv": 9, "wo": 10, "k": 11, "v": 12}


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _normal(seed, kind, shape, sigma, dtype=torch.bfloat16, layer=0, expert=0):
    """N(0, sigma) of one stream of the seed, made on the GPU."""
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(((seed * 1009 + layer) * 257 + expert) * 31 + _KINDS[kind])
    return torch.randn(shape, generator=g, device=dev, dtype=dtype).mul_(sigma)


def _x(c, seed):
    return _normal(seed, "x", (c["T"], c["d"]), 1.0)


def _router(c, seed, layer):
    wr = _normal(seed, "router", (c["d"], c["E"]), 1.6 / math.sqrt(c["d"]), torch.float32, layer)
    bias = _normal(seed, "bias", (c["E"],), 1.0, torch.float32, layer) if c.get("skew") else None
    return wr, bias


def _expert(c, seed, layer, e):
    s_in, s_out = 1.5 / math.sqrt(c["d"]), 1.0 / math.sqrt(c["f"])
    return (_normal(seed, "gate", (c["d"], c["f"]), s_in, layer=layer, expert=e),
            _normal(seed, "up", (c["d"], c["f"]), s_in, layer=layer, expert=e),
            _normal(seed, "down", (c["f"], c["d"]), s_out, layer=layer, expert=e))


def _attn_weights(c, seed, layer):
    nqkv = (c["heads"] + 2 * c["kv"]) * c["hd"]
    gamma = _normal(seed, "gamma", (c["d"],), 0.1, torch.float32, layer).add_(1.0)
    wqkv = _normal(seed, "wqkv", (c["d"], nqkv), 1.5 / math.sqrt(c["d"]), layer=layer)
    wo = _normal(seed, "wo", (c["heads"] * c["hd"], c["d"]), 1.0 / math.sqrt(c["heads"] * c["hd"]), layer=layer)
    return gamma, wqkv, wo


def _gamma2(c, seed, layer):
    return _normal(seed, "gamma2", (c["d"],), 0.1, torch.float32, layer).add_(1.0)


def _prefix(c, seed, layer):
    """Keys and values of positions 0 .. pos0-1, [kv heads, pos0, head_dim]."""
    shape = (c["kv"], c["pos0"], c["hd"])
    return (_normal(seed, "k", shape, 1.5, layer=layer), _normal(seed, "v", shape, 1.5, layer=layer))


# ------------------------------------------------------------- preparation --

def _make_moe(c, seed):
    cfg = moe.make_config(c["d"], c["f"], c["E"], c["k"], c.get("begin", 0), c.get("local", c["E"]),
                          c["layers"], c["T"], moe.MOE_PARTIAL_F32 if c.get("f32") else 0)
    layer = moe.MoeLayer(cfg)
    for l in range(c["layers"]):
        layer.load_router(l, *_router(c, seed, l))
        for e in range(cfg.expert_begin, cfg.expert_begin + cfg.n_local_experts):
            layer.load_expert(l, e, *_expert(c, seed, l, e))
    return layer


def _make_attn(c, seed, layers):
    T, pos0 = c["T"], c["pos0"]
    max_seq = max(4096, (pos0 + T + 255) // 256 * 256)
    cfg = moe.make_attn_config(c["d"], c["heads"], c["kv"], c["hd"], layers, max_seq, max(T, 16), THETA, EPS)
    att = moe.AttnLayer(cfg)
    new = []
    for l in range(layers):
        att.load_layer(l, *_attn_weights(c, seed, l))
        att.load_post_norm(l, _gamma2(c, seed, l))
        kc, vc = (t.view(torch.bfloat16) for t in att.cache_views(l))
        kp, vp = _prefix(c, seed, l)
        kc[:, :pos0].copy_(kp)
        vc[:, :pos0].copy_(vp)
        new += [kc[:, pos0:pos0 + T], vc[:, pos0:pos0 + T]]
    return att, new


def prepare(case, seed):
    c = case
    s = {"case": c, "x": _x(c, seed)}
    if c["kind"] == "moe":
        s["moe"] = _make_moe(c, seed)
        s["y"] = torch.empty((c["T"], c["d"]), dtype=torch.float32 if c["f32"] else torch.bfloat16, device="cuda")
    else:
        s["attn"], s["new"] = _make_attn(c, seed, c.get("layers", 1))
        s["y"] = torch.empty_like(s["x"])
        if c["kind"] == "decoder":
            s["moe"] = _make_moe(c, seed)
            s["z"] = torch.empty_like(s["x"])
    return s


def run(state):
    c, x, y = state["case"], state["x"], state["y"]
    if c["kind"] == "moe":
        if c["layers"] == 1:
            state["moe"].forward(0, x, y)
        else:
            y.copy_(x)   # the stack works in place
            state["moe"].forward_stack(y)
        return y
    if c["kind"] == "attn":
        state["attn"].forward(0, x, y, c["pos0"])
        return {"y": y, "new": state["new"]}   # the block's output and the keys and values it appends
    z = state["z"]
    for l in range(c["layers"]):
        state["attn"].forward_norm(l, x, y, z, c["pos0"])
        state["moe"].forward_residual(l, z, y)
        x = y
    return {"y": y, "z": z, "new": state["new"]}


# ---------------------------------------------------------------- the work --

def _moe_work(c):
    """Per layer: the experts that T tokens touch (the mean over uniform routings), the router,
    tokens in and out; the products of the routed rows."""
    T, d, f, n, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    local = c.get("local", n)
    touched = local * (1.0 - (1.0 - k / n) ** T)
    rows = T * k * local / n
    out = 4 if c.get("f32") else 2
    return (touched * 6.0 * d * f + 4.0 * d * n + T * d * (2 + out), 6.0 * rows * d * f + 2.0 * T * d * n)


def _attn_work(c):
    T, pos0, d, H, G, hd = c["T"], c["pos0"], c["d"], c["heads"], c["kv"], c["hd"]
    nqkv = (H + 2 * G) * hd
    weights = 2.0 * d * (nqkv + H * hd)
    cache = 2.0 * 2 * G * hd * (pos0 + T) + 2.0 * 2 * G * hd * T
    seen = T * pos0 + T * (T + 1) / 2.0
    return (weights + cache + 4.0 * d + 4.0 * T * d, T * weights + 4.0 * H * hd * seen)


def work(case):
    c, n = case, case.get("layers", 1)
    b = f = 0.0
    if c["kind"] in ("moe", "decoder"):
        mb, mf = _moe_work(c)
        b, f = b + n * mb, f + n * mf
    if c["kind"] in ("attn", "decoder"):
        ab, af = _attn_work(c)
        b, f = b + n * ab, f + n * af
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Four times what the outputs differ by from the 64-bit results rounded to bf16 at the same
    points (measured: one MoE layer 4e-4, its fp32 partial sum 8e-5, the attention block 9.5e-4,
    chains of two layers 4e-3; at most 8e-3, 5e-3, 8e-3 and 2e-2 per value).  Sums in another
    order move a few bf16 roundings: of the activations between the two expert products, of the
    normalised input, of q, k, v and the attention output, and of the result.  fp32 partial sums
    keep only the first kind.  In a chain every layer adds."""
    if case["kind"] == "decoder" or case.get("layers", 1) > 1:
        return {"rel": 1.6e-2, "max": 8e-2}
    if case["kind"] == "attn":
        return {"rel": 4e-3, "max": 3.2e-2}
    if case["f32"]:
        return {"rel": 4e-4, "max": 2e-2}
    return {"rel": 1.6e-3, "max": 3.2e-2}


# ----------------------------------------------------------- 64-bit results --

def _bf16(v):
    return v.to(torch.float32).to(torch.bfloat16)


def _exact_moe(c, seed, layer, x):
    """The layer on bf16 x in 64 bits; the activations between the expert products are bf16, as
    the layer is defined."""
    xd = x.double()
    wr, bias = _router(c, seed, layer)
    logits = (xd @ wr.double()).float()
    if bias is not None:
        logits = logits + bias
    v, idx = torch.sort(logits, dim=1, descending=True, stable=True)
    idx = idx[:, :c["k"]]
    w = torch.softmax(v[:, :c["k"]].double(), dim=1)
    y = torch.zeros_like(xd)
    begin = c.get("begin", 0)
    for e in range(begin, begin + c.get("local", c["E"])):
        t, j = torch.nonzero(idx == e, as_tuple=True)
        if not t.numel():
            continue
        gate, up, down = _expert(c, seed, layer, e)
        a = xd[t]
        g = a @ gate.double()
        u = a @ up.double()
        h = _bf16(g * torch.sigmoid(g) * u).double()
        y.index_add_(0, t, (h @ down.double()) * w[t, j].unsqueeze(1))
    return y


def _norm64(x, gamma):
    xd = x.double()
    m = xd.mean(1, keepdim=True)
    var = ((xd - m) ** 2).mean(1, keepdim=True)
    return _bf16((xd - m) / torch.sqrt(var + EPS) * gamma.double())


def _exact_attn(c, seed, layer, x):
    """(x + attention in 64 bits, the new keys, the new values); q, k, v, the normalised input
    and the attention output are bf16, as the block is defined."""
    T, pos0, H, G, hd = c["T"], c["pos0"], c["heads"], c["kv"], c["hd"]
    gamma, wqkv, wo = _attn_weights(c, seed, layer)
    qkv = _norm64(x, gamma).double() @ wqkv.double()
    q, k, v = qkv.view(T, H + 2 * G, hd).split([H, G, G], dim=1)
    pos = torch.arange(pos0, pos0 + T, device=x.device, dtype=torch.float64)
    ang = pos[:, None] * THETA ** (-2.0 * torch.arange(hd // 2, device=x.device, dtype=torch.float64) / hd)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def turn(t):
        a, b = t[..., :hd // 2], t[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)

    q, k_new, v_new = _bf16(turn(q)), turn(k), v
    kp, vp = _prefix(c, seed, layer)
    keys = torch.cat([kp, _bf16(k_new).transpose(0, 1)], dim=1)       # [kv, positions, hd]
    vals = torch.cat([vp, _bf16(v_new).transpose(0, 1)], dim=1)
    seen = torch.arange(pos0 + T, device=x.device)[None, :] <= pos[:, None]
    a = torch.empty((T, H, hd), dtype=torch.bfloat16, device=x.device)
    for j in range(H):
        g = j // (H // G)
        s = (q[:, j].double() @ keys[g].double().t()) / math.sqrt(hd)
        p = torch.softmax(s.masked_fill(~seen, -math.inf), dim=1)
        a[:, j] = _bf16(p @ vals[g].double())
    y = x.double() + a.view(T, H * hd).double() @ wo.double()
    return y, k_new.transpose(0, 1), v_new.transpose(0, 1)


def exact(case, seed):
    c = case
    x = _x(c, seed)
    if c["kind"] == "moe":
        if c["layers"] == 1:
            return _exact_moe(c, seed, 0, x)
        for l in range(c["layers"]):
            y = x.double() + _bf16(_exact_moe(c, seed, l, x)).double()
            x = _bf16(y)
        return y
    if c["kind"] == "attn":
        y, k, v = _exact_attn(c, seed, 0, x)
        return {"y": y, "new": [k, v]}
    new = []
    for l in range(c["layers"]):
        y, k, v = _exact_attn(c, seed, l, x)
        new += [k, v]
        y = _bf16(y)
        z = _norm64(y, _gamma2(c, seed, l))
        out = y.double() + _bf16(_exact_moe(c, seed, l, z)).double()
        x = _bf16(out)
    return {"y": out, "z": z.double(), "new": new}
