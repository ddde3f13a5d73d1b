"""The workloads this library's speed is measured on.

A case is a dict of plain values; `listed()` names twelve and `draw(rng)`
gives more of the same ranges.  `prepare` makes what a program holds before
a call (inputs, packed weights, workspaces), `run` is one pass through the
public entry points, `work` the bytes and operations a pass cannot do
without, `exact` the same outputs in 64-bit torch, `tolerance` how far two
correct implementations may differ.

Three kinds of pass:
  layer   one MoE layer over a batch of tokens: route, group, expert FFN
          (and, by option, top-K slots, a permanent expert, the gate weight);
  stack   a decode step: group, then L pre-norm residual layers, then back
          to token order;
  router  the pre-gating router block over a batch of requests.
"""
import math

import torch

from paper_2410_19123_amd import _lib as L

DEV = "cuda:0"
RMS_EPS = 1e-5
# Logit bias of expert 0 in the skewed prefill (16 experts, about 40% of the
# tokens on expert 0).
SKEW_BIAS0 = 0.2826


def _layer(name, T, d, E, I, **opt):
    c = dict(kind="layer", name=name, T=T, d=d, E=E, I=I, dtype="bf16", ids="router",
             bias="zipf", K=1, slices=0, form="fused")
    c.update(opt)
    return c


def _stack(name, T, d, E, I, layers, ids):
    return dict(kind="stack", name=name, T=T, d=d, E=E, I=I, layers=layers, ids=ids,
                bias="zipf")


def _router(name, T, requests, cut, D=512, F=512, V=32000, E=8):
    return dict(kind="router", name=name, T=T, requests=requests, cut=cut, D=D, F=F, V=V, E=E)


def listed():
    return [
        # The small fp32 layer: launch latency and the fp32 kernels.
        _layer("layer_f32_256", 256, 512, 4, 512, dtype="f32", bias="none"),
        # A middle-sized layer of odd sizes in its separate calls (gather, FFN,
        # scale and ungroup), each output weighted by its gate probability.
        _layer("layer_weighted_1021", 1021, 2048, 8, 1000, form="weighted"),
        # A Llama-7B-shaped layer (11008 = 8 x 1376 neurons) over 2048 tokens.
        _layer("layer_2048", 2048, 4096, 8, 1376),
        # The same with a permanent expert every token passes through.
        _layer("layer_perm_2048", 2048, 4096, 8, 1376, slices=1),
        # The same with each token on its two highest-logit experts.
        _layer("layer_top2_2048", 2048, 4096, 8, 1376, K=2),
        # Prefill: many tokens, 16 experts, a skewed load.
        _layer("prefill_skew16", 16384, 4096, 16, 688, bias="skew"),
        # An expert-aware batch of 256 requests of 32 tokens whose experts are
        # known ahead (no router call), at the largest layer width.
        _layer("requests_256x32", 8192, 8192, 8, 3584, ids="requests", bias="none"),
        # Decode of a single request through all 32 layers: the smallest step.
        _stack("decode_1", 1, 4096, 8, 1376, 32, "router"),
        # Decode of 64 requests, routed once, through all 32 layers.
        _stack("decode_64", 64, 4096, 8, 1376, 32, "router"),
        # Decode of 64 requests that the expert-aware scheduler put on one
        # expert; the scheduler knows the counts.
        _stack("decode_64_batched", 64, 4096, 8, 1376, 32, "batched"),
        # The router block over the request batch, and over long prompts.
        _router("router_256x32", 8192, 256, "even"),
        _router("router_8x1024", 8192, 8, "even"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "stack", "stack", "router"])
    while True:
        if kind == "router":
            c = _router("", _log_int(rng, 1, 16384), 1, rng.choice(["even", "ragged"]),
                        D=128 * rng.choice([2, 4, 4, 4, 8]), F=_log_int(rng, 128, 1536),
                        V=rng.choice([1000, 32000]), E=rng.randint(1, 24))
            c["requests"] = _log_int(rng, max(1, c["T"] // 2048), max(1, c["T"] // 4))
        elif kind == "stack":
            c = _stack("", _log_int(rng, 1, 320), 64 * _log_int(rng, 16, 96), rng.randint(1, 24),
                       _log_int(rng, 256, 3584), rng.randint(2, 32),
                       rng.choice(["router", "fifo", "batched"]))
        else:
            f32 = rng.random() < 0.15
            c = _layer("", _log_int(rng, 1, 2048 if f32 else 16384),
                       64 * _log_int(rng, 8, 32 if f32 else 128), _log_int(rng, 1, 64),
                       _log_int(rng, 64, 1536 if f32 else 4096),
                       dtype="f32" if f32 else "bf16",
                       ids=rng.choice(["router", "router", "requests"]),
                       bias=rng.choice(["none", "zipf", "skew"]))
            if c["ids"] == "router":
                form = rng.choice(["fused", "fused", "weighted", "perm", "topk"])
                if form == "weighted":
                    c["form"] = form
                elif form == "perm":
                    c["slices"] = rng.randint(1, 2)
                elif form == "topk":
                    c["K"] = rng.randint(1, min(4, c["E"]))
        if _fits(c):
            del c["name"]
            return c


def _fits(c):
    w = work(c)
    if kind_bytes(c) > 10e9:
        return False
    return w["bytes"] <= 7.5e9 and w["flops"] <= (9e10 if c.get("dtype") == "f32" else 1.4e12)


def kind_bytes(c):
    """Bytes of the case's packed weights."""
    if c["kind"] == "router":
        return 2.0 * (c["V"] * c["D"] + 4 * c["D"] ** 2 + 3 * c["D"] * c["F"])
    s = 4 if c.get("dtype") == "f32" else 2
    Ip = (c["I"] + 63) // 64 * 64
    return 3.0 * s * c["d"] * Ip * (c["E"] + c.get("slices", 0)) * c.get("layers", 1)


# --- inputs ------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype=torch.bfloat16):
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    if std != 1.0:
        t.mul_(std)
    return t.to(dtype)


def _bias(c):
    e = torch.arange(c["E"], dtype=torch.float64)
    if c["bias"] == "none":
        return None
    if c["bias"] == "zipf":
        b = -torch.log(e + 1.0)
    else:
        b = -1.2 * torch.log(e.clamp(min=1.0))
        b[0] = SKEW_BIAS0
    return b.float().to(DEV)


def _features(c, seed):
    """Token features and, where the case routes, the router's weights."""
    g = _gen(seed)
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
    x = _normal(g, (c["T"], c["d"]), 1.0, dt)
    wr = _normal(g, (c["E"], c["d"]), 0.02, dt) if c["ids"] == "router" else None
    return x, wr, _bias(c)


def _given_ids(c, seed):
    """Expert ids known before the call: per request (32 tokens each), from a
    first-come batch (popularity 1/(e+1)), or a batch on one expert."""
    g = _gen(seed + 7919)
    T, E = c["T"], c["E"]
    if c["ids"] == "requests":
        r = torch.randint(E, ((T + 31) // 32,), generator=g, device=DEV)
        return r.repeat_interleave(32)[:T].int().contiguous()
    if c["ids"] == "fifo":
        p = 1.0 / torch.arange(1, E + 1, device=DEV, dtype=torch.float32)
        return torch.multinomial(p, T, replacement=True, generator=g).int()
    return torch.randint(E, (1,), generator=g, device=DEV).int().repeat(T)


def _weights(c, seed, layer):
    g = _gen(seed * 1009 + 104729 * (layer + 1))
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
    E, I, d = c["E"], c["I"], c["d"]
    return (_normal(g, (E, I, d), 0.02, dt), _normal(g, (E, I, d), 0.02, dt),
            _normal(g, (E, d, I), 0.02, dt))


def _permanent(c, seed):
    g = _gen(seed * 1009 + 15485863)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    P, d = c["I"] * c["slices"], c["d"]
    return (_normal(g, (P, d), 0.02, dt), _normal(g, (P, d), 0.02, dt),
            _normal(g, (d, P), 0.02, dt))


def _router_inputs(c, seed):
    g = _gen(seed)
    D, F, V, E, T, R = c["D"], c["F"], c["V"], c["E"], c["T"], c["requests"]
    w = dict(emb=_normal(g, (V, D), 1.0), wq=_normal(g, (D, D), 0.02),
             wk=_normal(g, (D, D), 0.02), wv=_normal(g, (D, D), 0.02),
             wo=_normal(g, (D, D), 0.02), w1=_normal(g, (F, D), 0.02),
             w3=_normal(g, (F, D), 0.02), w2=_normal(g, (D, F), 0.02),
             gate=_normal(g, (E, D), 0.02))
    w["tokens"] = torch.randint(V, (T,), generator=g, device=DEV).int()
    if c["cut"] == "even":
        offs = torch.arange(R + 1, device=DEV) * T // R
    else:
        cuts = torch.randint(T + 1, (R - 1,), generator=g, device=DEV).sort().values
        offs = torch.cat([torch.zeros(1, device=DEV), cuts, torch.full((1,), T, device=DEV)])
    w["req"] = offs.int().contiguous()
    return w


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "router":
        w = _router_inputs(c, seed)
        ws = L.readme_router_tf_workspace_bytes(c["T"], c["D"], c["F"])
        packed = L.readme_router_tf_pack(*(w[n] for n in ("wq", "wk", "wv", "wo", "w1", "w3",
                                                          "w2")))
        return dict(c=c, tokens=w["tokens"], req=w["req"], emb=w["emb"], gate=w["gate"],
                    packed=packed, ids=torch.empty(c["T"], dtype=torch.int32, device=DEV),
                    logits=torch.empty(c["T"], c["E"], dtype=torch.float32, device=DEV),
                    ws=torch.empty(ws, dtype=torch.uint8, device=DEV))
    x, wr, bias = _features(c, seed)
    T, d, E, I = c["T"], c["d"], c["E"], c["I"]
    n = T * c.get("K", 1)
    i32 = dict(dtype=torch.int32, device=DEV)
    s = dict(c=c, x=x, wr=wr, bias=bias if wr is not None else None,
             ids=torch.empty(T, **i32) if wr is not None else _given_ids(c, seed),
             counts=torch.empty(E, **i32), offsets=torch.empty(E + 1, **i32),
             perm=torch.empty(n, **i32), inv=torch.empty(n, **i32))
    if c["kind"] == "stack":
        s["x32"] = x.float()
        s["xres"], s["y"] = torch.empty_like(s["x32"]), torch.empty_like(s["x32"])
        s["packed"] = [L.readme_pack_experts(*_weights(c, seed, k)) for k in range(c["layers"])]
        s["ws"] = torch.empty(L.readme_moe_ffn_stack_workspace_bytes(T, d, I),
                              dtype=torch.uint8, device=DEV)
        s["host_counts"] = None
        if wr is None:  # the scheduler that formed the batch knows its counts
            s["host_counts"] = torch.bincount(s["ids"].long(), minlength=E).int().cpu().numpy()
        return s
    dt = x.dtype
    if c["slices"]:
        P = I * c["slices"]
        s["packed"] = L.readme_pack_experts_permanent(*_weights(c, seed, 0), *_permanent(c, seed))
        ws = L.readme_moe_ffn_permanent_workspace_bytes(dt, T, I, P)
    else:
        s["packed"] = L.readme_pack_experts(*_weights(c, seed, 0))
        ws = L.readme_moe_ffn_workspace_bytes(dt, n, I)
    s["ws"] = torch.empty(ws, dtype=torch.uint8, device=DEV)
    s["y"] = torch.empty_like(x)
    if c["K"] > 1 or c["form"] == "weighted":
        s["logits"] = torch.empty(T, E, dtype=torch.float32, device=DEV)
    if c["K"] > 1:
        s["pair_ids"] = torch.empty(n, **i32)
        s["gates"] = torch.empty(n, dtype=torch.float32, device=DEV)
        s["y_pairs"] = torch.empty(n, d, dtype=dt, device=DEV)
    if c["form"] == "weighted":
        s["xg"], s["yg"] = torch.empty_like(x), torch.empty_like(x)
        s["scale"] = torch.empty(T, dtype=torch.float32, device=DEV)
    return s


# --- one pass ----------------------------------------------------------------

def run(s):
    c = s["c"]
    if c["kind"] == "router":
        ids, logits, _ = L.readme_router_tf(s["tokens"], s["req"], s["emb"], s["packed"], c["F"],
                                            s["gate"], None, RMS_EPS, s["ids"], s["logits"],
                                            s["ws"])
        return {"ids": ids, "logits": logits}
    E, I, K = c["E"], c["I"], c.get("K", 1)
    if s["wr"] is not None:
        L.readme_route(s["x"], s["wr"], s["bias"], s["ids"], s.get("logits"))
    meta = (s["counts"], s["offsets"], s["perm"], s["inv"])
    if c["kind"] == "stack":
        L.readme_group_by_expert(s["ids"], E, s["x32"], *meta, s["xres"])
        L.readme_moe_ffn_stack(s["xres"], s["offsets"], s["packed"], E, I, RMS_EPS, s["ws"],
                               s["host_counts"])
        return {"ids": s["ids"], "y": L.readme_ungroup(s["xres"], s["inv"], s["y"])}
    if K > 1:
        L.readme_topk(s["logits"], K, s["pair_ids"], s["gates"])
        L.readme_group_by_expert(s["pair_ids"], E, None, *meta)
        L.readme_moe_ffn_topk(s["x"], s["perm"], s["offsets"], s["packed"], E, I, K,
                              s["y_pairs"], s["ws"])
        L.readme_combine_topk(s["y_pairs"], s["gates"], K, s["y"])
        return {"ids": s["pair_ids"], "gates": s["gates"], "perm": s["perm"], "y": s["y"]}
    if c["form"] == "weighted":
        L.readme_group_by_expert(s["ids"], E, s["x"], *meta, s["xg"])
        L.readme_moe_ffn(s["xg"], s["offsets"], s["packed"], E, I, s["yg"], s["ws"])
        L.readme_gate_weights(s["logits"], s["ids"], s["inv"], s["scale"])
        L.readme_ungroup_scaled(s["yg"], s["inv"], s["scale"], s["y"])
        return {"ids": s["ids"], "logits": s["logits"], "perm": s["perm"], "y": s["y"]}
    L.readme_group_by_expert(s["ids"], E, None, *meta)
    if c["slices"]:
        L.readme_moe_ffn_permanent_fused(s["x"], s["perm"], s["offsets"], s["packed"], E, I,
                                         I * c["slices"], s["y"], s["ws"])
    else:
        L.readme_moe_ffn_fused(s["x"], s["perm"], s["offsets"], s["packed"], E, I, s["y"],
                               s["ws"])
    return {"ids": s["ids"], "counts": s["counts"], "perm": s["perm"], "y": s["y"]}


# --- what a pass cannot do without -------------------------------------------

def _active(c):
    """Expected number of experts with tokens."""
    E, n = c["E"], c["T"] * c.get("K", 1)
    if c["ids"] == "batched":
        return 1.0
    if c["ids"] == "requests":
        n, p = (c["T"] + 31) // 32, [1.0 / E] * E
    elif c["ids"] == "fifo" or c["bias"] == "zipf":
        p = [1.0 / (e + 1) for e in range(E)]
    elif c["bias"] == "skew":
        p = [math.exp(SKEW_BIAS0)] + [e ** -1.2 for e in range(1, E)]
    else:
        p = [1.0] * E
    t = sum(p)
    return min(float(n), sum(1.0 - (1.0 - v / t) ** n for v in p))


def work(case):
    c = case
    T = c["T"]
    if c["kind"] == "router":
        D, F, E = c["D"], c["F"], c["E"]
        pairs = T * (T / c["requests"] + 1) / 2
        rows = min(T, c["V"])
        return {"bytes": 2 * (rows * D + 4 * D * D + 3 * D * F + E * D) + 4 * T * (2 + E),
                "flops": T * (8 * D * D + 6 * D * F + 2 * D * E) + 4 * D * pairs}
    d, E, I, K = c["d"], c["E"], c["I"], c.get("K", 1)
    s = 4 if c.get("dtype") == "f32" else 2
    layers = c.get("layers", 1)
    router = c["ids"] == "router"
    weights = 3 * I * d * s * (_active(c) + c.get("slices", 0))
    rows = T * d * (4 + 4 + 2 * router if c["kind"] == "stack" else 2 * s)
    return {"bytes": layers * weights + rows + router * E * d * s + 4 * T * K,
            "flops": layers * 6 * T * d * I * (K + c.get("slices", 0)) + router * 2 * T * d * E}


def tolerance(case):
    """About four times the difference seen between this library and the same
    layer in torch with the same roundings and its own summation order: 3.5e-4
    (one bf16 unit at most) for a bf16 layer, 5e-7 for fp32, 9e-3 for 32
    stacked layers, where one rounding travels through the rest."""
    c = case
    if c["kind"] == "router":
        return {"rel": 4e-3, "max": 4e-2, "differ": 1e-2}
    if c["kind"] == "stack":
        return {"rel": 3e-2, "max": 2e-1, "differ": 0.0}
    if c["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5, "differ": 0.0}
    return {"rel": 2e-3, "max": 3.2e-2, "differ": 0.0}


# --- the same outputs in 64 bits ---------------------------------------------

def _silu(z):
    return z / (1.0 + torch.exp(-z))


def _ffn64(x, ids, w):
    """Rows of x through their expert's SwiGLU FFN, in 64 bits."""
    y = torch.zeros_like(x)
    for e in range(w[0].shape[0]):
        at = (ids == e).nonzero().flatten()
        if at.numel():
            h = x[at]
            h = _silu(h @ w[0][e].double().T) * (h @ w[1][e].double().T)
            y[at] = h @ w[2][e].double().T
    return y


def _route64(c, x, wr, bias, seed):
    if wr is None:
        return _given_ids(c, seed).long(), None
    logits = x @ wr.double().T
    if bias is not None:
        logits = logits + bias.double()
    return logits.argmax(1), logits


def _rms64(x):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + RMS_EPS)


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "router":
        return _exact_router(c, seed)
    x, wr, bias = _features(c, seed)
    x = x.double()
    ids, logits = _route64(c, x, wr, bias, seed)
    if c["kind"] == "stack":
        for k in range(c["layers"]):
            x = x + _ffn64(_rms64(x), ids, _weights(c, seed, k))
        return {"ids": None, "y": x}
    w = _weights(c, seed, 0)
    if c["K"] > 1:
        top, slot = logits.sort(dim=1, descending=True, stable=True)
        gates = torch.softmax(top[:, :c["K"]], 1)
        y = sum(gates[:, k:k + 1] * _ffn64(x, slot[:, k], w) for k in range(c["K"]))
        return {"ids": None, "gates": gates.flatten(), "perm": None, "y": y}
    y = _ffn64(x, ids, w)
    if c["form"] == "weighted":
        y = y * torch.softmax(logits, 1).gather(1, ids[:, None])
        return {"ids": None, "logits": logits, "perm": None, "y": y}
    if c["slices"]:
        y = y + _ffn64(x, torch.zeros_like(ids), [p[None] for p in _permanent(c, seed)])
    return {"ids": None, "counts": None, "perm": None, "y": y}


def _exact_router(c, seed):
    w = {k: v.double() if v.is_floating_point() else v.long()
         for k, v in _router_inputs(c, seed).items()}
    T, D = c["T"], c["D"]
    t = torch.arange(T, device=DEV)
    req = torch.searchsorted(w["req"], t, right=True) - 1  # the last request starting at or before t
    pos = (t - w["req"][req]).double()
    x = w["emb"][w["tokens"]]
    a = _rms64(x)
    q, k, v = (a @ w[n].T for n in ("wq", "wk", "wv"))
    ang = pos[:, None] * 10000.0 ** (-torch.arange(64, device=DEV, dtype=torch.float64) / 64.0)
    cos, sin = torch.cos(ang), torch.sin(ang)
    see = (req[:, None] == req[None, :]) & (t[:, None] >= t[None, :])
    o = torch.empty_like(x)
    for h in range(D // 128):
        at = slice(128 * h, 128 * h + 128)

        def turn(z):
            lo, hi = z[:, :64], z[:, 64:]
            return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], 1)

        p = turn(q[:, at]) @ turn(k[:, at]).T / math.sqrt(128.0)
        p = torch.softmax(p.masked_fill_(~see, -math.inf), 1)
        o[:, at] = p @ v[:, at]
        del p
    x = x + o @ w["wo"].T
    m = _rms64(x)
    x = x + (_silu(m @ w["w1"].T) * (m @ w["w3"].T)) @ w["w2"].T
    return {"ids": None, "logits": _rms64(x) @ w["gate"].T}
