"""The work this library is measured on: one MoE layer through the package's public calls.

Every case is one layer of a model: a forward pass (``moe_layer_forward``) as serving runs it, or a training step
(input-major weight copies where the weights have just been updated, ``moe_layer_forward``, ``moe_layer_backward``).
Shapes are those of the repository's workloads (``workloads/moe_inputs.py``), of its decode and backward benches, and
generic ones around them: few tokens, ragged token counts, feature counts that are no multiple of a kernel's tile,
routers wider than 64 experts, float32 experts.
"""
from __future__ import annotations

import math

import torch

import paper_2205_10034_amd as M
from workloads.moe_inputs import WORKLOADS, zipf_masses


def _case(name, **kw):
    c = dict(kind="layer", T=0, d=0, f=0, E=0, k=1, cf=0.0, renorm=False, act="gelu", dtype="bf16", layout="output_major",
             bias=False, router_bias="none", residual=False, refresh=False, grads="f32")
    c.update(kw)
    if name:
        c["name"] = name
    return c


def _of(workload):
    wl = WORKLOADS[workload]
    return dict(T=wl.T, d=wl.d_model, f=wl.d_ff, E=wl.E, k=wl.k, cf=wl.capacity_factor, renorm=wl.renormalize, act=wl.act,
                dtype=wl.dtype, router_bias=wl.router_bias)


def listed():
    ring, gpt, large = _of("ring"), _of("gpt"), _of("large")
    return [
        # one request generating one token on a layer of the 64-expert stack: the smallest call, launches and latency
        _case("decode_one", **{**ring, "T": 1, "residual": True}),
        # a handful of requests generating: up to sixteen experts of that layer are read for eight tokens
        _case("decode_few", **{**ring, "T": 8, "residual": True}),
        # a serving batch generating on a layer of large experts: a few rows per expert, all weights read
        _case("decode_batch", **{**large, "T": 96, "cf": 0.0, "residual": True}),
        # the smallest configuration, all float32: a correctness run, or a probe model
        _case("f32_tiny", **_of("tiny")),
        # float32 experts of the GPT-style layer (debugging a training run, reference outputs), weights as a
        # framework that stores [in, out] matrices hands them over
        _case("f32_layer", **{**gpt, "T": 2048, "dtype": "f32", "layout": "input_major", "bias": True}),
        # a batch through the GPT-style layer (prefill or evaluation)
        _case("layer_gpt", **gpt),
        # multi-task routing, one expert per token, the most popular expert takes over half of them
        _case("layer_top1", **{**_of("skew"), "residual": True}),
        # a batch through one layer of the 64-expert stack: about 128 rows per expert, weights streamed
        _case("layer_ring", **{**ring, "residual": True}),
        # many small experts, several per token, a router wider than 64, ragged token count and feature counts
        _case("layer_fine", T=3001, d=1600, f=832, E=128, k=6, renorm=True, act="swiglu", residual=True),
        # the largest single-GPU layer
        _case("layer_large", **large),
        # a training step of the GPT-style layer with biases; the optimizer has changed the weights, so the transposed
        # copies that the backward pass reads are made again
        _case("train_gpt", **{**gpt, "kind": "train", "bias": True, "residual": True, "refresh": True}),
        # a micro-batch of a training step of a SwiGLU layer (gradient accumulation: weights unchanged), bf16 gradients
        _case("train_swiglu", kind="train", T=4099, d=2048, f=5632, E=8, k=2, cf=1.25, renorm=True, act="swiglu",
              residual=True, grads="bf16"),
    ]


# ---- sizes ------------------------------------------------------------------------------------------

def _mats(c):
    return 3 if c["act"] == "swiglu" else 2


def _rows(c):
    """Dispatched rows: every assignment, or what the capacity lets through of evenly spread ones."""
    A = c["k"] * c["T"]
    if c["cf"] <= 0:
        return A
    return min(A, c["E"] * max(1, math.ceil(A * c["cf"] / c["E"])))


def _active(c):
    """Experts that get at least one row, expected under an even router."""
    p_miss = (1.0 - c["k"] / c["E"]) ** c["T"]
    return max(c["k"], min(c["E"], c["E"] * (1.0 - p_miss)))


def work(case):
    c = case
    es = 4 if c["dtype"] == "f32" else 2
    T, d, f, E = c["T"], c["d"], c["f"], c["E"]
    R, m = _rows(c), _mats(c)
    experts = _active(c) * m * d * f * es
    router = d * E * 4
    tokens = T * d * es
    flops = 2.0 * R * m * d * f + 2.0 * T * d * E
    nbytes = experts + router + tokens * (2 + (1 if c["residual"] else 0))
    if c["kind"] == "train":
        g = 2 if c["grads"] == "bf16" else 4
        # backward: every product twice more (inputs and weights); pre-activations are not kept by the forward pass
        flops += 2.0 * flops
        nbytes += experts + E * m * d * f * g + 2 * router + 3 * tokens
        if c["refresh"]:
            nbytes += 2 * E * m * d * f * es
    return {"bytes": float(nbytes), "flops": float(flops)}


LIMIT_FLOPS = 20e12           # (the largest listed case: 23e12 flops)
LIMIT_WEIGHT_BYTES = 5 << 30


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, m):
    return m * max(1, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / m)))


def draw(rng):
    while True:
        kind = rng.choice(["decode", "decode", "f32", "layer", "layer", "layer", "train"])
        act = rng.choice(["gelu", "swiglu"])
        residual = rng.random() < 0.6
        if kind == "decode":
            E = rng.choice([8, 16, 24, 32, 64])
            c = _case(None, T=_log(rng, 1, 256), d=_mult(rng, 1024, 4096, 128), f=_mult(rng, 2048, 14336, 256), E=E,
                      k=rng.choice([1, 2, 2, 4]), renorm=rng.random() < 0.5, act=act, residual=residual)
        elif kind == "f32":
            E = rng.choice([4, 7, 8, 16])
            c = _case(None, T=_log(rng, 64, 4096), d=_mult(rng, 128, 1024, 64), f=_mult(rng, 512, 4096, 64), E=E,
                      k=rng.choice([1, 2]), cf=rng.choice([0.0, 1.25]), act=act, dtype="f32", residual=residual,
                      layout=rng.choice(["output_major", "input_major"]), bias=act == "gelu" and rng.random() < 0.5)
        elif kind == "layer":
            E = rng.choice([4, 8, 12, 16, 32, 64, 96, 128])
            c = _case(None, T=_log(rng, 257, 32768), d=_mult(rng, 512, 4096, rng.choice([64, 256])),
                      f=_mult(rng, 768, 14336, rng.choice([64, 256])), E=E, k=rng.choice([1, 2, 2, min(E, 6)]),
                      cf=rng.choice([0.0, 1.0, 1.25]), renorm=rng.random() < 0.6, act=act, residual=residual,
                      bias=act == "gelu" and rng.random() < 0.4, router_bias=rng.choice(["none", "none", "zipf"]))
        else:
            E = rng.choice([4, 8, 16, 32, 64])
            c = _case(None, kind="train", T=_log(rng, 257, 8192), d=_mult(rng, 512, 2048, 256), f=_mult(rng, 1024, 6144, 256),
                      E=E, k=rng.choice([1, 2, 2]), cf=rng.choice([0.0, 1.25]), renorm=rng.random() < 0.6, act=act,
                      residual=residual, bias=act == "gelu" and rng.random() < 0.5, refresh=act == "gelu" and rng.random() < 0.5,
                      grads=rng.choice(["f32", "bf16"]))
        es = 4 if c["dtype"] == "f32" else 2
        if work(c)["flops"] > (LIMIT_FLOPS if c["dtype"] == "bf16" else 0.15e12):
            continue
        if c["E"] * _mats(c) * c["d"] * c["f"] * es > LIMIT_WEIGHT_BYTES:
            continue
        if c["k"] * c["T"] * c["f"] * es > (2 << 30):
            continue
        return c


# ---- inputs -----------------------------------------------------------------------------------------

def _config(c):
    return M.MoEConfig(T=c["T"], d_model=c["d"], d_ff=c["f"], E=c["E"], k=c["k"], capacity_factor=c["cf"],
                       renormalize=c["renorm"], act=c["act"], dtype=c["dtype"])


def _inputs(c, seed):
    """Tokens, parameters and upstream gradient (device tensors, from the seed alone).  Standard normals scaled by
    fan_in^-1/2 for the matrices, the log of Zipf masses as the skewed router's bias."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    T, d, f, E = c["T"], c["d"], c["f"], c["E"]

    def normal(shape, std, dtype=dt):
        out = torch.empty(shape, dtype=dtype, device="cuda")
        if len(shape) < 3:
            return out.copy_(torch.randn(shape, generator=g, device="cuda") * std)
        for e in range(shape[0]):  # one expert at a time: no float32 copy of the whole stack
            out[e].copy_(torch.randn(shape[1:], generator=g, device="cuda") * std)
        return out

    def matrix(n_in, n_out):
        return normal((E, n_out, n_in) if c["layout"] == "output_major" else (E, n_in, n_out), n_in ** -0.5)

    t = {"x": normal((T, d), 1.0), "w_router": normal((d, E), d ** -0.5, torch.float32)}
    if c["act"] == "gelu":
        t["w1"], t["w2"] = matrix(d, f), matrix(f, d)
        if c["bias"]:
            t["b1"], t["b2"] = normal((E, f), 0.1), normal((E, d), 0.1)
    else:
        t["w_gate_proj"], t["w_up"], t["w_down"] = matrix(d, f), matrix(d, f), matrix(f, d)
    if c["router_bias"] == "zipf":
        t["b_router"] = torch.tensor([math.log(v) for v in zipf_masses(E, 1.2)], dtype=torch.float32, device="cuda")
    if c["kind"] == "train":
        t["d_out"] = normal((T, d), 1.0)
    return t


def prepare(case, seed):
    c = case
    cfg = _config(c)
    t = _inputs(c, seed)
    T, d, f, E = c["T"], c["d"], c["f"], c["E"]
    params = {n: v for n, v in t.items() if n not in ("x", "d_out")}
    n = M.moe_router_pack_bytes(d, E) if c["dtype"] == "bf16" else 0
    if n:  # the gate's pre-split copy of the router, made once where the weights are loaded
        params["w_router_packed"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        M.moe_pack_router(params["w_router"], params["w_router_packed"])
    s = {"case": c, "cfg": cfg, "x": t["x"], "weights": M.Weights(params, c["layout"]), "out": torch.empty_like(t["x"]),
         "ws": torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")}
    if c["kind"] == "train":
        f32 = dict(dtype=torch.float32, device="cuda")
        gw = dict(dtype=torch.bfloat16 if c["grads"] == "bf16" else torch.float32, device="cuda")
        sw = c["act"] == "swiglu"
        s["d_out"] = t["d_out"]
        s["w1_im"] = torch.empty(E, d, (2 if sw else 1) * f, dtype=torch.bfloat16, device="cuda")
        s["w2_im"] = torch.empty(E, f, d, dtype=torch.bfloat16, device="cuda")
        if sw:
            M.moe_transpose_expert_weights(torch.cat([t["w_gate_proj"], t["w_up"]], dim=1), s["w1_im"])
            M.moe_transpose_expert_weights(t["w_down"], s["w2_im"])
        else:
            M.moe_transpose_expert_weights(t["w1"], s["w1_im"])
            M.moe_transpose_expert_weights(t["w2"], s["w2_im"])
        s["bws"] = torch.empty(M.moe_layer_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        s["d_x"] = torch.empty_like(t["x"])
        s["d_w_router"] = torch.empty(d, E, **f32)
        s["d_b_router"] = torch.empty(E, **f32) if "b_router" in t else None
        s["d_w1"] = torch.empty(E, (2 if sw else 1) * f, d, **gw)
        s["d_w2"] = torch.empty(E, d, f, **gw)
        s["d_b1"] = torch.empty(E, f, **f32) if "b1" in t else None
        s["d_b2"] = torch.empty(E, d, **f32) if "b2" in t else None
    return s


# ---- one pass ---------------------------------------------------------------------------------------

def run(s):
    c, cfg, W, x = s["case"], s["cfg"], s["weights"], s["x"]
    residual = x if c["residual"] else None
    if c["kind"] == "train" and c["refresh"]:
        M.moe_transpose_expert_weights(W.tensors["w1"], s["w1_im"])
        M.moe_transpose_expert_weights(W.tensors["w2"], s["w2_im"])
    M.moe_layer_forward(cfg, W, x, residual, s["out"], s["ws"])
    if c["kind"] != "train":
        return {"out": s["out"]}
    M.moe_layer_backward(cfg, W, s["w1_im"], s["w2_im"], x, s["d_out"], s["d_out"] if c["residual"] else None, s["ws"],
                         s["d_x"], s["d_w_router"], s["d_b_router"], s["d_w1"], s["d_b1"], s["d_w2"], s["d_b2"], s["bws"])
    r = {n: s[n] for n in ("out", "d_x", "d_w_router", "d_b_router", "d_w1", "d_b1", "d_w2", "d_b2")}
    return {n: v for n, v in r.items() if v is not None}


# ---- the same in 64 bits ----------------------------------------------------------------------------

def _exact_route(c, x, w_router, b_router):
    """(experts [T, k], probabilities [T, E], kept [T, k] bool) by float64 logits; first choices before second ones
    under the capacity, token order inside a choice."""
    T, E, k = c["T"], c["E"], c["k"]
    z = x @ w_router + (0 if b_router is None else b_router)
    idx = torch.sort(z.detach(), dim=1, descending=True, stable=True).indices[:, :k]
    if c["cf"] <= 0:
        return idx, torch.softmax(z, dim=1), torch.ones_like(idx, dtype=torch.bool)
    cap = max(1, math.ceil(k * T * c["cf"] / E))
    e = idx.t().reshape(-1)  # assignments in priority order
    onehot = torch.zeros(k * T, E, dtype=torch.int32, device=e.device)
    onehot[torch.arange(k * T, device=e.device), e] = 1
    place = torch.cumsum(onehot, 0)[torch.arange(k * T, device=e.device), e]
    return idx, torch.softmax(z, dim=1), (place <= cap).reshape(k, T).t()


def exact(case, seed):
    c = case
    t = _inputs(c, seed)
    train = c["kind"] == "train"
    f64 = {n: v.double().requires_grad_(train) for n, v in t.items() if n in ("x", "w_router", "b_router")}
    x, w_router, b_router = f64["x"], f64["w_router"], f64.get("b_router")
    idx, p, kept = _exact_route(c, x, w_router, b_router)
    w = torch.gather(p, 1, idx)
    if c["renorm"]:
        w = w / w.sum(1, keepdim=True)
    out = x.detach().clone() if c["residual"] else torch.zeros_like(x)
    d_out = t["d_out"].double() if train else None
    d_x = (d_out.clone() if c["residual"] else torch.zeros_like(d_out)) if train else None
    d_w = torch.zeros_like(w) if train else None
    sw = c["act"] == "swiglu"
    names = ["w_gate_proj", "w_up", "w_down"] if sw else ["w1", "w2"] + (["b1", "b2"] if c["bias"] else [])
    grads = {n: [] for n in names}
    for e in range(c["E"]):
        tok, j = torch.nonzero((idx == e) & kept, as_tuple=True)
        P = {}
        for n in names:
            v = t[n][e].double()
            if v.dim() == 2 and c["layout"] == "input_major":
                v = v.t()
            P[n] = v.requires_grad_(train)
        xd = x.detach()[tok].requires_grad_(train)
        if sw:
            g = xd @ P["w_gate_proj"].t()
            y = (torch.sigmoid(g) * g * (xd @ P["w_up"].t())) @ P["w_down"].t()
        else:
            u = xd @ P["w1"].t() + (P["b1"] if c["bias"] else 0)
            h = 0.5 * u * torch.special.erfc(-u * math.sqrt(0.5))
            y = h @ P["w2"].t() + (P["b2"] if c["bias"] else 0)
        wj = w.detach()[tok, j].unsqueeze(1)
        out.index_put_((tok,), wj * y.detach(), accumulate=True)
        if train:
            dy = d_out[tok]
            gs = torch.autograd.grad(y, [xd] + [P[n] for n in names], wj * dy)
            d_x.index_put_((tok,), gs[0], accumulate=True)
            d_w[tok, j] = (dy * y.detach()).sum(1)
            for n, v in zip(names, gs[1:]):
                grads[n].append(v)
    r = {"out": out.detach()}
    if train:
        leaves = [x, w_router] + ([b_router] if b_router is not None else [])
        gate = torch.autograd.grad(w, leaves, d_w)
        r["d_x"] = d_x + gate[0]
        r["d_w_router"] = gate[1]
        if b_router is not None:
            r["d_b_router"] = gate[2]
        st = {n: torch.stack(v) for n, v in grads.items()}
        r["d_w1"] = torch.cat([st["w_gate_proj"], st["w_up"]], dim=1) if sw else st["w1"]
        if c["bias"]:
            r["d_b1"] = st["b1"]
        r["d_w2"] = st["w_down"] if sw else st["w2"]
        if c["bias"]:
            r["d_b2"] = st["b2"]
    return r


def tolerance(case):
    """float32: sums of up to a few thousand terms in another order.  bf16: the hidden activations, the experts'
    outputs and the result are rounded to bf16 once each; the backward pass rounds four more intermediates."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] == "train":
        return {"rel": 1.5e-2}
    return {"rel": 1e-2}
