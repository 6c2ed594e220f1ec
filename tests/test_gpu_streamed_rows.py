"""The weight-streaming shape of 256 weight rows and 192 rows, whose rows have two LDS stages beside three of weights: every
remainder of its K loop of six steps, ragged feature counts, experts with no rows, a few, exactly a tile, two tiles; with
and without gathered rows and the fused combine of one choice per token."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

from gpu_util import product_kernel

pytestmark = pytest.mark.gpu

ROWS = [192, 1, 0, 191, 193, 97, 160, 15, 130, 128, 16, 159, 129, 200, 100, 209]   # 120 on average


@pytest.mark.parametrize("act,d,f", [("gelu", 1152, 4352), ("gelu", 1216, 4544), ("gelu", 1280, 4416), ("gelu", 1344, 4352), ("gelu", 1408, 4352),
                                     ("gelu", 1472, 4352), ("swiglu", 1152, 2240), ("swiglu", 1344, 2368)])
@pytest.mark.parametrize("k", [1, 2])
def test_streamed_rows(act, d, f, k):
    E = 16
    T = sum(ROWS) // k if k == 1 else 965
    print(act, d, f, k, flush=True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, act=act, dtype="bf16")
    assert product_kernel(cfg, 0) == "stream 256x192" and product_kernel(cfg, 1) in ("stream 256x192", "stream 128x192")
    g = torch.Generator(device="cuda").manual_seed(d + f + k)
    mat = lambda o, i: (torch.randn(E, o, i, generator=g, device="cuda") * i ** -0.5).bfloat16()
    t = {"w1": mat(f, d), "w2": mat(d, f), "b1": torch.randn(E, f, generator=g, device="cuda").bfloat16(), "b2": torch.randn(E, d, generator=g, device="cuda").bfloat16()} \
        if act == "gelu" else {"w_gate_proj": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)}
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    # a router that sends ROWS[e] tokens to expert e first (and, with two choices, the next expert second): the expert's number
    # is written into the first E features
    first = torch.tensor(np.repeat(np.arange(E), ROWS)[:T], device="cuda")
    x[:, :E] = 0
    x[torch.arange(T), first] = 4.0
    x[torch.arange(T), (first + 1) % E] = 2.0
    router = torch.zeros(d, E, device="cuda")
    router[:E] = torch.eye(E, device="cuda")
    W = M.Weights({**t, "w_router": router}, "output_major")
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    runs = []
    for _ in range(3):
        ws.fill_(0xAB)
        out = torch.full_like(x, float("nan"))
        M.moe_layer_forward(cfg, W, x, x, out, ws)
        torch.cuda.synchronize()
        runs.append(out)
    assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2])
    p = torch.softmax(x[:, :E].double(), 1)
    want = x.double()
    for j in range(k):
        e_of = (first + j) % E
        for e in range(E):
            tok = torch.nonzero(e_of == e).flatten()
            m = {n: v[e].double() for n, v in t.items()}
            xe = x[tok].double()
            if act == "gelu":
                y = torch.nn.functional.gelu(xe @ m["w1"].t() + m["b1"]) @ m["w2"].t() + m["b2"]
            else:
                y = (torch.nn.functional.silu(xe @ m["w_gate_proj"].t()) * (xe @ m["w_up"].t())) @ m["w_down"].t()
            want.index_put_((tok,), p[tok, e].unsqueeze(1) * y, accumulate=True)
    # the hidden activations, the experts' outputs and the result are rounded to bf16 (2^-9) once each
    assert float((runs[0].double() - want).norm() / want.norm()) < 3 * 2.0 ** -9
    assert float((runs[0].double() - want).abs().max() / want.abs().max()) < 3 * 2.0 ** -8
