"""Layers whose expert weights exceed the last-level cache, which the few-row kernels then load non-temporally: one token
(matrix-vector kernels), a few, and enough on one expert that its row tiles share the weights (ordinary loads beside the
others' non-temporal ones); the same sizes with few enough active experts to fit."""
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


def reference(cfg, t, x, idx, w):
    """float64 experts on the routing the library chose."""
    out = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
    for e in idx.unique().tolist():
        tok, j = torch.nonzero(idx == e, as_tuple=True)
        xe, m = x[tok].double(), {n: v[e].double() for n, v in t.items() if v.dim() == 3}
        if cfg.act == "gelu":
            y = torch.nn.functional.gelu(xe @ m["w1"].t()) @ m["w2"].t()
        else:
            y = (torch.nn.functional.silu(xe @ m["w_gate_proj"].t()) * (xe @ m["w_up"].t())) @ m["w_down"].t()
        out.index_put_((tok,), w[tok, j].double().unsqueeze(1) * y, accumulate=True)
    return out


@pytest.mark.parametrize("act,T,k,d,f,E,hot", [
    ("gelu", 1, 2, 4096, 10240, 8, 0.0),        # 336 MB active: two experts
    ("gelu", 2, 4, 4096, 5120, 8, 0.0),
    ("swiglu", 9, 1, 4096, 4096, 8, 0.0),
    ("gelu", 24, 2, 2048, 5120, 8, 0.0),
    ("gelu", 90, 2, 2048, 5120, 8, 9.0),        # every first choice on one expert: three row tiles of it
    ("swiglu", 90, 1, 2048, 3584, 8, 9.0),
    ("gelu", 1, 1, 4096, 5120, 8, 0.0)])        # one active expert: fits
def test_streamed_weights(act, T, k, d, f, E, hot):
    print(act, T, k, d, f, E, hot, flush=True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, act=act, dtype="bf16")
    g = torch.Generator(device="cuda").manual_seed(T + f)
    mat = lambda o, i: (torch.randn(E, o, i, generator=g, device="cuda") * i ** -0.5).bfloat16()
    t = {"w1": mat(f, d), "w2": mat(d, f)} if act == "gelu" else {"w_gate_proj": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)}
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    router = torch.randn(d, E, generator=g, device="cuda") * d ** -0.5
    bias = torch.zeros(E, device="cuda")
    bias[0] = hot
    W = M.Weights({**t, "w_router": router, "b_router": bias}, "output_major")
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    first = None
    for _ in range(3):
        out = torch.full_like(x, float("nan"))
        M.moe_layer_forward(cfg, W, x, None, out, ws)
        torch.cuda.synchronize()
        first = out if first is None else first
        assert torch.equal(out, first)
    p, idx = torch.topk(torch.softmax(x.double() @ router.double() + bias.double(), 1), k, dim=1)
    want = reference(cfg, t, x, idx, p)
    # the hidden activations, the experts' outputs and the result are rounded to bf16 (2^-9) once each
    assert float((first.double() - want).norm() / want.norm()) < 3 * 2.0 ** -9
