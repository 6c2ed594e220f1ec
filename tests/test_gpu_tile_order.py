"""SwiGLU over a few rows per expert where the eighths of the XCDs are a multiple of 16 MB of weights apart, so that each starts at another
place: every tile once, with a last eighth that is short, second row tiles, eighths shorter and longer than the shift."""
import pytest
import torch

import paper_2205_10034_amd as M
from gpu_util import product_kernel

pytestmark = pytest.mark.gpu


# eighths of 64 tiles of 32 features x 32 rows (the last of 60, of 62 with a second row tile, full ones), of 128
@pytest.mark.parametrize("T,E,k,d,f,first", [(40, 2, 1, 4096, 8128, 20), (48, 2, 1, 4096, 5440, 36), (48, 8, 2, 4096, 2048, 12), (24, 4, 2, 4096, 8192, 12)])
def test_every_tile_once(T, E, k, d, f, first):
    print(T, E, k, d, f, first, flush=True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, act="swiglu")
    assert product_kernel(cfg, 0) == "stream 64x32"
    g = torch.Generator(device="cuda").manual_seed(T + E + f)
    mat = lambda n, m: (torch.randn(E, n, m, generator=g, device="cuda") * m ** -0.5).bfloat16()
    t = {"w_router": torch.randn(d, E, generator=g, device="cuda") * d ** -0.5, "w_gate_proj": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)}
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    t["w_router"][0] = torch.tensor([10.0] + [0.0] * (E - 1))     # expert 0 gets the first tokens and no others
    x[:first, 0], x[first:, 0] = 4.0, -4.0
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xFF)   # (h: NaN where no tile writes)
    out = torch.empty_like(x)
    M.moe_layer_forward(cfg, M.Weights(t, "output_major"), x, None, out, ws)
    torch.cuda.synchronize()
    lay = M.moe_workspace_layout(cfg)
    off = ws[lay["expert_offsets"]:lay["expert_offsets"] + 4 * (E + 1)].view(torch.int32).tolist()
    r2a = ws[lay["row_to_assign"]:lay["row_to_assign"] + 4 * k * T].view(torch.int32)
    h = ws[lay["h"]:lay["h"] + 2 * k * T * f].view(torch.bfloat16).view(k * T, f)
    assert off[1] == first and off[E] == k * T
    assert sum(-(-(b - a) // 32) for a, b in zip(off, off[1:])) * (f // 32) in range(8 * 64 - 7, 8 * 64 + 1) or E == 4
    for e in range(E):
        xd = x[(r2a[off[e]:off[e + 1]] % T).long()].double()
        u = xd @ t["w_gate_proj"][e].double().t()
        ref = u * torch.sigmoid(u) * (xd @ t["w_up"][e].double().t())
        # one rounding to bf16 (2^-9 relative); sums of up to 4096 terms, 41 in all, in float32: 41 x 2^-24 x 20 at most in earnest
        assert ((h[off[e]:off[e + 1]].double() - ref).abs() <= 2 ** -8 * ref.abs() + 1e-4).all(), e
