"""Combine of a few tokens, a token's row dealt out over several wavefronts: row lengths around whole trips of 64 vectors, token
counts on both sides of the last split, dropped choices, with and without a residual, both data types."""
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,d,k", [(1, 64, 1), (1, 8192, 8), (3, 576, 2), (5, 1088, 2), (97, 4096, 2), (255, 1600, 3), (2045, 1024, 2), (2052, 1024, 1)])
def test_combine_split(T, d, k, dtype):
    print(T, d, k, dtype, flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=64, E=8, k=k, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(T + d + k)
    yd = torch.randn(k * T, d, generator=g, device="cuda").to(dt)
    w = torch.rand(T, k, generator=g, device="cuda")
    a2r = torch.randperm(k * T, generator=g, device="cuda").to(torch.int32)
    a2r[torch.rand(k * T, generator=g, device="cuda") < 0.2] = -1
    res = torch.randn(T, d, generator=g, device="cuda").to(dt)
    for r in (None, res):
        out = torch.full((T, d), float("nan"), device="cuda").to(dt)
        M.moe_combine(cfg, yd, a2r, w, r, out)
        ref = torch.zeros(T, d, dtype=torch.float64, device="cuda") if r is None else r.double()
        for j in range(k):
            rows = a2r[j * T:(j + 1) * T].long()
            ref += torch.where(rows[:, None] >= 0, w[:, j, None].double() * yd[rows.clamp(min=0)].double(), 0.0)
        # k fused multiply-adds in float32, one rounding to the type
        scale = 1 + ref.abs()
        assert ((out.double() - ref).abs() / scale).max() < (2.0 ** -8 if dtype == "bf16" else (k + 1) * 2.0 ** -23)
