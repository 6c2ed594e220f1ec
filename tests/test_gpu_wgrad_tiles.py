"""Weight gradients on either side of the tile rule: enough 256x256 tiles for a round of the chip (with few and with many
rows per expert, which changes the order of the tiles), and the 128x128 tiles that serve fewer.  float32 sums of exact
products against float64; the bf16 form is the float32 one rounded once."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu

RAGGED = [0, 1, 31, 32, 33, 64, 95, 96, 97, 7]


# tile edge and columns of tiles per block, for float32 and bf16 gradients
@pytest.mark.parametrize("E,scale,N1,N2,tile,wide,wide_bf16", [
    (64, 1, 512, 512, 256, 2, 2),                                           # 256 tiles of 256
    (70, 1, 256, 1280, 256, 5, 5), (19, 4, 512, 1280, 256, 5, 5),           # few, but as 128 in blocks of eight and two columns
    (100, 1, 256, 1280, 256, 5, 5), (24, 1, 768, 2560, 256, 10, 10),        # rows of five and ten tiles: whole rows, partial blocks of them
    (16, 1, 256, 8192, 256, 8, 8), (18, 1, 256, 6144, 256, 8, 8), (256, 1, 256, 8192, 256, 8, 32),  # 32 columns: whole rows of large 16-bit gradients
    (80, 3, 512, 768, 256, 3, 3), (24, 3, 768, 2560, 256, 8, 8), (16, 3, 256, 8192, 256, 8, 8),  # more rows per expert
    (60, 3, 512, 768, 128, 6, 6), (3, 4, 768, 1280, 128, 8, 8), (40, 1, 256, 512, 128, 4, 4)])
def test_wgrad_tiles(E, scale, N1, N2, tile, wide, wide_bf16):
    print(E, scale, N1, N2, flush=True)
    f = M.lib().moe_test_wgrad_tiles
    f.restype, f.argtypes = C.c_int32, [C.c_int32] * 4 + [C.c_int64]
    assert f(96, 512, 5120, M.binding.MOE_F32, 16) == 25620 and f(24, 768, 4096, M.binding.MOE_F32, 16) == 25608
    assert f(E, N1, N2, M.binding.MOE_F32, max(RAGGED) * scale) == tile * 100 + wide
    assert f(E, N1, N2, M.binding.MOE_BF16, max(RAGGED) * scale) == tile * 100 + wide_bf16
    rows = [RAGGED[i % len(RAGGED)] * scale for i in range(E)]
    offsets = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32)
    g = torch.Generator(device="cuda").manual_seed(E + N2)
    a = torch.randn(sum(rows), N1, generator=g, device="cuda").bfloat16()
    b = torch.randn(sum(rows), N2, generator=g, device="cuda").bfloat16()
    c = torch.full((E, N1, N2), float("nan"), device="cuda")
    h = torch.full((E, N1, N2), float("nan"), dtype=torch.bfloat16, device="cuda")
    sums = torch.full((E, N1), float("nan"), device="cuda")
    M.moe_expert_wgrad(a, b, offsets.cuda(), c, max(rows))
    M.moe_expert_wgrad(a, b, offsets.cuda(), h, max(rows), a_column_sums=sums)
    torch.cuda.synchronize()
    assert torch.equal(h, c.bfloat16())
    for e in range(E):
        ae, be = (t[offsets[e]:offsets[e + 1]].double() for t in (a, b))
        want = ae.t() @ be
        # a float32 sum of n terms of size one is within n * 2^-24 * sqrt(n) of the exact one, element by element
        tol = max(rows[e], 1) ** 1.5 * 2.0 ** -23
        assert float((c[e].double() - want).abs().max()) <= 8 * tol and float((sums[e].double() - ae.sum(0)).abs().max()) <= 8 * tol
