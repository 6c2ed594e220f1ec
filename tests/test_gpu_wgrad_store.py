"""Weight gradients on the three tiles the rules choose between (128 x 256, 256 x 256 for long sums, 128 x 128 for few tiles),
numbers of tiles that leave the last unit of an XCD short, and sums that end in the first, the second and the third of the
stages: the loads past the end clear a stage that other wavefronts have just read."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,rows,N1,N2,n1_edge,n2_edge", [
    (33, [96, 64, 33, 32, 1, 0, 191], 512, 768, 128, 256),        # 2 x 3 big tiles per expert: 198 of a round of 256
    (13, [1408, 1400, 1431], 1024, 1024, 256, 256),               # long sums, one round
    (3, [700, 0, 65], 512, 512, 128, 128)])
def test_wgrad_tile_shapes(E, rows, N1, N2, n1_edge, n2_edge):
    print(E, rows, N1, N2, flush=True)
    n = [rows[i % len(rows)] for i in range(E)]
    for dt in (M.binding.MOE_F32, M.binding.MOE_BF16):
        tile, edge = M.lib().moe_test_wgrad_tiles, M.lib().moe_test_wgrad_n1_edge
        for f in (tile, edge):
            f.restype, f.argtypes = C.c_int32, [C.c_int32] * 4 + [C.c_int64]
        assert tile(E, N1, N2, dt, max(n)) // 100 == n2_edge and edge(E, N1, N2, dt, max(n)) == n1_edge
    off = np.concatenate([[0], np.cumsum(n)])
    g = torch.Generator(device="cuda").manual_seed(E + N1)
    a = torch.randn(int(off[-1]), N1, generator=g, device="cuda").bfloat16()
    b = torch.randn(int(off[-1]), N2, generator=g, device="cuda").bfloat16()
    offsets = torch.tensor(off, dtype=torch.int32, device="cuda")
    first = None
    for rep in range(4):  # (each over outputs that hold something else)
        c = torch.full((E, N1, N2), float("nan"), device="cuda")
        h = torch.full((E, N1, N2), float("nan"), dtype=torch.bfloat16, device="cuda")
        sums = torch.full((E, N1), float("nan"), device="cuda")
        M.moe_expert_wgrad(a, b, offsets, c, max(n), a_column_sums=sums if rep % 2 else None)
        M.moe_expert_wgrad(a, b, offsets, h, max(n))
        torch.cuda.synchronize()
        first = c if first is None else first
        assert torch.equal(c, first) and torch.equal(h, c.bfloat16())
        if rep % 2:
            for e in range(E):
                want = a[off[e]:off[e + 1]].double().sum(0)
                assert float((sums[e].double() - want).abs().max()) <= 8 * max(n[e], 1) ** 1.5 * 2.0 ** -23
    for e in range(E):
        want = a[off[e]:off[e + 1]].double().t() @ b[off[e]:off[e + 1]].double()
        # a float32 sum of n terms of size one is within n * 2^-24 * sqrt(n) of the exact one, element by element
        assert float((first[e].double() - want).abs().max()) <= 8 * max(n[e], 1) ** 1.5 * 2.0 ** -23
