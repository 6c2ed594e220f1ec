"""float32 expert products on the tiles of whole 16-row units: every number of units a tile can hold, with a full and a ragged
last unit, experts of one tile, several and none, feature counts that end inside a tile, both weight layouts, pointers on odd
floats; and the lines of the rule beside them."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

from gpu_util import alloc_ws

pytestmark = pytest.mark.gpu


def tile_rows(cfg, second, layout="output_major"):
    f = M.lib().moe_test_f32_tile_rows
    f.restype = C.c_int32
    return f(C.byref(cfg.c()), second + 2 * (layout == "input_major"))


UNITS = [0, 1, 15, 16, 17, 32, 33, 48, 50, 64, 79, 80, 81, 160, 161, 128]      # 80-row tiles of one to five units
LARGE = [161, 160, 159, 144, 130, 128, 112, 99, 96, 80, 65, 64, 33, 0, 170, 177]  # 160-row tiles of one to ten


# T is what an evenly loaded expert would hold, which picks the kernel; the rows themselves are RAGGED
@pytest.mark.parametrize("act,T,rows,d,f,shift,first,second", [
    ("gelu", 66 * 16, UNITS, 896, 1792, 0, 80, 80), ("swiglu", 66 * 16, UNITS, 896, 1792, 1, 80, 80),
    ("gelu", 256 * 16, LARGE, 1024, 4032, 0, 160, 160), ("swiglu", 256 * 16, LARGE, 1024, 1984, 1, 160, 160)])
@pytest.mark.parametrize("layout", ["output_major", "input_major"])
def test_f32_units(act, T, rows, d, f, shift, first, second, layout):
    print(act, T, d, f, shift, layout, flush=True)
    E, R = len(rows), sum(rows)
    assert R <= T
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(d + f)

    def rand(*shape, std=1.0):  # `shift` floats off the allocation's alignment
        n = int(np.prod(shape))
        buf = torch.empty(n + shift, device="cuda")
        t = buf[shift:].view(shape)
        return t.copy_(torch.randn(shape, generator=g, device="cuda") * std)

    def mat(n_in, n_out):
        return rand(E, n_out, n_in, std=n_in ** -0.5) if layout == "output_major" else rand(E, n_in, n_out, std=n_in ** -0.5)

    t = {"w1": mat(d, f), "w2": mat(f, d), "b1": rand(E, f), "b2": rand(E, d)} if act == "gelu" else \
        {"w_gate_proj": mat(d, f), "w_up": mat(d, f), "w_down": mat(f, d)}
    xd = rand(R, d)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=1, act=act, dtype="f32")
    assert tile_rows(cfg, 0, layout) == first and tile_rows(cfg, 1, layout) == second
    guard = torch.full((R + 1, d), 7.0, device="cuda")
    W = M.Weights({**t, "w_router": torch.zeros(d, E, device="cuda")}, layout)
    M.moe_expert_ffn(cfg, W, xd, torch.from_numpy(off).cuda(), guard[:R], alloc_ws(cfg, 2))
    torch.cuda.synchronize()
    assert bool((guard[R] == 7.0).all())                       # nothing past the last row
    want = torch.empty(R, d, dtype=torch.float64, device="cuda")
    for e in range(E):
        m = {n: v[e].double() for n, v in t.items()}
        if layout == "input_major":
            m = {n: v.t() if v.dim() == 2 else v for n, v in m.items()}
        x = xd[off[e]:off[e + 1]].double()
        if act == "gelu":
            y = torch.nn.functional.gelu(x @ m["w1"].t() + m["b1"]) @ m["w2"].t() + m["b2"]
        else:
            y = (torch.nn.functional.silu(x @ m["w_gate_proj"].t()) * (x @ m["w_up"].t())) @ m["w_down"].t()
        want[off[e]:off[e + 1]] = y
    err = float((guard[:R].double() - want).norm() / want.norm())
    print("rel fro", err, flush=True)
    # float32 sums of n terms of size n^-1/2: rounding errors of n^1/2 * 2^-24 of the result, n up to 4032
    assert err < 64 * 2.0 ** -24


@pytest.mark.parametrize("rows,E,N,K,want", [
    (262, 16, 448, 512, 80), (787, 8, 192, 2944, 80), (435, 8, 512, 1856, 64), (512, 8, 704, 2944, 64),
    (256, 16, 1024, 4096, 160), (599, 8, 960, 3264, 80), (16, 16, 1024, 4096, 32)])
def test_f32_rule(rows, E, N, K, want):
    assert tile_rows(M.MoEConfig(T=rows * E, d_model=N, d_ff=K, E=E, k=1, dtype="f32"), 1) == want
