"""float32 layers whose first product gathers the tokens and whose second, with one expert per token, combines: every kernel shape,
both layouts and activations, capacities that drop, tokens without a row, in place."""
import ctypes as C

import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


def tile_rows(cfg, which):
    f = M.lib().moe_test_f32_tile_rows
    f.restype, f.argtypes = C.c_int32, [C.c_void_p, C.c_int32]
    c = cfg.c()
    return f(C.byref(c), which)


@pytest.mark.parametrize("T,d,f,E,k,cf,act,layout,rows", [
    (1, 64, 64, 4, 1, 0.0, "gelu", "output_major", (32, 32)), (256, 128, 512, 4, 1, 1.25, "gelu", "output_major", (32, 32)),
    (37, 192, 320, 3, 2, 0.0, "swiglu", "input_major", (32, 32)), (33, 1024, 64, 5, 1, 0.5, "gelu", "input_major", (32, 32)),
    (3001, 256, 1088, 7, 1, 1.0, "gelu", "output_major", None), (1000, 960, 1408, 16, 2, 1.25, "gelu", "input_major", None),
    (900, 576, 1024, 8, 1, 0.0, "swiglu", "output_major", None), (1111, 320, 4096, 8, 1, 0.5, "swiglu", "input_major", None),
    (2048, 1024, 4096, 16, 2, 1.25, "gelu", "input_major", (160, 160)), (4096, 1024, 4096, 16, 1, 1.0, "gelu", "output_major", (160, 160)),
    (2500, 768, 3072, 8, 1, 0.0, "gelu", "output_major", None),
    (4096, 1024, 128, 4, 1, 0.0, "gelu", "output_major", None), (2048, 1024, 704, 8, 2, 0.0, "swiglu", "input_major", None)])   # (rows copied apart)
@pytest.mark.parametrize("mode", ["plain", "in_place", "nan"])
def test_f32_layer(T, d, f, E, k, cf, act, layout, rows, mode):
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, capacity_factor=cf, act=act, dtype="f32")
    im = 2 if layout == "input_major" else 0
    got = (tile_rows(cfg, im), tile_rows(cfg, 1 + im))
    print(T, d, f, E, k, cf, act, layout, mode, got, flush=True)
    assert rows is None or got == rows
    g = torch.Generator(device="cuda").manual_seed(T + d)
    mat = lambda n, m: torch.randn((E, n, m) if not im else (E, m, n), generator=g, device="cuda") * m ** -0.5
    t = {"w_router": torch.randn(d, E, generator=g, device="cuda") * d ** -0.5}
    if act == "gelu":
        t.update(w1=mat(f, d), w2=mat(d, f), b1=torch.randn(E, f, generator=g, device="cuda"), b2=torch.randn(E, d, generator=g, device="cuda"))
    else:
        t.update(w_gate_proj=mat(f, d), w_up=mat(f, d), w_down=mat(d, f))
    x = torch.randn(T, d, generator=g, device="cuda")
    if mode == "nan":
        x[T // 2, 3] = float("nan")
    W = M.Weights(t, layout)
    lay = M.moe_workspace_layout(cfg)
    ws, ws2 = (torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xFF) for _ in range(2))
    out, out2 = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    # the stages one by one on tables of their own: rows copied by moe_dispatch, combine in its kernel
    M.moe_layer_route(cfg, W, x, ws2)
    seg = lambda w, n, c, dt=torch.float32: w[lay[n]:lay[n] + 4 * c].view(dt)
    a2r, tw = seg(ws2, "assign_to_row", k * T, torch.int32), seg(ws2, "topk_w", k * T).view(T, k)
    offsets = seg(ws2, "expert_offsets", E + 1, torch.int32)
    R = int(offsets[-1])
    yd = torch.zeros(lay["r_max"], d, device="cuda")
    M.moe_expert_ffn(cfg, W, seg(ws2, "xd", lay["r_max"] * d).view(-1, d), offsets, yd, torch.empty(M.moe_workspace_bytes(cfg, 2), dtype=torch.uint8, device="cuda"))
    res = None if mode == "plain" else x
    M.moe_combine(cfg, yd, a2r, tw, res, out2)
    target = x.clone() if mode == "in_place" else x
    o = target if mode == "in_place" else out
    M.moe_layer_forward(cfg, W, target, target if res is not None else None, o, ws)
    torch.cuda.synchronize()
    for n in ("assign_to_row", "topk_w"):
        assert torch.equal(seg(ws, n, k * T, torch.int32), seg(ws2, n, k * T, torch.int32)), n
    # the same kernels on the same values: every bit the same (as integers, where a value may be NaN)
    bits = lambda v: v.contiguous().view(torch.int32)
    assert torch.equal(bits(seg(ws, "xd", R * d)), bits(seg(ws2, "xd", R * d)))
    assert torch.equal(bits(seg(ws, "yd", R * d)), bits(yd[:R].reshape(-1)))
    assert torch.equal(o.isnan(), out2.isnan()) and torch.equal(o.nan_to_num(0.0), out2.nan_to_num(0.0))
