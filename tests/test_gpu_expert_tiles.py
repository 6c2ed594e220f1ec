"""Expert products (bf16) where their tiles end beside the data: the weight-streaming kernels in every shape (the rule is on
rows per expert and tile counts), and the grouped GEMM with feature counts that are no multiple of its tile.  The bar is
the bf16 one of the other tests: relative Frobenius error below 1e-2 (measured 2-3e-3: h, yd and out rounded once each)."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M
from oracle import moe_oracle as O
from workloads import WORKLOADS, bf16_round, make_layer

from gpu_util import alloc_ws, product_kernel, rel_fro, run_layer, to_dev, to_np, upload_weights

pytestmark = pytest.mark.gpu

TOL = 1e-2
RAGGED = [0, 1, 15, 16, 17, 31, 32, 33, 0, 47, 48, 49, 63, 64, 65, 2]


def ffn_case(act, rows, T, d, f, seed, bias=True):
    rng = np.random.default_rng(seed)
    E, R = len(rows), sum(rows)
    assert R <= T
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    xd = bf16_round(rng.standard_normal((R, d)).astype(np.float32))
    names = [("w1", d, f), ("w2", f, d)] if act == "gelu" else [("w_gate_proj", d, f), ("w_up", d, f), ("w_down", f, d)]
    L = {n: bf16_round((rng.standard_normal((E, a, b)) * a ** -0.5).astype(np.float32)) for n, a, b in names}
    if act == "gelu" and bias:
        L["b1"], L["b2"] = (bf16_round(rng.standard_normal((E, n)).astype(np.float32)) for n in (f, d))
    ref = O.expert_ffn(xd, offsets, L, act)
    L["w_router"] = np.zeros((d, E), np.float32)
    W = upload_weights(L, "bf16")
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=1, act=act)
    yd = torch.full((T + 1, d), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = alloc_ws(cfg, 2)
    ws.fill_(0xAB)  # (nothing in the workspace is expected to be clear)
    M.moe_expert_ffn(cfg, W, to_dev(xd, "bf16"), torch.from_numpy(offsets).cuda(), yd, ws)
    torch.cuda.synchronize()
    assert bool((yd[R:] == 7.0).all())                                   # nothing past the last row
    err = rel_fro(to_np(yd[:R]), ref)
    print("rel fro", err, flush=True)
    assert err < TOL


# T only says what an evenly loaded expert would hold, which is what picks the shape (named for the first and second product of
# GELU and of SwiGLU experts; a "grouped" one is in another case's name); the rows themselves are ragged
SHAPES = [
    (24, 40, 64, 64, "64x32 64x32", "64x32 64x32"), (20, 40, 128, 320, "64x32 64x32", "64x32 64x32"),      # one to thirteen stages,
    (9, 60, 832, 192, "64x32 64x32", "64x32 64x32"),                                                       # ragged last tiles
    (36, 24, 192, 320, "128x64 128x64", "128x64 128x64"), (30, 24, 512, 448, "128x64 128x64", "128x64 128x64"),
    (40, 16, 320, 192, "64x64 64x64", "64x64 64x64"), (150, 4, 320, 1088, "64x64 64x64", "64x64 64x64"),   # few tiles
    (500, 3, 64, 128, "64x64 64x64", "64x64 64x64"), (31, 40, 64, 64, "64x64 64x64", "128x64 64x64"),
    (60, 24, 576, 576, "64x64 64x64", "128x128 64x64"), (60, 32, 576, 576, "128x128 128x128", "grouped 128x128"),
    (90, 40, 512, 832, "grouped 128x128", "grouped 128x128"), (60, 32, 2048, 576, "128x128 256x128", "128x128 256x128"),
    (330, 16, 128, 1216, "128x128 64x64", "grouped 64x64"),
    (120, 32, 512, 576, "128x192 128x192", "grouped 128x192"), (250, 16, 704, 1216, "grouped 128x192", "grouped 128x192"),
    (120, 16, 320, 832, "64x64 64x64", "128x192 64x64"),
    (40, 128, 512, 448, "256x64 256x64", "grouped 256x64"), (80, 128, 512, 448, "256x128 256x128", "grouped 256x128"),
    (40, 128, 832, 448, "256x64 grouped", "256x64 grouped"), (80, 128, 832, 448, "256x128 grouped", "256x128 grouped"),
    (40, 64, 1024, 1024, "256x64 256x64", "256x64 256x64")]


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("mean,E,d,f,gelu,swiglu", SHAPES)
def test_stream_shapes(act, mean, E, d, f, gelu, swiglu):
    print(act, mean, E, d, f, flush=True)
    some = RAGGED if mean > 24 else [r if r < 34 else r - 40 for r in RAGGED]   # (on average 13 rows instead of 31)
    rows = [some[(3 * i + E) % len(some)] for i in range(E)]
    rows[E // 2] += max(0, mean * E - sum(rows)) // 2                    # one expert far above the mean
    T = max(mean * E, sum(rows))
    assert max(rows) > -(-T // E)
    got = [product_kernel(M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=1, act=act), second) for second in (0, 1)]
    want = (gelu if act == "gelu" else swiglu).split()
    assert all(g == "stream " + w or g.startswith(w) for g, w in zip(got, want)), got
    ffn_case(act, rows, T, d, f, mean + E)


@pytest.mark.parametrize("name,kw", [
    ("gpt", dict(T=60, E=16, k=2, capacity_factor=0.0)), ("large", dict(T=130, E=8, k=2, d_model=320, d_ff=448)),
    ("skew", dict(T=150, E=8, d_model=192, d_ff=320)), ("skew", dict(T=700, E=8, d_model=320, d_ff=832, capacity_factor=0.8)),
    ("large", dict(T=300, E=4, k=1, d_model=192, d_ff=320, capacity_factor=0.0)), ("gpt", dict(T=24, E=2, k=1, d_model=64, d_ff=64))],
    ids=str)
def test_stream_layer(name, kw):
    """Rows gathered from x, the top-1 combine in the second product (with drops), a residual that is also the output."""
    wl = WORKLOADS[name].scaled(**kw)
    print(wl, flush=True)
    L = make_layer(wl, with_bias=True)
    ref = O.layer_forward(L["x"], L, E=wl.E, k=wl.k, capacity_factor=wl.capacity_factor, renormalize=wl.renormalize, act=wl.act)
    cfg, W, x = M.MoEConfig.from_workload(wl), upload_weights(L, "bf16"), to_dev(L["x"], "bf16")
    assert rel_fro(run_layer(cfg, W, x)["out"], ref["out"]) < TOL
    res = to_dev(L["x"][::-1].copy(), "bf16")
    M.moe_layer_forward(cfg, W, x, res, res, alloc_ws(cfg))
    torch.cuda.synchronize()
    assert rel_fro(to_np(res) - L["x"][::-1], ref["out"]) < 2 * TOL      # (the sum's rounding is counted against the term)


@pytest.mark.parametrize("mfma", [16, 32])
@pytest.mark.parametrize("act,d,f", [("gelu", 320, 1088), ("swiglu", 320, 192), ("swiglu", 448, 832), ("gelu", 576, 256)])
def test_grouped_gemm_ragged_features(act, d, f, mfma):
    print(act, d, f, mfma, flush=True)
    M.moe_set_tuning(M.MOE_TUNE_GEMM_MFMA, mfma)
    try:
        rows = [700, 0, 257, 256, 1, 130, 63, 320]
        for bias in (True, False):
            ffn_case(act, rows, sum(rows), d, f, d + mfma, bias)
        wl = WORKLOADS["skew"].scaled(T=900, E=4, d_model=d, d_ff=f, act=act, capacity_factor=0.7)   # top-1: combine in the epilogue
        L = make_layer(wl, with_bias=True)
        ref = O.layer_forward(L["x"], L, E=wl.E, k=1, capacity_factor=0.7, renormalize=False, act=act)
        cfg, W, x = M.MoEConfig.from_workload(wl), upload_weights(L, "bf16"), to_dev(L["x"], "bf16")
        out = x.clone()
        M.moe_layer_forward(cfg, W, x, out, out, alloc_ws(cfg))
        torch.cuda.synchronize()
        assert rel_fro(to_np(out) - L["x"], ref["out"]) < 2 * TOL
    finally:
        M.moe_set_tuning(M.MOE_TUNE_GEMM_MFMA, 0)


def test_workspace_counters_between_kernels():
    """First product streaming, second product on the grouped GEMM and the reverse, run twice from one routing: each leaves
    the other's tile counters as it needs them."""
    for d, f in ((2048, 256), (256, 2048)):
        wl = WORKLOADS["gpt"].scaled(T=1300, E=16, k=2, d_model=d, d_ff=f, capacity_factor=0.0)
        names = [product_kernel(M.MoEConfig.from_workload(wl), second) for second in (0, 1)]
        assert names == (["stream 64x64", "grouped 256"] if f < d else ["grouped 256", "stream 64x64"])
        L = make_layer(wl)
        cfg, W, x = M.MoEConfig.from_workload(wl), upload_weights(L, "bf16"), to_dev(L["x"], "bf16")
        ws = alloc_ws(cfg)
        ws.fill_(0xAB)
        outs = [torch.empty_like(x) for _ in range(3)]
        M.moe_layer_forward(cfg, W, x, None, outs[0], ws)
        M.moe_layer_experts(cfg, W, x, None, outs[1], ws)
        M.moe_layer_experts(cfg, W, x, None, outs[2], ws)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        ref = O.layer_forward(L["x"], L, E=wl.E, k=2, capacity_factor=0.0, renormalize=True, act="gelu")
        assert rel_fro(to_np(outs[0]), ref["out"]) < TOL


def test_sixteen_assignments_over_a_contraction_beyond_32_bit_tiles():
    """64 weight rows of 2^25 bf16 values are 4 GiB, past what the weight-streaming tiles can address: the matrix-vector
    kernel serves the second product.  Against the same product in float32 pieces (bar as above)."""
    T, d, f, P = 12, 64, 1 << 25, 1 << 22
    print(T, d, f, flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    w1 = torch.empty(1, f, d, dtype=torch.bfloat16, device="cuda").normal_(0, d ** -0.5, generator=g)
    w2 = torch.empty(1, d, f, dtype=torch.bfloat16, device="cuda").normal_(0, f ** -0.5, generator=g)
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=1, k=1)
    W = M.Weights({"w1": w1, "w2": w2, "w_router": torch.zeros(d, 1, device="cuda")})
    y = torch.full_like(x, float("nan"))
    M.moe_expert_ffn(cfg, W, x, torch.tensor([0, T], dtype=torch.int32, device="cuda"), y, alloc_ws(cfg, 2))
    want = torch.zeros(T, d, dtype=torch.float64, device="cuda")
    for i in range(0, f, P):
        h = torch.nn.functional.gelu(x.float() @ w1[0, i:i + P].float().t()).bfloat16().float()
        want += (h @ w2[0, :, i:i + P].float().t()).double()
    err = float((y.double() - want).norm() / want.norm())
    print("rel fro", err, flush=True)
    assert err < TOL


@pytest.mark.parametrize("name,kw", [
    ("ring", dict(T=8, d_model=256, d_ff=512, E=64)), ("gpt", dict(T=6, E=2, d_model=256, d_ff=4096, capacity_factor=0.0)),
    ("skew", dict(T=13, d_model=256, d_ff=512)), ("large", dict(T=7, d_model=512, d_ff=1024, E=4))], ids=str)
def test_matrix_vector_kernel_of_nine_to_sixteen_assignments(name, kw):
    """Its 4 x 16 shape, with the weight-streaming kernels kept out by a tuning key."""
    wl = WORKLOADS[name].scaled(**kw)
    print(wl, flush=True)
    L = make_layer(wl, with_bias=True)
    ref = O.layer_forward(L["x"], L, E=wl.E, k=wl.k, capacity_factor=wl.capacity_factor, renormalize=wl.renormalize, act=wl.act)
    M.moe_set_tuning(M.MOE_TUNE_GEMM_TILE_ROWS, 256)
    try:
        assert rel_fro(run_layer(M.MoEConfig.from_workload(wl), upload_weights(L, "bf16"), to_dev(L["x"], "bf16"))["out"], ref["out"]) < TOL
    finally:
        M.moe_set_tuning(M.MOE_TUNE_GEMM_TILE_ROWS, 0)
