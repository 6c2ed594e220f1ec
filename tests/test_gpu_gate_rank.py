"""Routing of up to 256 tokens through slices of the contraction index and one ranking workgroup: tables exact against float64 at the
edges of token tiles, of the logits per thread, of the expert groups and of the rule; and one-token layers whose first product ranks."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

from gpu_util import routing

pytestmark = pytest.mark.gpu


def tables(cfg, x, router, bias):
    T, E, k = cfg.T, cfg.E, cfg.k
    z = (x.double() @ router.double() + bias.double()).cpu()
    idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :k].numpy()
    p = np.take_along_axis(torch.softmax(z, 1).numpy(), idx, 1)
    if cfg.renormalize:
        p = p / p.sum(1, keepdims=True)
    cap = max(1, int(np.ceil(k * T * cfg.capacity_factor / E))) if cfg.capacity_factor else k * T
    counts, a2r = np.bincount(idx.reshape(-1), minlength=E), np.full(T * k, -1)
    offsets = np.concatenate([[0], np.cumsum(np.minimum(counts, cap))])
    seen, r2a = np.zeros(E, int), np.zeros(offsets[-1], int)
    for a, e in enumerate(idx.T.reshape(-1)):
        if seen[e] < cap:
            a2r[a] = offsets[e] + seen[e]
            r2a[a2r[a]] = a
        seen[e] += 1
    return idx, p, counts, offsets, a2r, r2a


def reader(ws, cfg):
    lay = M.moe_workspace_layout(cfg)
    return lambda n, c, dt=torch.int32: ws[lay[n]:lay[n] + 4 * c].view(dt).cpu().numpy()


def check_tables(read, cfg, x, router, bias):
    T, E, k = cfg.T, cfg.E, cfg.k
    idx, p, counts, offsets, a2r, r2a = tables(cfg, x, router, bias)
    assert np.array_equal(read("topk_idx", T * k).reshape(T, k), idx)
    # float32 exponentials, their sum and one division: a few units in the last place
    assert np.abs(read("topk_w", T * k, torch.float32).reshape(T, k) - p).max() < 16 * 2.0 ** -24
    assert np.array_equal(read("expert_counts", E), counts) and np.array_equal(read("expert_offsets", E + 1), offsets)
    assert np.array_equal(read("assign_to_row", T * k), a2r) and np.array_equal(read("row_to_assign", offsets[-1]), r2a)
    assert not read("tile_counters", 8).any()


def problem(T, d, E):
    g = torch.Generator(device="cuda").manual_seed(d + E + T)
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    router = torch.randn(d, E, generator=g, device="cuda") * d ** -0.5
    router[:, 3] = router[:, 1]                            # exact ties
    bias = torch.randn(E, generator=g, device="cuda")
    bias[3] = bias[1] = 1.5
    return g, x, router, bias


@pytest.mark.parametrize("T,d,E,k,cf", [
    (1, 64, 5, 1, 0.0), (2, 64, 4, 4, 1.0), (15, 192, 17, 3, 0.0), (16, 1024, 64, 8, 1.0), (17, 2112, 65, 2, 0.0), (31, 1600, 128, 6, 1.25),
    (32, 256, 256, 8, 0.0), (33, 320, 200, 2, 0.0), (64, 1088, 64, 2, 1.0), (96, 4096, 8, 2, 0.0), (97, 1472, 9, 2, 1.0), (97, 1536, 9, 2, 1.0),
    (128, 2048, 64, 8, 0.0), (129, 2048, 64, 2, 0.0), (255, 1536, 12, 4, 0.5), (256, 2048, 32, 4, 0.0), (256, 4160, 33, 2, 0.0), (257, 2048, 8, 1, 0.0)])
def test_gate_rank(T, d, E, k, cf):
    print(T, d, E, k, cf, flush=True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=2048, E=E, k=k, capacity_factor=cf, renormalize=bool(T & 1))
    assert routing(cfg, 1) == ("split" if T == 257 or (T, d) == (97, 1472) or T * E > 8192 else "slices")
    _, x, router, bias = problem(T, d, E)
    one = torch.zeros(1, dtype=torch.bfloat16, device="cuda")
    W = M.Weights({"w1": one, "w2": one, "w_router": router, "b_router": bias}, "output_major")
    W.need = lambda c: None                                # (routing reads no expert)
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB)
    for _ in range(2):
        M.moe_layer_route(cfg, W, x, ws)
        torch.cuda.synchronize()
        check_tables(reader(ws, cfg), cfg, x, router, bias)


@pytest.mark.parametrize("d,f,E,k,act,special", [
    (64, 64, 4, 2, "gelu", ""), (128, 512, 64, 8, "gelu", ""), (576, 192, 24, 2, "swiglu", ""), (1088, 8192, 9, 2, "gelu", ""), (1024, 16384, 8, 2, "gelu", ""),
    (4096, 2048, 8, 2, "gelu", ""), (4096, 3584, 8, 2, "swiglu", ""), (4160, 8128, 9, 2, "gelu", ""), (4608, 64, 16, 2, "swiglu", ""), (6208, 64, 4, 3, "gelu", ""),
    (4096, 8192, 4, 2, "gelu", ""), (4096, 4096, 8, 2, "swiglu", ""),
    (2048, 8192, 64, 4, "swiglu", ""), (1024, 2048, 33, 8, "gelu", "nan"), (1024, 2048, 16, 4, "swiglu", "masked"), (1024, 2048, 16, 2, "gelu", "inf")])
def test_one_token_layer(d, f, E, k, act, special):
    """The whole layer against routing and experts in two calls, which rank in a kernel of their own: the same bits."""
    print(d, f, E, k, act, special, flush=True)
    cfg = M.MoEConfig(T=1, d_model=d, d_ff=f, E=E, k=k, act=act, renormalize=bool(E & 1))
    assert (routing(cfg, 0), routing(cfg, 1)) == ("parts + ranking product", "parts + ranking")
    g, x, router, bias = problem(1, d, E)
    if special == "nan":
        x[0, 7] = float("nan")
    if special == "masked":
        bias[2:] = -float("inf")
    if special == "inf":
        bias[3] = float("inf")
    mat = lambda n, k_: (torch.randn(E, n, k_, generator=g, device="cuda") * k_ ** -0.5).bfloat16()
    t = {"w_router": router, "b_router": bias}
    if act == "gelu":
        t.update(w1=mat(f, d), w2=mat(d, f), b1=torch.randn(E, f, generator=g, device="cuda").bfloat16(), b2=torch.randn(E, d, generator=g, device="cuda").bfloat16())
    else:
        t.update(w_gate_proj=mat(f, d), w_up=mat(f, d), w_down=mat(d, f))
    W = M.Weights(t, "output_major")
    ws, ws2 = (torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB) for _ in range(2))
    out, out2 = torch.empty_like(x), torch.empty_like(x)
    M.moe_layer_route(cfg, W, x, ws2)
    M.moe_layer_experts(cfg, W, x, x, out2, ws2)
    for _ in range(2):
        M.moe_layer_forward(cfg, W, x, x, out, ws)
        torch.cuda.synchronize()
        a, b = reader(ws, cfg), reader(ws2, cfg)
        for n, c in (("topk_idx", k), ("expert_counts", E), ("expert_offsets", E + 1), ("assign_to_row", k), ("tile_counters", 8)):
            assert np.array_equal(a(n, c), b(n, c)), n
        rows = int(a("expert_offsets", E + 1)[-1])
        assert np.array_equal(a("row_to_assign", rows), b("row_to_assign", rows))
        assert np.array_equal(a("h", rows * f // 2), b("h", rows * f // 2))  # the same sums in the same order
        if not special:
            check_tables(a, cfg, x, router, bias)
        assert np.array_equal(a("topk_w", k), b("topk_w", k))    # bits
        assert torch.equal(out.view(torch.int16), out2.view(torch.int16))


@pytest.mark.parametrize("T,d,E,k", [(1, 2048, 64, 2), (1, 1024, 16, 4), (1, 4096, 32, 8), (1, 576, 8, 2), (1, 512, 4, 4), (2, 1024, 8, 2), (3, 2048, 64, 8),
                                     (5, 320, 4, 2), (8, 2048, 64, 2), (9, 4096, 32, 2), (15, 1088, 16, 3), (16, 2048, 64, 8), (16, 64, 4, 4)])
@pytest.mark.parametrize("renorm", [False, True])
def test_weights_are_those_of_the_gate_alone(T, d, E, k, renorm):
    """Up to 16 tokens on 4, 8, 16, 32 or 64 experts: whichever kernel ranks inside a layer, its weights are moe_gate's, bit for bit
    (logits: float64 sums of exact products, so that their order does not show in float32; the softmax in the same order)."""
    print(T, d, E, k, renorm, flush=True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=512, E=E, k=k, renormalize=renorm)
    for seed in range(8):
        g, x, router, bias = problem(T, d + seed, E)
        x, router = x[:, :d].contiguous(), router[:d].contiguous()
        mat = lambda n, m: (torch.randn(E, n, m, generator=g, device="cuda") * m ** -0.5).bfloat16()
        W = M.Weights({"w_router": router, "b_router": bias, "w1": mat(512, d), "w2": mat(d, 512)}, "output_major")
        idx, w = torch.empty(T, k, dtype=torch.int32, device="cuda"), torch.empty(T, k, device="cuda")
        M.moe_gate(cfg, x, router, bias, idx, w)
        out = torch.empty_like(x)
        for call in (lambda ws: M.moe_layer_route(cfg, W, x, ws), lambda ws: M.moe_layer_forward(cfg, W, x, None, out, ws)):
            ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB)
            call(ws)
            torch.cuda.synchronize()
            read = reader(ws, cfg)
            assert np.array_equal(read("topk_idx", T * k).reshape(T, k), idx.cpu().numpy())
            assert np.array_equal(read("topk_w", T * k).reshape(T, k), w.view(torch.int32).cpu().numpy())


@pytest.mark.parametrize("T,d,f,E,k", [(1, 2048, 8192, 64, 2), (1, 1024, 2048, 33, 8), (1, 512, 64, 16, 2), (1, 576, 192, 24, 2), (8, 2048, 2048, 64, 2), (96, 1024, 512, 8, 2)])
def test_routing_leaves_the_experts_outputs(T, d, f, E, k):
    """moe_layer_route may use h as scratch, and nothing else of what a pass before left in the workspace: yd stays as it is."""
    print(T, d, f, E, k, flush=True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k)
    _, x, router, bias = problem(T, d, E)
    one = torch.zeros(1, dtype=torch.bfloat16, device="cuda")
    W = M.Weights({"w1": one, "w2": one, "w_router": router, "b_router": bias}, "output_major")
    W.need = lambda c: None                                # (routing reads no expert)
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB)
    M.moe_layer_route(cfg, W, x, ws)
    torch.cuda.synchronize()
    check_tables(reader(ws, cfg), cfg, x, router, bias)
    lay = M.moe_workspace_layout(cfg)
    assert (ws[lay["yd"]:lay["yd"] + k * T * d * 2] == 0xAB).all()
