"""Experts masked by a router bias of -inf: never chosen while others are left, and where fewer are left than a token wants the
masked ones follow in order of their index with weight zero, each expert once.  Every gate kernel, and the routing tables."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


def problem(T, d, E, dtype, left, seed=3):
    g = torch.Generator(device="cuda").manual_seed(seed + T + d + E)
    x = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    router = torch.randn(d, E, generator=g, device="cuda") * d ** -0.5
    bias = torch.full((E,), -float("inf"), device="cuda")
    bias[[(5 * i + 2) % E for i in range(left)]] = 0.25
    return x, router, bias


def reference(x, router, bias, k, renorm):
    z = (x.double() @ router.double() + bias.double()).cpu()
    idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :k].numpy()
    p = np.take_along_axis(torch.softmax(z, 1).numpy(), idx, 1)
    return idx, p / p.sum(1, keepdims=True) if renorm else p


@pytest.mark.parametrize("T,d,E,dtype,packed", [
    (1, 512, 8, "bf16", False), (16, 512, 64, "bf16", False),                                   # a workgroup per token
    (300, 512, 7, "bf16", False), (300, 512, 16, "bf16", False), (999, 1024, 64, "bf16", False),  # split router weights
    (2048, 512, 40, "bf16", False), (100, 256, 100, "bf16", False), (33, 256, 256, "bf16", False), (70, 256, 9, "f32", False),
    (4097, 1024, 64, "bf16", True), (300, 512, 24, "bf16", True)])
@pytest.mark.parametrize("left,k", [(1, 2), (2, 4), (4, 4), (3, 2)])
def test_masked_experts(T, d, E, dtype, packed, left, k):
    print(T, d, E, dtype, packed, left, k, flush=True)
    x, router, bias = problem(T, d, E, dtype, left)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=64, E=E, k=k, dtype=dtype, renormalize=bool(left & 1))
    idx, w = torch.full((T, k), -7, dtype=torch.int32, device="cuda"), torch.full((T, k), float("nan"), device="cuda")
    if packed:
        pk = torch.empty(M.moe_router_pack_bytes(d, E), dtype=torch.uint8, device="cuda")
        M.moe_pack_router(router, pk)
        M.moe_gate_packed(cfg, x, router, bias, pk, idx, w)
    else:
        M.moe_gate(cfg, x, router, bias, idx, w)
    torch.cuda.synchronize()
    want_idx, want_w = reference(x, router, bias, k, cfg.renormalize)
    assert np.array_equal(idx.cpu().numpy(), want_idx)
    # float32 logits' exponentials and one division: a few units in the last place of numbers up to one
    assert np.abs(w.cpu().numpy() - want_w).max() < 64 * 2.0 ** -24


@pytest.mark.parametrize("T,d,E", [(1, 512, 8), (1, 2048, 64), (5, 2048, 64)])     # one token's own tables, router slices
@pytest.mark.parametrize("left,k", [(1, 2), (2, 4), (3, 2)])
def test_masked_experts_of_a_layer(T, d, E, left, k):
    print(T, d, E, left, k, flush=True)
    x, router, bias = problem(T, d, E, "bf16", left)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=4096, E=E, k=k)
    one = torch.zeros(1, dtype=torch.bfloat16, device="cuda")
    W = M.Weights({"w1": one, "w2": one, "w_router": router, "b_router": bias}, "output_major")
    W.need = lambda c: None                                # (routing reads no expert)
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB)
    M.moe_layer_route(cfg, W, x, ws)
    torch.cuda.synchronize()
    lay = M.moe_workspace_layout(cfg)
    read = lambda n, c: ws[lay[n]:lay[n] + 4 * c].view(torch.int32).cpu().numpy()
    idx = reference(x, router, bias, k, False)[0]
    e = idx.T.reshape(-1)
    a2r = np.empty(T * k, int)
    a2r[np.argsort(e, kind="stable")] = np.arange(T * k)
    assert np.array_equal(read("topk_idx", T * k).reshape(T, k), idx)
    assert np.array_equal(read("expert_counts", E), np.bincount(e, minlength=E))
    assert np.array_equal(read("expert_offsets", E + 1), np.concatenate([[0], np.cumsum(np.bincount(e, minlength=E))]))
    assert np.array_equal(read("assign_to_row", T * k), a2r)
    assert np.array_equal(read("row_to_assign", T * k), np.argsort(e, kind="stable"))
