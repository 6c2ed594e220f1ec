"""A token whose logits do not compare (NaN) is dropped: its assignments get no row, and the routing, tables, outputs and
gradients of the other tokens are those they have beside a token that is not NaN."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


def place(T):
    """Positions of the NaN tokens: first, middle, last, and two at once."""
    return [[0], [T // 2], [T - 1], [0, T - 1]] if T > 1 else [[0]]


def layer(d, f, E, T, k, seed=0, act="gelu", cf=0.0, dtype="bf16", renorm=False):
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, act=act, capacity_factor=cf, dtype=dtype, renormalize=renorm)
    g = torch.Generator(device="cuda").manual_seed(seed + d + E + T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    mat = lambda o, i: (torch.randn(E, o, i, generator=g, device="cuda") * i ** -0.5).to(dt)
    t = {"w1": mat(f, d), "w2": mat(d, f)} if act == "gelu" else {"w_gate_proj": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)}
    t["w_router"] = torch.randn(d, E, generator=g, device="cuda") * d ** -0.5
    t["b_router"] = torch.zeros(E, device="cuda")
    t["b_router"][E - 1] = 2.0                             # (an expert whose index has every bit set is popular)
    x = torch.randn(T, d, generator=g, device="cuda").to(dt)
    return cfg, M.Weights(t, "output_major"), x


def tables(idx, bad, E, cap):
    """counts, offsets, assignment -> row, row -> assignment of the selections idx [T, k] without the tokens in bad."""
    T, k = idx.shape
    e = idx.T.reshape(-1).copy()
    e[np.tile(np.isin(np.arange(T), bad), k)] = -1
    counts = np.bincount(e[e >= 0], minlength=E)
    offsets = np.concatenate([[0], np.cumsum(np.minimum(counts, cap))])
    a2r, r2a, seen = np.full(T * k, -1), np.zeros(offsets[-1], int), np.zeros(E, int)
    for a, i in enumerate(e):
        if i >= 0:
            if seen[i] < cap:
                a2r[a] = offsets[i] + seen[i]
                r2a[a2r[a]] = a
            seen[i] += 1
    return counts, offsets, a2r, r2a


def forward(cfg, W, x, residual, ws=None, fill=0.0):
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB) if ws is None else ws
    out = torch.full_like(x, fill)
    M.moe_layer_forward(cfg, W, x, residual, out, ws)
    torch.cuda.synchronize()
    lay = M.moe_workspace_layout(cfg)
    read = lambda n, c: ws[lay[n]:lay[n] + 4 * c].view(torch.int32).cpu().numpy()
    A, E = cfg.T * cfg.k, cfg.E
    offsets = read("expert_offsets", E + 1)
    return out, (read("expert_counts", E), offsets, read("assign_to_row", A), read("row_to_assign", int(offsets[E]))), ws


def check(cfg, W, x, bad, residual):
    """One layer with the tokens in bad NaN against the same layer with ordinary tokens in their place."""
    cap = max(1, int(np.ceil(cfg.k * cfg.T * cfg.capacity_factor / cfg.E))) if cfg.capacity_factor else cfg.k * cfg.T
    good = [t for t in range(cfg.T) if t not in bad]
    xn = x.clone()
    xn[bad, ::7] = float("nan")
    z = (x.double() @ W.tensors["w_router"].double() + W.tensors["b_router"].double()).cpu()
    idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :cfg.k].numpy()
    ref, _, _ = forward(cfg, W, x, x if residual else None)
    for fill in (3.0, float("nan")):
        out, got, _ = forward(cfg, W, xn, xn if residual else None, fill=fill)
        for want, have in zip(tables(idx, bad, cfg.E, cap), got):
            assert np.array_equal(want, have), (cfg, bad)
        if not cfg.capacity_factor:                        # (a dropped token may make room for another one)
            assert torch.equal(out[good], ref[good]), (cfg, bad)


@pytest.mark.parametrize("d,f,E,k", [(2048, 1024, 64, 2), (2048, 512, 64, 8), (16384, 256, 8, 2)])
@pytest.mark.parametrize("T", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("cf", [0.0, 1.0])
def test_sliced_gate(d, f, E, k, T, cf):
    cfg, W, x = layer(d, f, E, T, k, cf=cf)
    for bad in place(T):
        print(d, E, T, k, cf, bad, flush=True)
        check(cfg, W, x, bad, residual=True)


@pytest.mark.parametrize("d,f,E", [(1024, 512, 64), (2048, 512, 8), (512, 256, 4), (2048, 1024, 64)])   # (the last: slices)
@pytest.mark.parametrize("k", [2, 4])
@pytest.mark.parametrize("residual", [False, True])
def test_one_token(d, f, E, k, residual):
    print(d, E, k, residual, flush=True)
    cfg, W, x = layer(d, f, E, 1, k)
    check(cfg, W, x, [0], residual)
    xn = torch.full_like(x, float("nan"))
    out, (counts, offsets, a2r, _), ws = forward(cfg, W, xn, xn if residual else None, fill=3.0)
    assert not counts.any() and not offsets.any() and (a2r == -1).all()
    assert bool(out.isnan().all() if residual else (out == 0).all())     # (its residual; no expert added anything)
    ref = forward(cfg, W, x, x)[0]
    assert torch.equal(forward(cfg, W, x, x, ws=ws)[0], ref)             # the workspace serves the next step


@pytest.mark.parametrize("T,E,k,act,renorm", [(300, 8, 2, "gelu", False), (300, 8, 2, "swiglu", True), (131, 20, 1, "gelu", True), (8, 64, 2, "gelu", False)])
def test_backward(T, E, k, act, renorm):
    """Gradients of a layer with NaN tokens against those with ordinary tokens in their place whose upstream gradient is
    zero: alike for the experts and the other tokens, NaN for the router and the NaN tokens."""
    print(T, E, k, act, renorm, flush=True)
    d, f = (2048, 512) if E == 64 else (512, 512)
    cfg, W, x = layer(d, f, E, T, k, act=act, renorm=renorm)
    g = torch.Generator(device="cuda").manual_seed(5)
    G = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    bad = [0, T // 2, T - 1]
    good = [t for t in range(T) if t not in bad]
    G[bad] = 0
    im = lambda n: W.tensors[n].transpose(1, 2).contiguous()
    w1, w2 = (torch.cat([im("w_gate_proj"), im("w_up")], 2), im("w_down")) if act == "swiglu" else (im("w1"), im("w2"))
    f1 = 2 * f if act == "swiglu" else f

    def step(xs):
        nan = lambda *shape: torch.full(shape, float("nan"), device="cuda")
        d_x, d_wr, d_br, d_w1, d_w2 = torch.full_like(x, float("nan")), nan(d, E), nan(E), nan(E, f1, d), nan(E, d, f)
        ws = forward(cfg, W, xs, xs)[2]
        bws = torch.empty(M.moe_layer_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        M.moe_layer_backward(cfg, W, w1, w2, xs, G, None, ws, d_x, d_wr, d_br, d_w1, None, d_w2, None, bws)
        torch.cuda.synchronize()
        return d_x, d_wr, d_br, d_w1, d_w2

    xn = x.clone()
    xn[bad, ::7] = float("nan")
    want, got = step(x), step(xn)
    assert torch.equal(got[0][good], want[0][good]) and bool(got[0][bad].isnan().all())
    assert bool(got[1].isnan().all()) and bool(got[2].isnan().all())
    for a, b in zip(got[3:], want[3:]):
        # the same float32 sums without a few terms that are zero: up to T roundings of 2^-24 in other places
        assert float((a - b).norm() / b.norm()) < 4 * T ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("T,E,d,f,kernel", [
    (1, 4, 512, 512, "gemv 8"), (7, 8, 1024, 512, "gemv 8"), (12, 8, 512, 512, "stream 64x32"), (40, 4, 512, 512, "stream 64x32"),
    (300, 2, 64, 256, "stream 64x64"), (2000, 3, 1024, 256, "stream 128x192"), (4000, 32, 1088, 2560, "stream 256x192"),
    (20000, 64, 128, 256, "grouped 128"), (2500, 6, 2048, 256, "grouped 256"), (24000, 24, 320, 256, "grouped 256"), (8000, 2, 2048, 256, "grouped 320")])
@pytest.mark.parametrize("residual", [False, True, "in place"])
def test_one_expert_per_token(T, E, d, f, kernel, residual):
    """k = 1: the second product's kernel writes `out` itself, also the rows that no tile holds."""
    from gpu_util import product_kernel
    cfg, W, x = layer(d, f, E, T, 1)
    print(T, E, d, f, residual, product_kernel(cfg, 1), flush=True)
    assert product_kernel(cfg, 1) == kernel
    ref = forward(cfg, W, x, x if residual else None)[0]
    for bad in place(T) + [list(range(T))]:
        good = [t for t in range(T) if t not in bad]
        xn = x.clone()
        xn[bad, 3] = float("nan")
        res = xn if residual else None
        ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB)
        out = xn if residual == "in place" else torch.full_like(x, 3.0)
        want = torch.zeros_like(x[bad]) if res is None else xn[bad].clone()
        M.moe_layer_forward(cfg, W, xn, res, out, ws)
        torch.cuda.synchronize()
        assert torch.equal(out[good], ref[good])
        assert torch.equal(out[bad].view(torch.int16), want.view(torch.int16))


def product_name(cfg, second):
    if cfg.dtype == "f32":
        import ctypes as C
        f = M.lib().moe_test_f32_tile_rows
        f.restype = C.c_int32
        return f"{f(C.byref(cfg.c()), second)} rows"
    from gpu_util import product_kernel
    return product_kernel(cfg, second)


@pytest.mark.parametrize("dtype,act,rows,E,d,f,k,kernels", [
    ("bf16", "gelu", 120, 16, 1280, 4416, 2, ("stream 256x192", "stream 128x192")), ("bf16", "swiglu", 110, 32, 1600, 2624, 2, ("stream 256x192",) * 2),
    ("bf16", "gelu", 2, 4, 512, 512, 1, ("gemv 8",) * 2), ("bf16", "gelu", 20, 8, 512, 512, 2, ("stream 64x32",) * 2),
    ("bf16", "swiglu", 700, 8, 1024, 1024, 2, ("grouped 256", "stream 128x192")), ("f32", "gelu", 66, 16, 896, 1792, 2, ("80 rows",) * 2),
    ("f32", "swiglu", 256, 16, 1024, 1984, 2, ("160 rows",) * 2), ("f32", "gelu", 40, 8, 256, 512, 1, ("32 rows",) * 2), ("f32", "gelu", 435, 8, 512, 1856, 1, ("64 rows",) * 2)])
def test_rows_of_an_expert_stay_apart(dtype, act, rows, E, d, f, k, kernels):
    """Rows with NaN or infinite activations (an expert's first, last and one inside, beside experts without any) leave every
    other row as it is, bit for bit."""
    print(dtype, act, rows, E, d, f, flush=True)
    n = [max(1, rows + (i % 3 - 1) * (rows // 4)) for i in range(E)]
    cfg, W, _ = layer(d, f, E, rows * E // k, k, act=act, dtype=dtype)
    assert (product_name(cfg, 0), product_name(cfg, 1)) == kernels
    n[-1] = rows * E - sum(n[:-1])
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn(int(off[-1]), d, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    bad = sorted({int(r) for e in range(0, E, 2) for r in (off[e], off[e] + n[e] // 2, off[e + 1] - 1)})
    good = sorted(set(range(int(off[-1]))) - set(bad))
    xn = x.clone()
    xn[bad, ::5] = float("nan")
    xn[bad[::2]] = float("inf")
    ws = torch.empty(M.moe_workspace_bytes(cfg, 2), dtype=torch.uint8, device="cuda")
    outs = []
    for a in (x, xn):
        y = torch.full_like(x, 7.0)
        ws.fill_(0xAB)
        M.moe_expert_ffn(cfg, W, a, torch.from_numpy(off).cuda(), y, ws)
        torch.cuda.synchronize()
        outs.append(y)
    assert torch.equal(outs[0][good], outs[1][good]) and bool(outs[0].isfinite().all())
    assert not bool(outs[1][bad].isfinite().any())


@pytest.mark.parametrize("E,rows,N1,N2", [(9, [70, 33, 0, 64, 1], 512, 768), (8, [1500, 1403], 512, 512), (3, [130, 65], 512, 512)])
def test_weight_gradients_of_experts_stay_apart(E, rows, N1, N2):
    """An expert whose rows hold NaN and infinities beside one that ends in the middle of a step: its own gradient only."""
    print(E, rows, N1, N2, flush=True)
    n = [rows[i % len(rows)] for i in range(E)]
    off = np.concatenate([[0], np.cumsum(n)])
    g = torch.Generator(device="cuda").manual_seed(E)
    a, b = (torch.randn(int(off[-1]), w, generator=g, device="cuda").bfloat16() for w in (N1, N2))
    offsets = torch.tensor(off, dtype=torch.int32, device="cuda")
    an, bn = a.clone(), b.clone()
    for e in range(1, E, 2):
        an[off[e]:off[e + 1]] = float("nan")
        bn[off[e]:off[e + 1], ::3] = float("inf")
    for dt in (torch.float32, torch.bfloat16):
        c = [torch.full((E, N1, N2), 7.0, dtype=dt, device="cuda") for _ in range(2)]
        s = [torch.full((E, N1), 7.0, device="cuda") for _ in range(2)]
        M.moe_expert_wgrad(a, b, offsets, c[0], max(n), a_column_sums=s[0])
        M.moe_expert_wgrad(an, bn, offsets, c[1], max(n), a_column_sums=s[1])
        torch.cuda.synchronize()
        assert torch.equal(c[0][::2], c[1][::2]) and torch.equal(s[0][::2], s[1][::2])
        assert all(bool(c[1][e].isnan().all()) for e in range(1, E, 2) if n[e])
