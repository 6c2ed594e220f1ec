"""Dispatch bookkeeping around the sizes where its kernels change (one workgroup of 256 threads, of 1024 with one, two and four
assignments each, several workgroups): exact tables with and without a capacity that drops, expert counts on both sides of
a wavefront, indices outside the range."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k", [(256, 1), (257, 1), (128, 2), (129, 2), (512, 2), (1025, 1), (1024, 2), (683, 3), (2048, 2), (4097, 1), (1366, 3)])
@pytest.mark.parametrize("E", [3, 64, 65, 256])
@pytest.mark.parametrize("cf", [0.0, 0.5])
def test_dispatch_sizes(T, k, E, cf):
    cfg = M.MoEConfig(T=T, d_model=64, d_ff=64, E=E, k=k, capacity_factor=cf)
    rng = np.random.default_rng(T * k + E)
    # a third on one expert; a few outside the range, which are dropped
    idx = np.where(rng.random((T, k)) < 0.3, E - 1, rng.integers(0, E, (T, k))).astype(np.int32)
    idx[rng.random((T, k)) < 0.02] = E
    idx[0, 0] = -1
    cap = max(1, int(np.ceil(k * T * np.float64(cf) / E))) if cf else k * T
    e = idx.T.reshape(-1)                              # priority order: first choices, in token order, before second ones
    counts = np.array([(e == i).sum() for i in range(E)], np.int32)
    offsets = np.concatenate([[0], np.cumsum(np.minimum(counts, cap))]).astype(np.int32)
    a2r = np.full(T * k, -1, np.int32)
    r2a = np.full(T * k, -7, np.int32)
    seen = np.zeros(E, np.int64)
    for a, i in enumerate(e):
        if 0 <= i < E:
            if seen[i] < cap:
                a2r[a] = offsets[i] + seen[i]
                r2a[a2r[a]] = a
            seen[i] += 1
    got = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (E, E + 1, T * k, T * k)]
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda").fill_(0xAB)
    M.moe_dispatch(cfg, None, torch.from_numpy(idx).cuda(), *got, None, ws)
    torch.cuda.synchronize()
    for want, t in zip((counts, offsets, a2r, r2a), got):
        assert np.array_equal(want, t.cpu().numpy())
