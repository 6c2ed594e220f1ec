"""Dispatch bookkeeping on both sides of the rule that hands the block bases to the scan kernel, and the weight
transpose's vector and element-wise kernels: integers and byte copies, so every comparison is exact."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M
from oracle import moe_oracle as O

from gpu_util import alloc_ws

pytestmark = pytest.mark.gpu


# blocks x experts: 2048 words (own sums), one block more (scan kernel); 1 and 255..256 experts; a last run of blocks
# that is empty (17 blocks over 16 runs of two), more experts than one scan workgroup serves
@pytest.mark.parametrize("T,E,k,cf", [(4096, 64, 2, 0.0), (4097, 64, 2, 1.0), (2175, 256, 2, 0.7), (1500, 255, 6, 0.0),
                                      (70000, 1, 1, 0.5), (41000, 16, 3, 1.25), (130000, 5, 1, 0.0), (2048, 128, 8, 1.0)])
def test_dispatch_tables(T, E, k, cf):
    rng = np.random.default_rng(T + E)
    p = rng.dirichlet(np.full(E, 0.7))
    z = np.log(p + 1e-9) + rng.gumbel(size=(T, E))
    idx = np.argsort(-z, axis=1, kind="stable")[:, :k].astype(np.int32)
    cfg = M.MoEConfig(T=T, d_model=64, d_ff=64, E=E, k=k, capacity_factor=cf)
    A = T * k
    C = O.capacity(T, E, k, cf)
    bufs = [torch.full((n,), -5, dtype=torch.int32, device="cuda") for n in (E, E + 1, A, A)]
    M.moe_dispatch(cfg, None, torch.from_numpy(idx).cuda(), *bufs, None, alloc_ws(cfg, 1))
    torch.cuda.synchronize()
    counts, offsets, a2r, r2a = (b.cpu().numpy() for b in bufs)
    rc, ro, ra, rr, _ = O.dispatch(np.zeros((T, 1)), idx, E, C)
    assert np.array_equal(counts, rc) and np.array_equal(offsets, ro) and np.array_equal(a2r, ra)
    assert np.array_equal(r2a[:int(ro[-1])], rr)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("E,rows,cols,shift", [(2, 64, 64, 0), (3, 72, 200, 0), (1, 8, 8, 0), (2, 1000, 520, 0),
                                               (2, 63, 64, 0), (2, 64, 65, 0), (1, 128, 128, 1)])
def test_transpose(E, rows, cols, shift, dtype):
    """Whole vectors and ragged ones; shift: pointers off the 16-byte grid."""
    n = E * rows * cols
    src = torch.randn(n + shift, device="cuda").to(dtype)[shift:].view(E, rows, cols)
    guard = torch.full((n + shift + 8,), 7.0, dtype=dtype, device="cuda")
    dst = guard[shift:shift + n].view(E, cols, rows)
    M.moe_transpose_expert_weights(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(dst, src.transpose(1, 2))
    assert bool((guard[shift + n:] == 7.0).all())
