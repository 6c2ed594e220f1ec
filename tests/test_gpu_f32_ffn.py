"""float32 expert FFN on the float32 matrix instructions: both kernels (the rule is on the tile count), both weight layouts,
experts whose rows end on and beside the tile edges, feature counts of one and several tiles, pointers on odd floats."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M
from oracle import moe_oracle as O

from gpu_util import alloc_ws, rel_fro

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 0, 63, 64, 65, 95, 96, 97, 128, 2]


# few tiles (split contraction index) and many; K of two chunks (six of the eight split wavefronts idle) to 34
@pytest.mark.parametrize("act,rows,d,f,shift", [
    ("gelu", EDGES, 64, 64, 0), ("swiglu", EDGES, 64, 128, 0), ("gelu", [5], 1088, 192, 0), ("swiglu", [0, 33], 320, 64, 1),
    ("gelu", EDGES * 2, 128, 1344, 0), ("swiglu", EDGES * 2, 192, 1024, 0), ("gelu", [700, 0, 0, 900], 576, 832, 1),
    ("gelu", [3] * 256, 64, 128, 0), ("swiglu", [1] * 255, 64, 192, 0)], ids=str)
@pytest.mark.parametrize("layout", ["output_major", "input_major"])
def test_f32_ffn(act, rows, d, f, shift, layout):
    print(act, len(rows), d, f, shift, layout, flush=True)
    rng = np.random.default_rng(d + f)
    E, R = len(rows), sum(rows)
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    xd = rng.standard_normal((R, d)).astype(np.float32)
    mats = {n: (rng.standard_normal((E, a, b)) * a ** -0.5).astype(np.float32)
            for n, a, b in ([("w1", d, f), ("w2", f, d)] if act == "gelu" else [("w_gate_proj", d, f), ("w_up", d, f), ("w_down", f, d)])}
    if act == "gelu":
        mats["b1"], mats["b2"] = rng.standard_normal((E, f)).astype(np.float32), rng.standard_normal((E, d)).astype(np.float32)
    ref = O.expert_ffn(xd, offsets, mats, act)

    def dev(a):  # `shift` floats off the allocation's alignment
        buf = torch.empty(a.size + shift, device="cuda")
        t = buf[shift:].view(a.shape)
        t.copy_(torch.from_numpy(np.ascontiguousarray(a)))
        return t

    t = {n: dev(a if layout == "input_major" or a.ndim < 3 else a.transpose(0, 2, 1)) for n, a in mats.items()}
    t["w_router"] = torch.zeros(d, E, device="cuda")
    cfg = M.MoEConfig(T=max(R, 1), d_model=d, d_ff=f, E=E, k=1, act=act, dtype="f32")
    guard = torch.full((R + 1, d), 7.0, device="cuda")
    M.moe_expert_ffn(cfg, M.Weights(t, layout), dev(xd), torch.from_numpy(offsets).cuda(), guard[:max(R, 1)], alloc_ws(cfg, 2))
    torch.cuda.synchronize()
    assert bool((guard[R] == 7.0).all())                       # nothing past the last row
    err = rel_fro(guard[:R].cpu().numpy(), ref)
    print("rel fro", err, flush=True)
    assert err < 1e-5                                          # float32 sums of at most 1344 terms: about 1e-6
