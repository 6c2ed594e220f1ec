"""The float64 gate: float32 activations, more than 64 experts, and many tokens on more than 16 experts.  Indices equal the
float64 oracle's; weights and probabilities carry the float32 softmax (a few ulp, 1e-6; 1e-5 as in the other gate tests)."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M
from oracle import moe_oracle as O

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


# every expert group of the kernel and its edges, routers read four, two and one weight at a time, one chunk of the
# contraction index and ragged numbers of them over the wavefronts, last workgroups of one to fifteen tokens
CASES = [("f32", 33, 64, 1, 1), ("f32", 100, 128, 16, 8), ("f32", 50, 320, 17, 3), ("f32", 31, 192, 30, 2), ("f32", 47, 64, 33, 5),
         ("f32", 29, 1088, 64, 2), ("f32", 40, 448, 65, 4), ("f32", 17, 128, 128, 2), ("f32", 20, 256, 130, 8), ("f32", 35, 64, 256, 1),
         ("bf16", 1, 64, 66, 2), ("bf16", 30, 1600, 128, 6), ("bf16", 18, 192, 127, 8), ("bf16", 33, 576, 255, 3),
         ("bf16", 45, 2048, 256, 8), ("bf16", 1024, 64, 17, 2), ("bf16", 1039, 320, 32, 2), ("bf16", 1030, 128, 31, 4),
         ("bf16", 1025, 704, 64, 8), ("bf16", 1024, 192, 63, 1)]


@pytest.mark.parametrize("dtype,T,d,E,k", CASES, ids=str)
def test_gate_float64(dtype, T, d, E, k):
    print(dtype, T, d, E, k, flush=True)
    rng = np.random.default_rng(T * E + k)
    x = rng.standard_normal((T, d)).astype(np.float32)
    if dtype == "bf16":
        x = (x.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    w = (rng.standard_normal((d, E)) * d ** -0.5).astype(np.float32)
    b = (0.3 * rng.standard_normal(E)).astype(np.float32)
    if E > 1:  # a pair of experts whose logits differ in the last bits of one weight
        w[:, E - 1] = w[:, 0]
        w[d // 2, E - 1] = np.nextafter(w[d // 2, 0], np.float32(9), dtype=np.float32)
        b[E - 1] = b[0]
    p_ref, idx_ref, w_ref = O.gate(x, w, b, k, True)
    cfg = M.MoEConfig(T=T, d_model=d, d_ff=64, E=E, k=k, renormalize=True, dtype=dtype)
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    tw = torch.empty((T, k), device="cuda")
    p = torch.empty((T, E), device="cuda")
    M.moe_gate(cfg, to_dev(x, dtype), to_dev(w, "f32"), to_dev(b, "f32"), idx, tw, p)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    assert np.allclose(tw.cpu().numpy(), w_ref, rtol=1e-5) and np.allclose(p.cpu().numpy(), p_ref, rtol=1e-5, atol=1e-12)
