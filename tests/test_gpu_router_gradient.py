"""The router's weight gradient at the edges of its kernel: expert counts on both sides of the 16- and 32-expert blocks and no
multiples of four, token counts on both sides of the 64-token slices and the 16-token shares of a wavefront, several column
blocks.  Nothing flows back from the output (d_out = 0), so the gradient is the auxiliary loss's alone and is known to float32
accuracy: the logits' gradients and the sums over the tokens carry float32 rounding, 1e-4 as for the auxiliary loss."""
import numpy as np
import pytest
import torch

import paper_2205_10034_amd as M
from oracle import moe_backward_oracle as B
from workloads import WORKLOADS, make_layer

from gpu_util import alloc_ws, rel_fro, to_dev, to_np, upload_weights
from test_gpu_backward import expert_grad_buffers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k", [(130, 256, 17, 2), (65, 512, 30, 2), (64, 256, 31, 1), (63, 256, 32, 3), (129, 256, 33, 2), (200, 256, 16, 2),
                                     (17, 768, 15, 1), (1, 256, 5, 1), (15, 256, 2, 1), (77, 256, 47, 2), (81, 256, 129, 2), (50, 256, 255, 1)])
def test_router_gradient(T, d, E, k):
    wl = WORKLOADS["gpt"].scaled(T=T, E=E, k=k, d_model=d, d_ff=256, capacity_factor=0.0)
    print(f"router gradient case {wl}", flush=True)
    L = make_layer(wl, with_bias=True)
    cfg, W, x = M.MoEConfig.from_workload(wl), upload_weights(L, wl.dtype), to_dev(L["x"], wl.dtype)
    ws_f = alloc_ws(cfg)
    M.moe_layer_forward(cfg, W, x, None, torch.empty_like(x), ws_f)
    ref = B.layer_backward(L["x"], L, np.zeros(L["x"].shape), E=E, k=k, capacity_factor=0.0, renormalize=wl.renormalize, act=wl.act, aux_coef=3.0)
    nan = lambda *shape: torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    d_wr, d_br, d_x = nan(d, E), nan(E), torch.full_like(x, float("nan"))
    ws_b = torch.full((M.moe_layer_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda")   # (NaNs wherever something is read unwritten)
    w1_im, w2_im, d_w1, d_b1, d_w2, d_b2 = expert_grad_buffers(wl, L)
    M.moe_layer_backward(cfg, W, w1_im, w2_im, x, torch.zeros_like(x), None, ws_f, d_x, d_wr, d_br, d_w1, d_b1, d_w2, d_b2, ws_b, aux_loss_coef=3.0)
    torch.cuda.synchronize()
    errs = rel_fro(d_wr.cpu().numpy(), ref["w_router"]), rel_fro(d_br.cpu().numpy(), ref["b_router"])
    print(errs, flush=True)
    assert np.abs(ref["w_router"]).max() > 0 and max(errs) < 1e-4
    assert rel_fro(to_np(d_x), ref["x"]) < 1e-2
