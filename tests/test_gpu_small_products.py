"""Products of few tiles entry by entry against 64 bits: contractions of one to seven steps of 32 in the general LDS kernel (four in flight; none, some
and all of them whole), rows that start at odd elements and not, and aligned products on both sides of K = 512."""
import numpy as np
import pytest
import torch

import paper_2604_24708_amd as H
from test_gpu_product_values import disagreements, inputs, reference

pytestmark = pytest.mark.gpu

# 120 tiles of 64 x 64 and more: beyond the fragment kernel.  Widths 300 and 301: whole dwords, odd elements.
CASES = [([k, 300, 301], 130, 8) for k in (5, 32, 33, 64, 129, 160, 161, 200)] + [([504, 520, 512], 200, 6), ([1032, 264, 1032], 136, 5)]


@pytest.mark.parametrize("widths,batch,n", CASES)
def test_loss_and_gradients_entry_by_entry(widths, batch, n):
    theta, x, y = inputs(widths, batch, n)
    P = theta.shape[1]
    stride, dev = (P + 3) // 4 * 4, "cuda:0"
    td, g, m, v = (torch.full((n, stride), 7.0, device=dev) for _ in range(4))
    td[:, :P] = torch.from_numpy(theta)
    cfg = H.make_config(n_replicas=n, sync_interval=4, total_steps=10, lr_max=1e-3, alpha=0.1, widths=widths, batch=batch,
                        model_kind=H.HDET_MLP, optimizer=H.HDET_ADAMW, precision=H.HDET_BF16_GEMM_FP32_MASTER)
    ws = torch.empty(max(H.hdet_workspace_bytes(cfg, stride)[2], 16), dtype=torch.uint8, device=dev)
    copy = torch.zeros((n, stride), dtype=torch.bfloat16, device=dev)
    h = H.hdet_create(cfg, td, m, v, grads=g, params_bf16=copy, workspace=ws, plane_stride=stride)
    losses = H.hdet_forward_backward(h, torch.from_numpy(x).to(dev), torch.from_numpy(y).to(dev), want_losses=True)
    got = g[:, :P].double().cpu().numpy()
    H.hdet_destroy(h)
    for r in (0, n - 1):
        assert disagreements(losses[r], got[r], reference(theta[r], x[r], y[r], widths)) == []
    assert np.isfinite(got).all()
