"""The general LDS kernel with one K step in flight, which grids of many blocks take, entry by entry against 64 bits: tiles of 64 and of 128, rows that
start at odd elements and not, contractions of one step, of whole steps and with a rest, forward products and both gradients."""
import numpy as np
import pytest
import torch

import paper_2604_24708_amd as H
from test_gpu_product_values import disagreements, inputs, reference

pytestmark = pytest.mark.gpu

# 64 x 64: 1320 blocks of the first product and of the gradient through it; 128 x 128: 1152 of both
CASES = [([k, 2052, 12], 260, 8) for k in (6, 31, 64, 130, 250, 516)] + [([36, 1500, 40], 1500, 8), ([37, 1501, 33], 1500, 8), ([130, 1492, 66], 1450, 8)]


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
