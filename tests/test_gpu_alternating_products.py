"""Products that the alternating 256 x 256 kernel takes, at its edges -- rows, columns and contractions that end inside a tile, odd and even
numbers of K steps, each operand order, plain, gated and fp32 results -- entry by entry against 64 bits."""
import pytest

from test_gpu_product_values import disagreements, inputs, reference

import numpy as np
import torch

import paper_2604_24708_amd as H

# (widths, batch, replicas): logits 1500 x 2056 over K = 520 and their weight gradient over K = 1500, 432 and 216 tiles;
# ReLU outputs 2000 x 2040 over K = 520 and the gradient through them over K = 1000, 256 tiles each;
# logits 3000 x 2056 over K = 392, 864 tiles
CASES = [([520, 2056], 1500, 8), ([520, 2040, 1000], 2000, 4), ([392, 2056], 3000, 8)]


@pytest.mark.gpu
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
