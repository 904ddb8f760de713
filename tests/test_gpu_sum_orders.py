"""Which terms of a long contraction are added to which.  A product of few tiles sums its contraction in quarters, one of less than a 64 x 64 tile a
compute unit whose rows are no whole 16-byte chunks from K = 1024 on in eighths, every other in one piece, whatever kernel forms it: in a ReLU network
another order moves stored activations to their neighbours and units across zero.  Two pairs of huge terms that cancel swallow the small terms
between them unless a piece ends there."""
import numpy as np
import pytest
import torch

import paper_2604_24708_amd as H

# sums of the steps of 16 terms; the pairs straddle the end of the first eighth and of the second quarter
STEPS = {0: 128.0, 4: 2.0 ** 30, 8: 32.0, 10: 32.0, 12: -2.0 ** 30, 28: 2.0 ** 29, 32: 16.0, 34: 16.0, 36: -2.0 ** 29}


def expected(k, pieces):
    n = k // 16
    per, total = -(-n // pieces), np.float32(0.0)
    for p in range(pieces):
        part = np.float32(0.0)
        for i in range(p * per, min((p + 1) * per, n)):
            part = np.float32(part + np.float32(STEPS.get(i, 0.0)))
        total = np.float32(total + part)
    return float(total)


def test_the_orders_differ():
    assert [expected(1024, p) for p in (1, 4, 8)] == [128.0, 160.0, 224.0]


@pytest.mark.gpu
@pytest.mark.parametrize("k,classes,batch,n,pieces", [
    (1024, 10, 7, 2, 4), (1027, 100, 65, 2, 4), (1030, 500, 64, 8, 4), (1024, 640, 130, 3, 4),        # few tiles
    (1027, 1000, 66, 4, 8), (1030, 1000, 128, 7, 8), (1039, 2000, 33, 4, 8),                            # rows of no whole chunks
    (1027, 1000, 130, 6, 1), (1019, 1000, 66, 4, 1),                                                    # ... more tiles, a shorter contraction
    (1024, 1000, 66, 4, 1), (1032, 2048, 128, 8, 1), (1024, 4096, 256, 4, 1)])                          # whole chunks
def test_order_of_the_sums(k, classes, batch, n, pieces):
    """Weights 2 for class 1, 0 for the others and label 0: the loss is the product's entry."""
    P, dev = classes * k + classes, "cuda:0"
    stride = (P + 3) // 4 * 4
    td, g, m, v = (torch.zeros((n, stride), device=dev) for _ in range(4))
    td[:, k:2 * k] = 2.0
    x = torch.zeros((n, batch, k))
    for i, s in STEPS.items():
        if abs(s) > 1e6:
            x[..., 16 * i + 5] = s / 2
        else:
            x[..., 16 * i:16 * i + 16] = s / 32
    cfg = H.make_config(n_replicas=n, sync_interval=4, total_steps=10, lr_max=1e-3, alpha=0.1, widths=[k, classes], batch=batch,
                        model_kind=H.HDET_MLP, optimizer=H.HDET_ADAMW, precision=H.HDET_BF16_GEMM_FP32_MASTER)
    ws = torch.empty(max(H.hdet_workspace_bytes(cfg, stride)[2], 16), dtype=torch.uint8, device=dev)
    copy = torch.zeros((n, stride), dtype=torch.bfloat16, device=dev)
    h = H.hdet_create(cfg, td, m, v, grads=g, params_bf16=copy, workspace=ws, plane_stride=stride)
    losses = H.hdet_forward_backward(h, x.to(dev), torch.zeros((n, batch), dtype=torch.int32, device=dev), want_losses=True)
    H.hdet_destroy(h)
    assert [losses[r] for r in range(n)] == [expected(k, pieces)] * n
