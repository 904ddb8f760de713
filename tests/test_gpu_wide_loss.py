"""The loss kernel for wide rows at widths around its steps (how many chunks a thread owns, which of them are masked): gradients
of a one-layer classifier against autograd in 64 bits, and the head bias gradient it forms beside a transformer's loss (from 8192
rows on) against the separate reduction that the same replica takes alone."""
import numpy as np
import pytest
import torch

from test_gpu_products import mlp_grads

import hdet_inputs as I
import paper_2604_24708_amd as H

pytestmark = pytest.mark.gpu

WIDTHS = [2048, 2052, 4096, 4100, 6148, 8192, 8196, 16384, 16388, 24580, 28672, 28676, 32768]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("classes", WIDTHS)
def test_classifier_gradients(classes, bf16):
    got, ref, slices = mlp_grads([16, classes], 5, 2, bf16=bf16)
    for s in slices:
        # fp32: a softmax over up to 32768 entries, summed in some order (2^-24 sqrt(32768) = 1.1e-5); bf16: logits of rounded
        # operands (2^-9, sixteen of them) move the output gradient by as much, which is rounded once more
        assert np.linalg.norm(got[:, s] - ref[:, s]) <= (1e-2 if bf16 else 1.2e-5) * np.linalg.norm(ref[:, s])


def _tf_grads(n, vocab, seed=4):
    d = dict(n_blocks=1, d_model=64, n_heads=1, d_ff=64, seq_len=64, vocab=vocab)
    batch, dev = 64, "cuda:0"
    P = I.transformer_param_count(d)
    stride = (P + 3) // 4 * 4
    g = torch.Generator(device=dev).manual_seed(seed)
    one = torch.randn(stride, device=dev, generator=g) * 0.1
    x = torch.randint(0, vocab, (1, batch, 64), generator=g, device=dev, dtype=torch.int32).repeat(n, 1, 1)
    y = torch.randint(0, vocab, (1, batch, 64), generator=g, device=dev, dtype=torch.int32).repeat(n, 1, 1)
    theta = one.repeat(n, 1)
    m, v, grads = torch.zeros_like(theta), torch.zeros_like(theta), torch.full_like(theta, 7.0)
    shadow = torch.zeros((n, stride), dtype=torch.bfloat16, device=dev)
    cfg = H.make_config(n_replicas=n, sync_interval=4, total_steps=8, warm_steps=0, lr_max=1e-3, alpha=0.1, model_kind=H.HDET_TRANSFORMER,
                        batch=batch, precision=H.HDET_BF16_GEMM_FP32_MASTER, **d)
    ws = torch.zeros(max(H.hdet_workspace_bytes(cfg, stride)[2], 16), dtype=torch.uint8, device=dev)
    h = H.hdet_create(cfg, theta, m, v, grads=grads, params_bf16=shadow, workspace=ws, plane_stride=stride)
    H.hdet_forward_backward(h, x, y)
    torch.cuda.synchronize()
    H.hdet_destroy(h)
    return grads[:, :P]


@pytest.mark.parametrize("vocab", [2048, 2056, 4104, 6152, 8200, 16392, 24584, 28680])
def test_head_bias_gradient_beside_the_loss(vocab):
    alone, both = _tf_grads(1, vocab)[0].double(), _tf_grads(2, vocab).double()
    assert torch.equal(both[0], both[1])
    a, b = alone[-vocab:], both[0, -vocab:]
    # sums of 4096 stored bf16 terms in two fp32 orders: sqrt(4096) 2^-24 of their size each, the terms nearly cancelling by half
    assert float((a - b).norm()) <= 2e-5 * float(a.norm())
    assert float(a.norm()) > 0.0 and abs(float(b.sum())) <= 1e-2 * float(b.abs().sum())
