"""The alternating 256 x 256 kernel under the epilogues that plain products do not reach, on tiles that the matrix fills in part: the update of a weight
matrix inside its gradient's product against the two separate calls, and the gradient through GELU with its column sums against the oracle."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
import paper_2604_24708_amd as H
from harness import check_bf16_tensor
from oracle import hdet_oracle as O
from oracle import transformer_oracle as T
from test_gpu_mlp import MlpRun, cfg0
from test_gpu_train_step import assert_same_bits
from test_gpu_transformer import TfRun, base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [904, 1000])
def test_update_inside_the_product_equals_two_calls_bit_for_bit(batch):
    """2032 x 2040 weights, four replicas: 256 tiles, the last row and column of them ragged; 15 and 16 K steps of 64, the last one cut short."""
    widths, n = [2040, 2032, 40], 4
    d = cfg0(n_replicas=n, optimizer=O.ADAMW, lr_max=2e-3, total_steps=12, warm_steps=4, weight_decay=0.01)
    two, one = MlpRun(d, widths, batch, bf16=True), MlpRun(d, widths, batch, bf16=True)
    for t in (1, 2):
        x, y = I.mlp_batch(n, batch, widths[0], I.SEED_DATA, t, widths, I.SEED_TEACHER)
        xd, yd = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
        H.hdet_forward_backward(two.h, xd, yd)
        H.hdet_fanout_step(two.h, None, 0)
        one.g.fill_(7.0)
        H.hdet_train_step(one.h, xd, yd, 0)
        assert torch.all(one.g[:, :widths[0] * widths[1]] == 7.0)            # no gradient was written: the product carried the update
        assert_same_bits(two, one, t)
    two.close(); one.close()


def test_gradient_through_gelu_and_its_column_sums():
    """d = 2048: the contraction from which the gradient of the inner layer takes the kernel; 1000 tokens x 2040 inner units, eight replicas."""
    cfg, batch, n = dict(n_blocks=1, d_model=2048, n_heads=32, d_ff=2040, seq_len=100, vocab=64), 10, 8
    run = TfRun(base(n_replicas=n, optimizer=O.ADAMW, lr_max=2e-3), cfg, batch, bf16=True)
    ids, tgt, gl = run.forward_backward(1)
    r = n - 1
    loss, want = T.loss_and_grad(run.orc.theta[r], ids[r], tgt[r], cfg, bf16=True)
    assert abs(gl[r] - loss) <= 1e-2
    got, off = run.g[r, :run.P].cpu().numpy(), 0
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        if name in ("w_1.0", "b_1.0", "ln2_g.0", "ln2_b.0"):                 # what is formed from that product
            check_bf16_tensor(got[off:off + k], want[off:off + k], 4e-2, ("d2048", name))
        off += k
    run.close()
