"""The output layer with its loss formed inside the product (mixed precision, no label smoothing): every gradient tensor and the
losses against the oracle, at sizes whose last tiles are ragged in rows, columns and contraction."""
import numpy as np
import pytest
import torch

from test_gpu_transformer import TfRun, base, check_bf16_gradients

pytestmark = pytest.mark.gpu

# (replicas, batch, model, replicas compared)
CASES = [
    # 1800 x 1992: eight rows in the last tile, 200 columns; K = 192 is three K steps, the fourth empty
    (6, 36, dict(n_blocks=1, d_model=192, n_heads=3, d_ff=64, seq_len=50, vocab=1992), (0, 5)),
    # wide rows, 8 columns in the last tile, K no multiple of a step
    (4, 52, dict(n_blocks=1, d_model=200, n_heads=4, d_ff=64, seq_len=50, vocab=2056), (1, 3)),
    # more than four rounds of tiles, K of nine steps
    (5, 10, dict(n_blocks=1, d_model=576, n_heads=9, d_ff=64, seq_len=103, vocab=12296), (4,)),
]


@pytest.mark.parametrize("n,batch,cfg,compared", CASES)
def test_loss_and_gradients(n, batch, cfg, compared):
    run = TfRun(base(n_replicas=n), cfg, batch, bf16=True)
    ids, tgt, losses = run.forward_backward(1)
    first = run.g.clone()
    run.g.fill_(7.0)
    run.forward_backward(1)
    assert torch.equal(first, run.g)                       # every sum has a fixed order
    only = np.array(compared)
    run.n = len(only)
    run.orc.dropout_table = lambda: np.zeros(len(only))
    run.orc.label_smoothing_table = lambda: np.zeros(len(only))
    run.orc.attn_temp_table = lambda: np.ones(len(only))
    ref_losses, ref = run.oracle_grads(run.orc.theta[only], ids[only], tgt[only], 1)
    got = run.g.cpu().numpy()
    for i, r in enumerate(compared):
        # a loss is a mean of over a thousand rows whose logits are products of rounded operands (2^-9 of logits of size 1)
        assert abs(losses[r] - ref_losses[i]) <= 1e-3
        check_bf16_gradients(cfg, got[r, :run.P], ref[i], 4e-2, ("head loss", cfg["vocab"], r))
    run.close()


def test_bias_product_of_several_rounds():
    """qkv of 3500 x 1584 over K = 528 in 686 tiles: rows, columns and K end inside the last tiles and steps of blocks that walk over them."""
    cfg, n, batch = dict(n_blocks=1, d_model=528, n_heads=8, d_ff=64, seq_len=70, vocab=96), 7, 50
    run = TfRun(base(n_replicas=n), cfg, batch, bf16=True)
    ids, tgt, losses = run.forward_backward(1)
    r = n - 1
    run.n = 1
    run.orc.dropout_table = lambda: np.zeros(1)
    run.orc.label_smoothing_table = lambda: np.zeros(1)
    run.orc.attn_temp_table = lambda: np.ones(1)
    ref_loss, ref = run.oracle_grads(run.orc.theta[r:], ids[r:], tgt[r:], 1)
    assert abs(losses[r] - ref_loss[0]) <= 1e-3
    check_bf16_gradients(cfg, run.g.cpu().numpy()[r, :run.P], ref[0], 4e-2, ("walk", r))
    run.close()
