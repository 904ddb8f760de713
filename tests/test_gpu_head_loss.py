"""The output layer with its loss formed inside the product (mixed precision, no label smoothing): every gradient tensor and the
losses against the oracle, at sizes whose last tiles are ragged in rows, columns and contraction."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
from test_gpu_transformer import TfRun, base, check_bf16_gradients, norm_err

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


def slices(cfg):
    """Where the tensors lie in a plane, and their shapes."""
    out, off = {}, 0
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        out[name] = slice(off, off + k), shape
        off += k
    return out


def test_bias_is_added_to_the_finished_sum():
    """Values 1 + (16 terms of 0.375 or 0.25 units in the last place of 1) - 1, each term in another step of the contraction: 6 and 4 such units when
    the bias comes last, nothing when the terms are added to it one by one.  The gradient of the output projection is proportional to them."""
    d = 528
    cfg, n, batch = dict(n_blocks=1, d_model=d, n_heads=8, d_ff=64, seq_len=70, vocab=96), 7, 50
    run = TfRun(base(n_replicas=n), cfg, batch, bf16=True)
    flat, part = run.orc.theta[0].copy(), slices(cfg)
    par = {k: flat[at].reshape(shape) for k, (at, shape) in part.items()}
    par["ln1_g.0"][:], par["ln1_b.0"][:] = 0.0, 1.0                  # every operand of the product is one
    par["w_qkv.0"][2 * d:], par["b_qkv.0"][2 * d:] = 0.0, 1.0
    for c in range(d):
        par["w_qkv.0"][2 * d + c, 0:512:32] = (0.375 if c % 2 else 0.25) * 2.0 ** -23
    par["w_qkv.0"][2 * d:, 527] = -1.0
    run.orc.theta[:] = flat
    run.theta[:, :run.P] = torch.from_numpy(flat).to(run.theta.device)
    run.shadow[:, :run.P] = run.theta[:, :run.P].to(torch.bfloat16)
    ids, tgt, _ = run.forward_backward(1)
    r = n - 1
    run.n = 1
    run.orc.dropout_table = lambda: np.zeros(1)
    run.orc.label_smoothing_table = lambda: np.zeros(1)
    run.orc.attn_temp_table = lambda: np.ones(1)
    _, ref = run.oracle_grads(run.orc.theta[r:], ids[r:], tgt[r:], 1)
    w_o = part["w_o.0"][0]
    assert norm_err(run.g.cpu().numpy()[r, w_o], ref[0][w_o]) <= 4e-2          # the bound of these models' tensors
    run.close()
