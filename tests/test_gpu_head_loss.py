"""The output layer with its loss formed inside the product (mixed precision, no label smoothing): every gradient tensor and the
losses against the oracle, at sizes whose last tiles are ragged in rows, columns and contraction."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
import paper_2604_24708_amd as H
from oracle import hdet_oracle as O
from test_gpu_transformer import TfRun, base, check_bf16_gradients, norm_err

pytestmark = pytest.mark.gpu

# (replicas, batch, model, replicas compared)
CASES = [
    # 1800 x 1992: eight rows in the last tile, 200 columns; K = 192 is three K steps, the fourth empty
    (7, 36, dict(n_blocks=1, d_model=192, n_heads=3, d_ff=64, seq_len=50, vocab=1992), (0, 6)),
    # wide rows, 8 columns in the last tile, K no multiple of a step
    (4, 52, dict(n_blocks=1, d_model=200, n_heads=4, d_ff=64, seq_len=50, vocab=2056), (1, 3)),
    # more than four rounds of tiles, K of nine steps
    (5, 10, dict(n_blocks=1, d_model=576, n_heads=9, d_ff=64, seq_len=103, vocab=12296), (4,)),
]


def slices(cfg):
    """Where the tensors lie in a plane, and their shapes."""
    out, off = {}, 0
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        out[name] = slice(off, off + k), shape
        off += k
    return out


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


@pytest.mark.parametrize("size", [1.0, 30.0, 300.0])
@pytest.mark.parametrize("n,batch,cfg", [c[:3] for c in CASES])
def test_loss_of_known_logits(n, batch, cfg, size):
    """A head of no weights: every row's logits are the head's biases, known to the last bit, and so are the loss and the bias gradient in 64 bits.
    Classes next to the row's maximum lie in all column tiles, a hundred others are masked by -inf, one tile's whole 256 among them (a loss kernel that reads
    the logits from memory has no finite loss there: these sizes do take the path)."""
    run = TfRun(base(n_replicas=n), cfg, batch, bf16=True)
    V, M = cfg["vocab"], batch * cfg["seq_len"]
    part = slices(cfg)
    ids, tgt = I.zipf_tokens(n, batch, cfg["seq_len"], V, I.SEED_DATA, 1)
    rng = np.random.Generator(np.random.Philox(11))
    flat = run.orc.theta.copy()
    z = np.zeros((n, V))
    for r in range(n):
        b = (size * rng.standard_normal(V)).astype(np.float32)
        top = rng.permutation(V)[:40]
        b[top] = b.max() - rng.uniform(0, 3, 40).astype(np.float32)
        b[1024:1280] = -np.inf
        b[rng.permutation(V)[:100]] = -np.inf
        seen = np.unique(tgt[r])
        b[seen] = np.where(np.isfinite(b[seen]), b[seen], np.float32(0))
        flat[r, part["w_head"][0]], flat[r, part["b_head"][0]], z[r] = 0.0, b, b
    run.theta[:, :run.P] = torch.from_numpy(flat).to(run.theta.device)
    run.shadow[:, :run.P] = run.theta[:, :run.P].to(torch.bfloat16)
    _, _, losses = run.forward_backward(1)
    got = run.g.cpu().numpy()[:, part["b_head"][0]]
    for r in range(n):
        e = np.exp(z[r] - z[r].max())
        lse = z[r].max() + np.log(e.sum())
        # a row's loss is rounded once, from sums that are off by a few 1e-7; the logits enter through a log2(e) rounded to 2^-26
        want = lse - z[r][tgt[r].reshape(-1)].mean()
        assert abs(losses[r] - want) <= 4e-7 * abs(want) + 3e-7
        p = e / e.sum()
        hits = np.bincount(tgt[r].reshape(-1), minlength=V)
        # M equal terms, each with one rounding of its exponent (2^-24 of at most 8 where a probability counts), summed in fp32 in parts of 128
        free = hits == 0
        assert norm_err(got[r][free], p[free]) <= 8e-7
        assert np.max(np.abs(got[r] - (p - hits / M))) <= 2e-6
    run.close()


def test_label_that_is_no_class():
    """-1 in the label's place (rows that a caller pads): the row's loss is log sum exp of its logits, whatever the call before left there."""
    n, batch, cfg = CASES[1][:3]
    run = TfRun(base(n_replicas=n), cfg, batch, bf16=True)
    part = slices(cfg)
    ids, tgt = I.zipf_tokens(n, batch, cfg["seq_len"], cfg["vocab"], I.SEED_DATA, 1)
    b = np.random.Generator(np.random.Philox(12)).standard_normal(cfg["vocab"]).astype(np.float32)
    flat = run.orc.theta[0].copy()
    flat[part["w_head"][0]], flat[part["b_head"][0]] = 0.0, b
    run.theta[:, :run.P] = torch.from_numpy(flat).to(run.theta.device)
    run.shadow[:, :run.P] = run.theta[:, :run.P].to(torch.bfloat16)
    run.forward_backward(1)
    tgt[:, 1::3, ::5] = -1
    out = H.hdet_forward_backward(run.h, torch.from_numpy(ids).to("cuda:0"), torch.from_numpy(tgt).to("cuda:0"), want_losses=True)
    for r in range(n):
        want = np.log(np.exp(b.astype(np.float64)).sum()) - np.where(tgt[r] >= 0, b[tgt[r]], 0.0).mean()
        assert abs(out[r] - want) <= 4e-7 * abs(want) + 3e-7
    run.close()


def test_one_call_equals_two_calls():
    n, batch, cfg = CASES[1][:3]
    two, one = (TfRun(base(n_replicas=n, optimizer=O.ADAMW, lr_max=2e-3), cfg, batch, bf16=True) for _ in range(2))
    for t in (1, 2):
        ids, tgt, losses = two.forward_backward(t)
        H.hdet_fanout_step(two.h, None, 0)
        got = H.hdet_train_step(one.h, torch.from_numpy(ids).to("cuda:0"), torch.from_numpy(tgt).to("cuda:0"), 0, want_losses=True)
        assert [got[r] for r in range(n)] == losses.tolist()
        for a, b in ((one.theta, two.theta), (one.m, two.m), (one.v, two.v)):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), t
    one.close()
    two.close()


def test_shared_gradients():
    """One weight gradient over all replicas' rows, from the same gradients of the logits; losses and head bias gradients stay per replica, bit for bit."""
    n, batch, cfg = CASES[2][:3]
    shared, own = (TfRun(base(n_replicas=n, optimizer=O.ADAMW, grad_mode=m), cfg, batch, bf16=True) for m in (O.GRAD_SHARED, O.GRAD_PER_REPLICA))
    _, _, ls = shared.forward_backward(1)
    _, _, lo = own.forward_backward(1)
    assert np.array_equal(ls, lo)
    part = slices(cfg)
    assert torch.equal(shared.g[:, part["b_head"][0]], own.g[:, part["b_head"][0]])
    a, b = shared.g[0, part["w_head"][0]].double(), own.g[:, part["w_head"][0]].double().sum(0)
    # 5150 rows in another order: 2^-24 sqrt(5150) = 4e-6
    assert float((a - b).norm() / b.norm()) <= 2e-5
    shared.close()
    own.close()


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
