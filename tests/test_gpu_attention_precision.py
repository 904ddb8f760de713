"""What the fused attention keeps in 32 bits: probabilities that sum to one however large the scores are, and the row dots of its backward."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
from harness import check_bf16_tensor, norm_err
from oracle import hdet_oracle as O
from test_gpu_transformer import TfRun, base

pytestmark = pytest.mark.gpu


def run_with(cfg, batch, set_parameters):
    """A run of two replicas whose parameters, a dict of views by name, `set_parameters` has changed."""
    run = TfRun(base(n_replicas=2, optimizer=O.ADAMW, lr_max=2e-3), cfg, batch, bf16=True)
    flat, off, par = run.orc.theta[0].copy(), 0, {}
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        par[name] = flat[off:off + k].reshape(shape)
        off += k
    set_parameters(par)
    run.orc.theta[:] = flat
    run.theta[:, :run.P] = torch.from_numpy(flat).to(run.theta.device)
    run.shadow[:, :run.P] = run.theta[:, :run.P].to(torch.bfloat16)
    return run


def gradients(cfg, flat):
    out, off = {}, 0
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        out[name] = flat[off:off + k].reshape(shape)
        off += k
    return out


@pytest.mark.parametrize("seq", [64, 192])
@pytest.mark.parametrize("size", [12.0, 100.0, 1000.0])
def test_probabilities_sum_to_one_at_large_scores(seq, size):
    """Every query and key the same vector: scores of 8 size^2, up to 8e6, all equal, so that row i averages its i + 1 values.  There fp32 numbers
    lie one apart, and a rounding of the row's maximum that the normalisation does not take back moves every probability by up to 40 %."""
    d = 64
    cfg = dict(n_blocks=1, d_model=d, n_heads=1, d_ff=64, seq_len=seq, vocab=40)

    def same_queries_and_keys(par):
        par["w_qkv.0"][:2 * d] = 0.0
        par["b_qkv.0"][:2 * d] = size
        par["w_qkv.0"][2 * d:] *= 8.0                      # the values count in the loss
        par["w_o.0"][:] *= 8.0

    run = run_with(cfg, 2, same_queries_and_keys)
    ids, tgt, gl = run.forward_backward(1)
    losses, grads = run.oracle_grads(run.orc.theta, ids, tgt, 1)
    assert np.max(np.abs(gl - losses)) <= 1e-2
    g_dev = run.g.cpu().numpy()[:, :run.P]
    for r in range(2):
        got, want = gradients(cfg, g_dev[r]), gradients(cfg, grads[r])
        for name in want:                                   # (the gradients of the queries and keys are sums that cancel)
            rows = slice(2 * d, None) if name in ("w_qkv.0", "b_qkv.0") else slice(None)
            check_bf16_tensor(got[name][rows], want[name][rows], 4e-2, ("large scores", seq, size, r, name))
    run.close()


@pytest.mark.parametrize("seq", [128, 448, 512])
def test_row_dots_keep_32_bits_of_the_output(seq):
    """All scores zero and all keys one vector: the gradient of the queries is that vector times the sum of ds over the row's keys, which is zero but for
    what p, ds and the row's dot were rounded to.  Values of +-8 and a hundredth of that, in pairs that the output projection sees as one: the dots are
    sums of large terms that cancel, and one from 16 bits of the attention's output makes that gradient several times what the rounding of ds does."""
    d = 64
    cfg = dict(n_blocks=1, d_model=d, n_heads=1, d_ff=64, seq_len=seq, vocab=40)

    def large_values(par):
        par["w_qkv.0"][:2 * d] = 0.0
        par["b_qkv.0"][:d] = 0.0
        par["b_qkv.0"][d:2 * d] = 1.0
        par["b_qkv.0"][2 * d:] = np.where(np.arange(d) % 2 == 0, 8.0, -8.0)
        par["w_qkv.0"][2 * d:] *= 0.1
        par["w_o.0"][:, 1::2] = par["w_o.0"][:, 0::2]

    run = run_with(cfg, 2, large_values)
    ids, tgt, gl = run.forward_backward(1)
    losses, grads = run.oracle_grads(run.orc.theta, ids, tgt, 1)
    assert np.max(np.abs(gl - losses)) <= 1e-2
    g_dev = run.g.cpu().numpy()[:, :run.P]
    for r in range(2):
        got, want = (gradients(cfg, g)["w_qkv.0"][:d] for g in (g_dev[r], grads[r]))
        assert norm_err(got, want) <= 0.3
    run.close()
