"""MLP units far outside the range of ordinary pre-activations (biases used as switches, a replica that diverges): gradients against the
oracle where the derivative of the GELU is 0 or 1, in the products' epilogues and in the element-wise kernel of odd widths."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
from test_gpu_transformer import TfRun, base, norm_err

pytestmark = pytest.mark.gpu

FAR = [-1e13, -1e12, -3.6e10, -1e6, -40.0, -11.0, -9.5, 9.5, 11.0, 40.0, 1e4, 1e8]


@pytest.mark.parametrize("bf16,cfg,batch", [
    (False, dict(n_blocks=1, d_model=64, n_heads=2, d_ff=256, seq_len=32, vocab=50), 4),          # fragments from global memory
    (False, dict(n_blocks=1, d_model=128, n_heads=2, d_ff=1024, seq_len=128, vocab=50), 8),       # through LDS
    (True, dict(n_blocks=1, d_model=24, n_heads=3, d_ff=50, seq_len=70, vocab=50), 2),            # the GELU in kernels of its own
])
def test_gradients_of_far_units(bf16, cfg, batch):
    run = TfRun(base(n_replicas=2), cfg, batch, bf16=bf16)
    flat, off, part = run.orc.theta[0].copy(), 0, {}
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        part[name] = slice(off, off + k)
        off += k
    far = np.array(FAR)
    flat[part["b_1.0"]][:len(far)] = far
    w2 = flat[part["w_2.0"]].reshape(cfg["d_model"], cfg["d_ff"])
    w2[:, :len(far)] /= np.maximum(1.0, far)                         # large outputs are scaled back, the shut units count in full
    run.orc.theta[:] = flat
    run.theta[:, :run.P] = torch.from_numpy(flat).to(run.theta.device)
    if bf16:
        run.shadow[:, :run.P] = run.theta[:, :run.P].to(torch.bfloat16)
    ids, tgt, gl = run.forward_backward(1)
    losses, grads = run.oracle_grads(run.orc.theta, ids, tgt, 1)
    # bounds of the ordinary gradient tests of the two precisions
    assert np.max(np.abs(gl - losses)) <= (5e-3 if bf16 else 1e-5) * np.max(losses)
    got = run.g.cpu().numpy()[:, :run.P]
    assert np.all(np.isfinite(got))
    for r in range(2):
        shut = got[r, part["b_1.0"]][:5]
        assert np.all(shut == 0), shut
        for name in ("b_1.0", "w_1.0", "ln2_g.0", "ln2_b.0", "w_o.0"):
            assert norm_err(got[r, part[name]], grads[r, part[name]]) <= (4e-2 if bf16 else 3e-5), (name, r)
    run.close()
