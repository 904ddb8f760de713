"""fp32 products that go through LDS (from about one 64 x 32 tile a CU on, operands of whole 16-byte chunks): tiles, contractions and
batches with remainders, weight, bias and input gradients alone and in one launch, against autograd and the oracle in 64 bits."""
import numpy as np
import pytest

import hdet_inputs as I
import paper_2604_24708_amd as H
from test_gpu_products import mlp_grads
from test_gpu_transformer import TfRun, base, norm_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("widths,batch,n", [
    ([132, 516, 260], 132, 8),          # 64 x 64 and 64 x 32 tiles, four rows, columns and k over
    ([36, 1028, 324, 4], 196, 6),       # K of 4 and of 36, a product of four columns
    ([64, 2048, 96], 64, 4),            # whole tiles
    ([260, 1032, 7], 100, 5),           # one operand of odd rows beside whole ones
    ([64, 1024, 68], 256, 4),           # a product of few tiles beside a large one: K of 256, which the large one hides
    ([48, 68, 8004], 252, 4),           # K of 8004, which it does not: in a launch of its own
])
def test_mlp_gradients(widths, batch, n, shared):
    got, ref, slices = mlp_grads(widths, batch, n, shared=shared)
    for s in slices:
        # chains of up to 2048 / 4 fp32 additions (2^-24 sqrt(512) = 1.3e-6), through up to three layers
        assert np.linalg.norm(got[:, s] - ref[:, s]) <= 1e-5 * np.linalg.norm(ref[:, s])
        assert np.max(np.abs(got[:, s] - ref[:, s])) <= 2e-4 * np.sqrt(np.mean(ref[:, s] ** 2))


@pytest.mark.parametrize("cfg,batch,n", [
    (dict(n_blocks=1, d_model=128, n_heads=2, d_ff=512, seq_len=132, vocab=516), 6, 3),        # attention's products in pairs, GELU, residual
    (dict(n_blocks=1, d_model=144, n_heads=4, d_ff=580, seq_len=68, vocab=1100), 8, 4),        # heads of 36, nothing a multiple of 32
])
def test_transformer_gradients(cfg, batch, n):
    run = TfRun(base(n_replicas=n), cfg, batch)
    H.hdet_set_launch_shape(run.h, 2, 0)               # attention as products, a batch item a head, also where one kernel would form it
    ids, tgt, gl = run.forward_backward(1)
    losses, grads = run.oracle_grads(run.orc.theta, ids, tgt, 1)
    assert np.max(np.abs(gl - losses)) <= 1e-5 * np.max(losses)
    got = run.g.cpu().numpy()
    for r in range(n):
        off = 0
        for name, shape in I.transformer_shapes(cfg):
            k = int(np.prod(shape))
            if name.split(".")[0] != "b_qkv":          # its middle third is zero but for rounding
                # a dozen fp32 products in a chain
                assert norm_err(got[r, off:off + k], grads[r, off:off + k]) <= 3e-5, (name, r)
            off += k
    run.close()
