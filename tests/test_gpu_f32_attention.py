"""Fused attention of the full-precision path: losses and every gradient tensor against the oracle, at sequences around the 32-row
blocks and the tiles a wavefront holds, every head size it takes, with the temperature channel; and against the unfused path."""
import numpy as np
import pytest

import hdet_inputs as I
import paper_2604_24708_amd as H
from test_gpu_transformer import TfRun, base, norm_err

pytestmark = pytest.mark.gpu


def model(seq, heads, dh):
    return dict(n_blocks=1, d_model=heads * dh, n_heads=heads, d_ff=16, seq_len=seq, vocab=17)


@pytest.mark.parametrize("seq,heads,dh,batch", [(1, 2, 8, 3), (31, 3, 16, 2), (32, 1, 24, 2), (33, 2, 32, 2), (77, 2, 40, 1), (128, 1, 48, 2), (129, 2, 56, 1),
                                                (130, 1, 64, 2), (256, 1, 16, 1), (257, 1, 64, 1), (511, 1, 8, 1), (512, 2, 24, 1)])
@pytest.mark.parametrize("temp", [False, True])
def test_against_oracle_and_unfused_path(seq, heads, dh, batch, temp):
    cfg, n = model(seq, heads, dh), 2
    extra = [(H.HDET_CH_ATTN_TEMP, 1.2, 0.3, 1e-3, 0.1, 4.0)] if temp else []
    run, plain = (TfRun(base(n_replicas=n, extra=extra), cfg, batch) for _ in range(2))
    H.hdet_set_launch_shape(plain.h, 2, 0)
    ids, tgt, gl = run.forward_backward(1)
    _, _, pl = plain.forward_backward(1)
    losses, grads = run.oracle_grads(run.orc.theta, ids, tgt, 1)
    assert np.max(np.abs(gl - losses)) <= 1e-5 * np.max(losses) and np.max(np.abs(gl - pl)) <= 1e-5 * np.max(losses)
    got, other = run.g.cpu().numpy(), plain.g.cpu().numpy()
    for r in range(n):
        off = 0
        for name, shape in I.transformer_shapes(cfg):
            k = int(np.prod(shape))
            part = slice(off, off + k)
            off += k
            if seq == 1 and name in ("w_qkv.0", "b_qkv.0"):     # one key: the gradients of queries and keys are zero
                part = slice(part.start + 2 * k // 3, part.stop)
            elif name.split(".")[0] == "b_qkv":                 # the keys' third is zero but for rounding
                continue
            # a dozen fp32 products in a chain
            assert norm_err(got[r, part], grads[r, part]) <= 3e-5, (name, r)
            assert norm_err(got[r, part], other[r, part]) <= 3e-5, (name, r, "unfused")
    run.close()
    plain.close()
