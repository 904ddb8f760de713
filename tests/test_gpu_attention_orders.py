"""The fused attention kernels where their walks and block orders have edges, against the path through separate products.

Sequences of one tile, of an odd number of tiles (the last block has two idle wavefronts) and of many; heads over all replicas that are a
multiple of the chip's eight dies, and not; few blocks (longest rows first) and more than eight a CU (all rows of a head together)."""
import numpy as np
import pytest

import paper_2604_24708_amd as H
from oracle import hdet_oracle as O
from test_gpu_transformer import TfRun, base, per_tensor_errors

pytestmark = pytest.mark.gpu


def cfg(heads, seq):
    return dict(n_blocks=1, d_model=64 * heads, n_heads=heads, d_ff=64, seq_len=seq, vocab=64)


@pytest.mark.parametrize("heads,seq,batch,n", [(1, 64, 1, 1), (1, 128, 3, 3), (3, 320, 1, 3), (2, 448, 2, 2), (1, 1984, 1, 2), (4, 192, 130, 4)])
def test_fused_attention_matches_separate_products(heads, seq, batch, n):
    c = cfg(heads, seq)
    fused, plain = (TfRun(base(n_replicas=n, optimizer=O.ADAMW, lr_max=2e-3), c, batch, bf16=True) for _ in range(2))
    H.hdet_set_launch_shape(plain.h, 2, 0)                # separate kernels, scores in device memory
    _, _, lf = fused.forward_backward(1)
    _, _, lp = plain.forward_backward(1)
    # both round p, ds and every stored tensor to bf16 at the same points; sums in another order flip a few of them
    assert np.max(np.abs(lf - lp)) <= 5e-4
    gf, gp = fused.g.cpu().numpy()[:, :fused.P], plain.g.cpu().numpy()[:, :fused.P]
    for r in range(n):
        bad = {k: v for k, v in per_tensor_errors(c, gf[r], gp[r]).items() if v > 5e-3}
        assert not bad, (heads, seq, batch, r, bad)
    fused.close(); plain.close()
