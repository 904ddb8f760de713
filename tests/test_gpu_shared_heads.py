"""Full precision with the shared gradient where a weight matrix is large enough that its gradient is one product over all
replicas' rows: its bias gradient, which stays per replica, comes from the loss kernel (wide rows), from the LayerNorm kernel
or from column sums in one or two stages.  Against the oracle."""
import numpy as np
import pytest

import hdet_inputs as I
import paper_2604_24708_amd as H
from oracle import hdet_oracle as O
from oracle import transformer_oracle as T
from test_gpu_transformer import TfRun, base, norm_err

pytestmark = pytest.mark.gpu

# (replicas, batch, model): from 32513 outputs of up to 256 inputs on a head is one product.  A vocabulary in the loss kernel's
# range with and without enough rows for its sums, one beyond it, one that is no multiple of 8; and the MLP of a wide block
CASES = [(32, 8, dict(n_blocks=1, d_model=8, n_heads=1, d_ff=16, seq_len=33, vocab=32520)),
         (3, 2, dict(n_blocks=1, d_model=8, n_heads=1, d_ff=16, seq_len=21, vocab=32520)),
         (2, 2, dict(n_blocks=1, d_model=16, n_heads=2, d_ff=16, seq_len=150, vocab=33000)),
         (2, 64, dict(n_blocks=1, d_model=512, n_heads=1, d_ff=16, seq_len=65, vocab=16392)),
         (2, 1, dict(n_blocks=1, d_model=12, n_heads=1, d_ff=16, seq_len=37, vocab=32515)),
         (2, 2, dict(n_blocks=2, d_model=1024, n_heads=4, d_ff=8192, seq_len=35, vocab=19))]


@pytest.mark.parametrize("n,batch,cfg,drop", [(*c, False) for c in CASES] + [(*CASES[-1], True)])
def test_bias_gradients_of_one_product_matrices(n, batch, cfg, drop):
    """drop: with a dropout channel, the bias gradients of the branches below are those of the dropped-out gradient."""
    extra = [(H.HDET_CH_DROPOUT, 0.2, 0.5, 1e-3, 0.0, 0.5)] if drop else []
    run = TfRun(base(n_replicas=n, grad_mode=O.GRAD_SHARED, extra=extra), cfg, batch)
    run.forward_backward(1)
    ids, tgt, losses = run.forward_backward(2)
    got = run.g.double().cpu().numpy()
    p = run.orc.dropout_table()
    summed = {}
    for r in range(n) if n <= 3 else (0, n - 1):
        dropout = dict(p=float(p[r]), seed=run.d["seed"], step=1, replica=r) if drop else None
        loss, ref = T.loss_and_grad(run.orc.theta[r], ids[r], tgt[r], cfg, dropout=dropout)
        assert abs(losses[r] - loss) <= 1e-5 * loss
        off = 0
        for name, shape in I.transformer_shapes(cfg):
            k = int(np.prod(shape))
            b = ref[off:off + k].astype(np.float64)
            base_name, rows, cols = name.split(".")[0], shape[0], shape[-1]
            if base_name[:2] == "w_" and -(-rows // 256) * -(-cols // 256) >= 128:
                summed.setdefault(name, [off, 0.0])[1] += b
            elif base_name != "b_qkv":                # its middle third is zero but for rounding
                a = got[r, off:off + k]
                # a dozen fp32 products in a chain, reductions of up to 8192 terms; a row of 30 to 300 left out of a sum is 6 % or more
                assert norm_err(a, b) <= 3e-5, (name, r)
                assert np.max(np.abs(a - b)) <= 1e-3 * np.sqrt(np.mean(b * b)), (name, r)
            off += k
    assert summed
    if n <= 3:
        for name, (off, total) in summed.items():
            assert norm_err(got[0, off:off + total.size], total) <= 3e-5, name
    run.close()
