"""The LayerNorm backward at every width class of its kernel (lanes to a row, rows side by side, one or two chunks a lane) on both
sides of the line where few blocks take more wavefronts, against the oracle: input gradient, gain and offset gradients and, in
mixed precision, the bias gradient of the branch below that comes with them."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
from oracle import transformer_oracle as T
from test_gpu_transformer import TfRun, base, check_bf16_gradients, norm_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("blocks", ["few", "many"])
@pytest.mark.parametrize("d", [8, 56, 64, 72, 128, 136, 200, 256, 264, 392, 512, 520, 776, 1024])
def test_gradients_at_every_width(d, blocks, bf16):
    # 32 rows to a block: 75 rows end inside a block and inside a wavefront's rows; 64 replicas of 267 make 576 blocks, more than two a
    # compute unit
    n, S, B = (2, 25, 3) if blocks == "few" else (64, 89, 3)
    assert (n * -(-S * B // 32) > 2 * torch.cuda.get_device_properties(0).multi_processor_count) == (blocks == "many")
    cfg = dict(n_blocks=1, d_model=d, n_heads=1, d_ff=16, seq_len=S, vocab=11)
    run = TfRun(base(n_replicas=n), cfg, B, bf16=bf16)
    ids, tgt, losses = run.forward_backward(1)
    got = run.g.double().cpu().numpy()
    for r in {0, n - 1}:
        loss, ref = T.loss_and_grad(run.orc.theta[r], ids[r], tgt[r], cfg, bf16=bf16)
        assert abs(losses[r] - loss) <= (2e-3 if bf16 else 1e-5) * loss
        if bf16:
            check_bf16_gradients(cfg, got[r], ref, 3e-2, ("ln", d, blocks, r))
            continue
        off = 0
        for name, shape in I.transformer_shapes(cfg):
            k = int(np.prod(shape))
            a, b = got[r, off:off + k], ref[off:off + k].astype(np.float64)
            off += k
            if name == "b_qkv.0":                   # the gradient of the keys' bias is zero but for rounding
                a, b = np.delete(a, slice(d, 2 * d)), np.delete(b, slice(d, 2 * d))
            # a chain of a dozen fp32 products and reductions of up to 1024 terms; one row of 75 or 267 left out of a sum is 6 %
            assert norm_err(a, b) <= 2e-5, name
            assert np.max(np.abs(a - b)) <= 2e-4 * np.sqrt(np.mean(b * b)), name
    run.close()
