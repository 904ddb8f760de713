"""Fused attention of the full-precision path: losses and every gradient tensor against the oracle, at sequences around the 32-row
blocks and the tiles a wavefront holds, every head size it takes, with the temperature channel; and against the unfused path."""
import numpy as np
import pytest
import torch

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
                parts = [part]
            elif name.split(".")[0] == "b_qkv":                 # the keys' third is zero but for rounding
                parts = [slice(part.start, part.start + k // 3), slice(part.start + 2 * k // 3, part.stop)]
            else:
                parts = [part]
            for part in parts:
                # a dozen fp32 products in a chain
                assert norm_err(got[r, part], grads[r, part]) <= 3e-5, (name, r)
                assert norm_err(got[r, part], other[r, part]) <= 3e-5, (name, r, "unfused")
    run.close()
    plain.close()


@pytest.mark.parametrize("seq,heads,dh,batch", [(32, 4, 16, 4), (64, 2, 32, 2), (128, 4, 64, 2), (192, 2, 64, 1), (512, 1, 64, 1)])
@pytest.mark.parametrize("keys,values", [(30.0, 0.0), (0.0, 30.0)])
def test_offsets_cancel_as_in_separate_products(seq, heads, dh, batch, keys, values):
    """Keys or values with a common offset: the gradients of queries and keys are sums that cancel.  Distance from 64 bits, rms over replicas and batches,
    against that of the path through separate products."""
    cfg, n = model(seq, heads, dh), 2
    d = heads * dh
    err = {}
    for variant in (0, 2):
        run = TfRun(base(n_replicas=n), cfg, batch)
        H.hdet_set_launch_shape(run.h, variant, 0)
        flat, off = run.orc.theta.copy(), 0
        for name, shape in I.transformer_shapes(cfg):
            k = int(np.prod(shape))
            if name == "b_qkv.0":
                flat[:, off + d:off + 2 * d] += keys
                flat[:, off + 2 * d:off + 3 * d] += values
            if name in ("w_qkv.0", "w_o.0"):
                flat[:, off:off + k] *= 10 / np.sqrt(d)          # outputs of the inputs' size
            if name == "w_qkv.0":
                w_qkv = slice(off, off + k)
            off += k
        run.orc.theta[:] = flat
        run.theta[:, :run.P] = torch.from_numpy(flat).to(run.theta.device)
        e = []
        for t in (1, 2, 3):
            ids, tgt, _ = run.forward_backward(t)
            _, ref = run.oracle_grads(flat, ids, tgt, t)
            got = run.g.cpu().numpy()
            e += [[norm_err(a, b) for a, b in zip(got[r, w_qkv].reshape(3, -1), ref[r, w_qkv].reshape(3, -1))] for r in range(n)]
        err[variant] = np.sqrt(np.mean(np.square(e), axis=0))
        run.close()
    # six samples of an error on either side: 0.7 to 1.1 of the separate products' where the row dots are sums of the dp that they are taken from,
    # 1.4 to 3 for the queries where they are not
    assert np.all(err[0] <= 1.25 * err[2]), (err[0], err[2])


def test_as_many_heads_as_the_separate_products_take():
    """2^23 heads, whose blocks of both kinds are more than a grid's 2^32 threads along one axis."""
    cfg, batch = dict(n_blocks=1, d_model=64, n_heads=8, d_ff=8, seq_len=1, vocab=9), 1 << 20
    got = []
    for variant in (0, 2):
        run = TfRun(base(n_replicas=1), cfg, batch)
        H.hdet_set_launch_shape(run.h, variant, 0)
        _, _, losses = run.forward_backward(1)
        got.append((losses[0], run.g.cpu().numpy()[0, :run.P]))
        run.close()
        del run
    assert abs(got[0][0] - got[1][0]) <= 1e-5
    off = 0
    for name, shape in I.transformer_shapes(cfg):
        k = int(np.prod(shape))
        part = slice(off + (2 * k // 3 if name.split(".")[0] in ("w_qkv", "b_qkv") else 0), off + k)     # one key: no gradient of queries and keys
        off += k
        # sums over 2^20 rows in four chains of 2^17 additions: independent roundings make 2^-24 sqrt(2^17) = 2.2e-5 on either side, of the size of the
        # largest partial sum, which is a few times the result's
        assert norm_err(got[0][1][part], got[1][1][part]) <= 2e-4, name
