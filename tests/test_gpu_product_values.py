"""Products of the mixed-precision MLP entry by entry against 64 bits.  The reference rounds to bfloat16 where the library
stores bfloat16, and no hidden unit is near its kink, so what is left is the rounding of fp32 sums and a rare stored value on the
other side of a rounding boundary: tight enough to see a contraction that loses its tail, a shifted element or a neighbour's
row, which the CPU test below plants in the reference."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
import paper_2604_24708_amd as H
from oracle.mlp_oracle import round_bf16, softmax_xent


def inputs(widths, batch, n, seed=5):
    """Weights U(+-1 / sqrt(fan in)), inputs N(0, 1): a product's entries spread by 0.58.  Hidden biases of +-2: every other unit is
    open, the rest shut, and the chance that one of a few hundred thousand lies within an fp32 rounding of its kink is 1e-3."""
    rng = np.random.Generator(np.random.Philox(seed))
    P = I.mlp_param_count(widths)
    theta = I.mlp_init(n, widths, seed) + 0.01 * rng.standard_normal((n, P), dtype=np.float32)
    off = 0
    for i in range(len(widths) - 1):
        off += widths[i + 1] * widths[i]
        if i + 2 < len(widths):
            theta[:, off:off + widths[i + 1]] = np.where(np.arange(widths[i + 1]) % 2 == 0, 2.0, -2.0)
        off += widths[i + 1]
    x = rng.standard_normal((n, batch, widths[0]), dtype=np.float32)
    y = rng.integers(0, widths[-1], (n, batch)).astype(np.int32)
    return theta.astype(np.float32), x, y


def bf16(a):
    return round_bf16(np.asarray(a, np.float32)).astype(np.float64)


def reference(theta, x, y, widths, slip=None):
    """One replica: loss, [(gradient, bound)] per tensor.  slip = (product, fault): "fwd0", "dgrad1", "wgrad0", ... formed wrongly."""
    def product(name, a, b):                       # a [m][k], b [k][n]
        if slip and slip[0] == name:
            k = a.shape[1]
            if slip[1] == "tail":                  # the last K mod 16 terms are lost (all of them belong to whole steps: one)
                a = a[:, :k - (k % 16 or 1)]
                b = b[:a.shape[1]]
            elif slip[1] == "shift":               # one row of the first operand (an open unit's) reads one element on
                a = a.copy()
                r = a.shape[0] // 4 * 2
                a[r] = np.roll(a[r], -1)
            elif slip[1] == "row":                 # a column of the result is another's (both open units')
                b = b.copy()
                b[:, (b.shape[1] - 1) // 2 * 2] = b[:, 0]
            elif slip[1] == "entry":               # one entry of the result is not written (an open unit's)
                c = a @ b
                c[(c.shape[0] - 1) // 2 * 2, (c.shape[1] - 1) // 2 * 2] = -2.0 if name[:3] == "fwd" and name != "fwd%d" % (len(widths) - 2) else 0.0
                return c
        return a @ b

    L, off, par = len(widths) - 1, 0, []
    for i in range(L):
        k = widths[i + 1] * widths[i]
        par.append((bf16(theta[off:off + k]).reshape(widths[i + 1], widths[i]), theta[off + k:off + k + widths[i + 1]].astype(np.float64)))
        off += k + widths[i + 1]
    act = [bf16(x)]
    for i in range(L):
        z = product("fwd%d" % i, act[i], par[i][0].T) + par[i][1]
        act.append(bf16(np.maximum(z, 0.0)) if i + 1 < L else z)
    loss, dz = softmax_xent(act[L], y.astype(np.int64))
    # What an fp32 rounding can push over a boundary of bfloat16, by size: of the output gradient (p - [label]) / B the p / B, whose
    # relative error stands against steps of up to 2^-7 (the label's own 1 / B does not move).
    out, loose = [], dz.copy()
    loose[np.arange(len(y)), y] += 1.0 / len(y)
    for i in range(L - 1, -1, -1):
        d = bf16(dz)
        # Fp32 sums of K terms: 16 x 2^-24 of the terms' sizes (a random walk of K up to 10^4 roundings stays below 4 x).  A stored
        # gradient an entry on the other side of a boundary, which is up to 2^-7 of it away, and a stored activation (no input is).
        out.append((d.sum(0), 2.0 ** -20 * np.abs(d).sum(0) + 2.0 ** -7 * loose.max(0)))
        moved = 2.0 ** -7 * (loose.max(0) + (np.abs(d).max(0) if i else 0.0))
        out.append((product("wgrad%d" % i, d.T, act[i]), 2.0 ** -20 * (np.abs(d).T @ np.abs(act[i])) + moved[:, None] * np.abs(act[i]).max(0)[None, :]))
        if i:
            open_ = act[i] > 0.0
            dz = np.where(open_, product("dgrad%d" % i, d, par[i][0]), 0.0)
            loose = np.abs(dz) + np.where(open_, np.sqrt((loose ** 2) @ (par[i][0] ** 2)), 0.0)
    return loss, out[::-1]                         # W_0, b_0, W_1, ...


def disagreements(loss, grads, ref):
    """What of a replica's loss and flat gradients is not the reference's."""
    want, tensors = ref
    bad = [] if abs(loss - want) <= 1e-5 * abs(want) else ["loss %.3e" % (abs(loss - want) / abs(want))]
    off = 0
    for i, (g, bound) in enumerate(tensors):
        e = np.abs(grads[off:off + g.size].reshape(g.shape) - g) / (bound + 1e-30)      # shut units: exactly 0
        off += g.size
        if not e.max() <= 1.0:
            bad.append("%s%d %.2f" % ("Wb"[i % 2], i // 2, e.max()))
    assert off == grads.size
    return bad


def compare_entry_by_entry(widths, batch, n, replicas):
    """The library's loss and gradients of a network against the reference, for the named replicas; all of them are finite."""
    theta, x, y = inputs(widths, batch, n)
    P = theta.shape[1]
    stride, dev = (P + 3) // 4 * 4, "cuda:0"
    td, g, m, v = (torch.full((n, stride), 7.0, device=dev) for _ in range(4))
    td[:, :P] = torch.from_numpy(theta)
    cfg = H.make_config(n_replicas=n, sync_interval=4, total_steps=10, lr_max=1e-3, alpha=0.1, widths=widths, batch=batch,
                        model_kind=H.HDET_MLP, optimizer=H.HDET_ADAMW, precision=H.HDET_BF16_GEMM_FP32_MASTER)
    ws = torch.empty(max(H.hdet_workspace_bytes(cfg, stride)[2], 16), dtype=torch.uint8, device=dev)
    copy = torch.zeros((n, stride), dtype=torch.bfloat16, device=dev)
    h = H.hdet_create(cfg, td, m, v, grads=g, params_bf16=copy, workspace=ws, plane_stride=stride)
    losses = H.hdet_forward_backward(h, torch.from_numpy(x).to(dev), torch.from_numpy(y).to(dev), want_losses=True)
    got = g[:, :P].double().cpu().numpy()
    H.hdet_destroy(h)
    for r in replicas:
        assert disagreements(losses[r], got[r], reference(theta[r], x[r], y[r], widths)) == []
    assert np.isfinite(got).all()


# bf16 operands of every alignment, one and two layers: few tiles (K in 4), long contractions over few tiles (K in 8), 64- and
# 128-wide tiles staged through LDS, and the LDS-direct kernel with rows of whole and of partial lines
CASES = [([33, 9], 7, 2), ([1503, 100], 97, 3), ([130, 36], 66, 3), ([4097, 1000], 37, 2), ([1031, 2111], 65, 2), ([512, 520], 300, 4), ([264, 2056], 130, 4),
         ([33, 31, 9], 7, 2), ([1503, 702, 100], 97, 6), ([130, 702, 36], 66, 3), ([1031, 2111, 10], 65, 2), ([787, 1501, 99], 96, 6),
         ([516, 2052, 12], 200, 5), ([999, 2055, 130], 260, 8), ([512, 1032, 264], 520, 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("widths,batch,n", CASES)
def test_loss_and_gradients_entry_by_entry(widths, batch, n):
    compare_entry_by_entry(widths, batch, n, range(n))


@pytest.mark.parametrize("widths,batch,n", [c for c in CASES if max(c[0]) < 1600])
def test_a_planted_mistake_is_seen(widths, batch, n):
    """Every product of the reference formed wrongly in every way, on the CPU: the comparison of the test above must tell."""
    theta, x, y = inputs(widths, batch, n)
    right = reference(theta[0], x[0], y[0], widths)
    flat = lambda ref: np.concatenate([g.ravel() for g, _ in ref[1]]).astype(np.float32).astype(np.float64)  # noqa: E731
    assert disagreements(np.float32(right[0]), flat(right), right) == []
    L = len(widths) - 1
    for name in ["fwd%d" % i for i in range(L)] + ["wgrad%d" % i for i in range(L)] + ["dgrad%d" % i for i in range(1, L)]:
        for fault in ("tail", "shift", "row", "entry"):
            wrong = reference(theta[0], x[0], y[0], widths, slip=(name, fault))
            assert disagreements(wrong[0], flat(wrong), right) != [], (name, fault)
