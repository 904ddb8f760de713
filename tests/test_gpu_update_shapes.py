"""The update's default kernels against the general one (forced by hdet_set_launch_shape), bit for bit: planes of fewer than
four parameters and of every remainder mod 4, and 17 to 64 replicas (two to four a wavefront), with one set of moments, with
SGD and its mean gradient, and with the converge standing alone."""
import numpy as np
import pytest
import torch

from test_gpu_flat import FlatRun, base_cfg, tol_at
from oracle import hdet_oracle as O

import paper_2604_24708_amd as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opt,mode,one_state", [(O.ADAMW, O.GRAD_SHARED, True), (O.SGDM, O.GRAD_SHARED, False),
                                                (O.SGDM, O.GRAD_PER_REPLICA, False)])
@pytest.mark.parametrize("n,P", [(1, 3), (2, 1), (5, 2), (16, 257), (17, 3), (18, 1022), (33, 259), (48, 5), (49, 256), (64, 1),
                                 (2, 4), (3, 1024), (16, 516), (2, 4000002)])
def test_default_kernels_equal_the_general_one(n, P, opt, mode, one_state):
    d = base_cfg(n_replicas=n, optimizer=opt, grad_mode=mode, shared_opt_state=one_state)
    a, b = FlatRun(d, P, stride=(P + 3) // 4 * 4 + 8, variant=1, blocks=3), FlatRun(d, P, stride=(P + 3) // 4 * 4 + 8)
    for t in range(1, 9):
        fuse = t == 4                       # t = 8: hdet_converge does it
        a.step(t, fuse); b.step(t, fuse)
        a.compare(tol_at(t)); b.compare(tol_at(t))
        assert torch.equal(a.theta, b.theta) and torch.equal(a.m, b.m) and torch.equal(a.v, b.v)
    a.close(); b.close()


@pytest.mark.parametrize("n", [8, 32])
def test_bf16_copy_of_trailing_parameters(n):
    """Widths 5-3: 18 parameters, two beyond the last whole column, with the copy that the products read."""
    P, stride = 18, 24
    g = torch.Generator(device="cuda:0").manual_seed(1)
    th = torch.randn((n, stride), device="cuda:0", generator=g)
    m, v, grads = (torch.zeros_like(th) for _ in range(3))
    sh = torch.full((n, stride), 3.0, dtype=torch.bfloat16, device="cuda:0")
    cfg = H.make_config(n_replicas=n, sync_interval=2, total_steps=8, warm_steps=0, lr_max=1e-2, alpha=0.1, model_kind=H.HDET_MLP,
                        widths=[5, 3], batch=2, precision=H.HDET_BF16_GEMM_FP32_MASTER)
    ws = torch.zeros(max(H.hdet_workspace_bytes(cfg, stride)[2], 16), dtype=torch.uint8, device="cuda:0")
    h = H.hdet_create(cfg, th, m, v, grads=grads, params_bf16=sh, workspace=ws, plane_stride=stride)
    for t in range(1, 5):
        grads[:, :P].normal_(generator=g)
        H.hdet_fanout_step(h, grads, H.HDET_FUSE_CONVERGE if t == 2 else 0)
        if t % 2 == 0:
            H.hdet_converge(h)
            H.hdet_autolr_update(h, np.linspace(1.0, 2.0, n).tolist())
        torch.cuda.synchronize()
        assert torch.equal(sh[:, :P].view(torch.int16), th[:, :P].to(torch.bfloat16).view(torch.int16))
        assert torch.all(sh[:, P:] == 3.0)
        assert (t % 2 == 1) or torch.equal(th[:, :P], th[:1, :P].expand(n, P))
    H.hdet_destroy(h)
