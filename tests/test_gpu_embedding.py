"""The token-embedding gradient against the position-embedding gradient: with one sequence per replica the latter holds the
gradient of every row, so that row sums by token id are the former.  Lengths around the 64 rows that a block orders and the 32
sorted rows that a wavefront adds up; ids all alike, all different, alternating, and descending."""
import numpy as np
import pytest
import torch

import hdet_inputs as I
import paper_2604_24708_amd as H
from oracle import transformer_oracle as T
from test_gpu_transformer import TfRun, base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("S,d,pattern", [(1, 8, "same"), (63, 8, "pairs"), (64, 16, "down"), (65, 8, "same"), (97, 12, "pairs"), (130, 520, "same"),
                                         (200, 8, "mixed"), (321, 24, "mixed")])
def test_token_gradient_is_the_sum_of_its_rows(S, d, pattern, bf16):
    n, V, dev = 2, 400, "cuda:0"
    cfg_d = dict(n_blocks=1, d_model=d, n_heads=1, d_ff=16, seq_len=S, vocab=V)
    P = I.transformer_param_count(cfg_d)
    stride = (P + 3) // 4 * 4
    g = torch.Generator(device=dev).manual_seed(S)
    theta = torch.zeros((n, stride), device=dev)
    theta[:, :P].normal_(0.0, 0.3, generator=g)
    m, v, grads = torch.zeros_like(theta), torch.zeros_like(theta), torch.full_like(theta, 7.0)
    pos = torch.arange(S, device=dev)
    ids = dict(same=torch.full_like(pos, 5), pairs=(pos * 7 + 3) % 2 * 399, down=V - 1 - pos,
               mixed=torch.where(pos % 3 == 0, torch.full_like(pos, 11), (pos * 37) % V))[pattern].to(torch.int32)
    ids = torch.stack([ids, ids.flip(0)]).view(n, 1, S).contiguous()
    y = torch.randint(0, V, (n, 1, S), generator=g, device=dev, dtype=torch.int32)
    cfg = H.make_config(n_replicas=n, sync_interval=4, total_steps=8, warm_steps=0, lr_max=1e-3, alpha=0.1, model_kind=H.HDET_TRANSFORMER,
                        batch=1, precision=H.HDET_BF16_GEMM_FP32_MASTER if bf16 else H.HDET_FP32, **cfg_d)
    shadow = torch.zeros((n, stride), dtype=torch.bfloat16, device=dev) if bf16 else None
    ws = torch.zeros(max(H.hdet_workspace_bytes(cfg, stride)[2], 16), dtype=torch.uint8, device=dev)
    h = H.hdet_create(cfg, theta, m, v, grads=grads, params_bf16=shadow, workspace=ws, plane_stride=stride)
    for _ in range(2):                                   # the second pass finds the first one's gradients in place
        H.hdet_forward_backward(h, ids, y)
    torch.cuda.synchronize()
    H.hdet_destroy(h)
    tok, dpos = grads[:, :V * d].view(n, V, d).double(), grads[:, V * d:V * d + S * d].view(n, S, d).double()
    for r in range(n):
        want = torch.zeros((V, d), dtype=torch.float64, device=dev).index_add_(0, ids[r, 0].long(), dpos[r])
        size = torch.zeros((V, d), dtype=torch.float64, device=dev).index_add_(0, ids[r, 0].long(), dpos[r].abs())
        # an fp32 sum of k <= S terms in any order: at most k 2^-24 of their absolute sum
        assert torch.all((tok[r] - want).abs() <= S * 2.0 ** -24 * size)
        assert float(size.max()) > 0.0


# rows times replicas on both sides of where counting the ids gives way to sorting them (800 rows a compute unit), each size of
# the sort, and rows that are no power of two
@pytest.mark.parametrize("n,S,B", [(3, 10, 13), (64, 64, 50), (64, 64, 51), (64, 25, 164), (26, 63, 127), (13, 64, 246), (13, 64, 256), (25, 61, 268)])
def test_embedding_gradients_against_the_oracle(n, S, B):
    cfg = dict(n_blocks=1, d_model=8, n_heads=1, d_ff=16, seq_len=S, vocab=150)
    run = TfRun(base(n_replicas=n), cfg, B)
    ids, tgt, losses = run.forward_backward(1)
    run.forward_backward(1)                                  # the second pass finds the first one's gradients in place
    got = run.g.double().cpu().numpy()
    k, m = 150 * 8, 150 * 8 + S * 8
    for r in {0, n // 2, n - 1}:
        loss, ref = T.loss_and_grad(run.orc.theta[r], ids[r], tgt[r], cfg)
        assert abs(losses[r] - loss) <= 1e-5 * loss
        # per row, in norm: a sum of up to a third of the M rows, each off by the few 2^-24 of a chain of fp32 products, and summed
        # in fp32 (a random walk of up to sqrt(5000) such roundings); one term more or less is 1 / 5000 of the largest sum at least
        for a, b in ((got[r, :k], ref[:k]), (got[r, k:m], ref[k:m])):
            a, b = a.reshape(-1, 8), b.reshape(-1, 8).astype(np.float64)
            assert np.all(np.linalg.norm(a - b, axis=1) <= 4e-5 * np.linalg.norm(b, axis=1) + 1e-6 * np.linalg.norm(b) / np.sqrt(len(b)))
    run.close()
