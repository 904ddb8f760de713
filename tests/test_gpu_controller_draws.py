"""Eq. 9's permutations, all channels, for 1 to 64 replicas; the seeds of the last cases are ones whose first draw at N = 64
refuses a word (found by search: about one permutation in three million does), in channel 0."""
import pytest
import torch

from oracle import hdet_oracle as O

import paper_2604_24708_amd as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,seed", [(1, 7), (2, 7), (3, 8), (31, 9), (64, 10), (64, 3579023), (64, 8440959)])
def test_permutations_of_all_channels(n, seed):
    extra = [(H.HDET_CH_WD, 0.05, 0.5, 1e-3, 0.0, 1.0)]
    th, m, v, g = (torch.zeros((n, 8), device="cuda:0") for _ in range(4))
    cfg = H.make_config(n_replicas=n, sync_interval=1, total_steps=100, warm_steps=0, lr_max=1e-2, alpha=0.1, autolr_enabled=1,
                        model_kind=H.HDET_FLAT, n_params=8, optimizer=H.HDET_ADAMW, seed=seed, extra=extra)
    h = H.hdet_create(cfg, th, m, v, plane_stride=8)
    for k in (1, 2):
        H.hdet_fanout_step(h, g, H.HDET_FUSE_CONVERGE)
        H.hdet_converge(h)
        H.hdet_autolr_update(h, [1.0 + 0.01 * r for r in range(n)])
        st = H.hdet_get_state(h)
        for j in range(2):
            assert [st.perm[j][r] for r in range(n)] == O.permutation(seed, k, j, n).tolist()
    H.hdet_destroy(h)
