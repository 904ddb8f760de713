"""The loss kernel for narrow rows at widths around its steps (how many classes a lane holds) and beyond them: gradients of a one-layer
classifier against autograd in 64 bits."""
import numpy as np
import pytest

from test_gpu_products import mlp_grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("classes", [2, 63, 64, 65, 256, 257, 511, 513, 1000, 1025, 2047, 2049])
def test_classifier_gradients(classes, bf16):
    got, ref, slices = mlp_grads([16, classes], 5, 2, bf16=bf16)
    for s in slices:
        # fp32: sums of up to 2049 terms in some order (2^-24 sqrt(2049) = 2.7e-6); bf16: logits of rounded operands (2^-9,
        # sixteen of them) move the output gradient by as much, which is rounded once more
        assert np.linalg.norm(got[:, s] - ref[:, s]) <= (1e-2 if bf16 else 5e-6) * np.linalg.norm(ref[:, s])
