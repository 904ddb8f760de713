"""Products that the alternating 256 x 256 kernel takes, at its edges -- rows, columns and contractions that end inside a tile, odd and even
numbers of K steps, each operand order, plain, gated and fp32 results -- entry by entry against 64 bits."""
import pytest

from test_gpu_product_values import compare_entry_by_entry

# (widths, batch, replicas): logits 1500 x 2056 over K = 520 and their weight gradient over K = 1500, 432 and 216 tiles;
# ReLU outputs 2000 x 2040 over K = 520 and the gradient through them over K = 1000, 256 tiles each;
# logits 3000 x 2056 over K = 392, 864 tiles
CASES = [([520, 2056], 1500, 8), ([520, 2040, 1000], 2000, 4), ([392, 2056], 3000, 8)]


@pytest.mark.gpu
@pytest.mark.parametrize("widths,batch,n", CASES)
def test_loss_and_gradients_entry_by_entry(widths, batch, n):
    compare_entry_by_entry(widths, batch, n, (0, n - 1))
