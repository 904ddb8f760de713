"""The general LDS kernel with one K step in flight, which grids of many blocks take, entry by entry against 64 bits: tiles of 64 and of 128, rows that
start at odd elements and not, contractions of one step, of whole steps and with a rest, forward products and both gradients."""
import pytest

from test_gpu_product_values import compare_entry_by_entry

pytestmark = pytest.mark.gpu

# 64 x 64: 1320 blocks of the first product and of the gradient through it; 128 x 128: 1152 of both
CASES = [([k, 2052, 12], 260, 8) for k in (6, 31, 64, 130, 250, 516)] + [([36, 1500, 40], 1500, 8), ([37, 1501, 33], 1500, 8), ([130, 1492, 66], 1450, 8)]


@pytest.mark.parametrize("widths,batch,n", CASES)
def test_loss_and_gradients_entry_by_entry(widths, batch, n):
    compare_entry_by_entry(widths, batch, n, (0, n - 1))
