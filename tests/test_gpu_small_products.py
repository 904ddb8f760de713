"""Products of few tiles entry by entry against 64 bits: contractions of one to seven steps of 32 in the general LDS kernel (four in flight; none, some
and all of them whole), rows that start at odd elements and not, and aligned products on both sides of K = 512."""
import pytest

from test_gpu_product_values import compare_entry_by_entry

pytestmark = pytest.mark.gpu

# 120 tiles of 64 x 64 and more: beyond the fragment kernel.  Widths 300 and 301: whole dwords, odd elements.
CASES = [([k, 300, 301], 130, 8) for k in (5, 32, 33, 64, 129, 160, 161, 200)] + [([504, 520, 512], 200, 6), ([1032, 264, 1032], 136, 5)]


@pytest.mark.parametrize("widths,batch,n", CASES)
def test_loss_and_gradients_entry_by_entry(widths, batch, n):
    compare_entry_by_entry(widths, batch, n, (0, n - 1))
