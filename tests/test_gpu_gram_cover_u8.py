"""All-pairs of U8 masks of 129 to 256 members, one unit of all row blocks: long
splits (the INT8 plan has at most one per CU, however many points), with odd and
even slab counts, splits of unequal length and a ragged last slab.  Exact."""
import pytest
import torch

from tests.test_gpu_gram_cover import _check

pytestmark = pytest.mark.gpu


# slabs of 128 points over 256 splits: 31, 31 or 32, 64, 165 or 166
@pytest.mark.parametrize("m", [31 * 32768, 31 * 32768 + 5 * 128 + 48, 64 * 32768, 165 * 32768 + 77 * 128 + 16])
@pytest.mark.parametrize("n", [129, 136, 160, 161, 192, 224, 256])
def test_long_splits(n, m):
    _check(n, m, torch.uint8)
