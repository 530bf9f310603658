"""Sorts of 2049 to 65536 keys: ranked by counting in one launch up to 8192
keys, the sample ranked by counting above.  Sizes around the change and around
the steps of the counting, with the key sets of the sample sort's test (equal
keys, sorted, few keys, all ones), for level-wise lookups and bulk loads."""
import pytest

import test_gpu_sample_sort as sample_sort

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", [2175, 2176, 8191, 8192, 8193, 16385, 32769])
def test_counted_ranks(n, width):
    sample_sort.test_levelwise_batch_and_bulk_load(n, width)
