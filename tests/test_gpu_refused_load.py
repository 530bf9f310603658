"""Loads refused for a repeated key that the sort's sample already meets: the
kernels behind it end at once and read nothing of what was not written then
(segment starts, splitters).  The next load in the same memory is exact."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_export_parity, mk_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", [9000, 65537, 1 << 20, (1 << 20) + 1, 3_000_001])
def test_one_key_then_distinct_keys(n, width):
    import paper_2604_21117_amd as g
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(n + width)
    keys = rng.permutation(np.unique(rng.integers(0, np.iinfo(dt).max, n, dtype=dt)))
    half = keys.copy()
    half[::2] = keys[0]
    for bad in (np.full(n, 7, dtype=dt), half):
        with pytest.raises(g.GtError) as e:
            mk_tree(bad, bad, width // 8, max_batch=4096)
        assert e.value.status == g.GT_ERR_DUPLICATE
        t = mk_tree(keys, keys ^ dt(5), width // 8, max_batch=4096)
        assert_export_parity(t, oracle.SortedArray(keys, keys ^ dt(5), width))
        t.close()
