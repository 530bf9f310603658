"""Inserts of many keys that fall into one leaf: on either side of the length
from which the leaf's old keys are searched for in the run, with old keys
below, between and above the new ones."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_export_parity, mk_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("run", [200, 255, 256, 257, 300, 2047, 2049, 9000])
def test_long_runs_into_one_leaf(width, run):
    dt = np.uint32 if width == 32 else np.uint64
    gap = 100 * run
    keys = (np.arange(1, 65, dtype=np.uint64) * gap).astype(dt)
    rng = np.random.default_rng(run)
    for at, step in ((0, 1), (20 * gap + 1, 3), (15 * gap + 7, 20 * gap // run), (63 * gap + 1, 1)):
        vals = synth.values_for(keys, 1, width)
        sa = oracle.SortedArray(keys, vals, width)
        t = mk_tree(keys, vals, width // 8, leaf_slack=1 << 12, max_batch=1 << 14, fill=0.75)
        k = (at + np.arange(run, dtype=np.uint64) * step).astype(dt)
        k = k[rng.permutation(run)]
        v = synth.values_for(k, 2, width)
        assert np.array_equal(t.insert(k, v), sa.insert(k, v)), (at, step)
        assert_export_parity(t, sa)
        t.close()
