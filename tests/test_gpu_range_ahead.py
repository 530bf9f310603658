"""Scans that read several leaves at once: batches at the sizes where the
number of leaves ahead changes (2048, 4096, 2^14 scans), on trees whose leaves
have consecutive references, on grown ones where most do not, after deletes
that give leaves up, and at the end of a leaf pool without a spare leaf."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_range_parity, key_set, mk_tree

pytestmark = pytest.mark.gpu


def scans(keys, B, seed, maxlen, width):
    lo, hi, mc = synth.range_starts_and_lengths(keys, B, seed, maxlen)
    rng = np.random.default_rng(seed)
    top = np.iinfo(keys.dtype).max
    hi = np.where(rng.random(B) < 0.5, top, hi).astype(keys.dtype)
    lo[:2], hi[:2], mc[:2] = 0, top, maxlen
    return lo, hi, mc


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("B,maxlen", [(1, 300), (2048, 70), (2049, 70), (4096, 33), (4097, 33), (1 << 14, 20),
                                      ((1 << 14) + 1, 20)])
def test_leaves_ahead(width, B, maxlen):
    seed = 400 + B
    keys = key_set(9000, width, seed, edges=True)
    vals = synth.values_for(keys, seed, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, max_batch=8192, leaf_slack=4096)
    assert_range_parity(t, sa, *scans(keys, B, seed, maxlen, width))
    more = key_set(6000, width, seed + 1)
    t.insert(more, synth.values_for(more, 5, width))
    sa.insert(more, synth.values_for(more, 5, width))
    assert_range_parity(t, sa, *scans(keys, B, seed + 2, maxlen, width))
    gone = np.sort(keys)[1000:6000]
    t.delete(gone)
    sa.delete(gone)
    assert_range_parity(t, sa, *scans(keys, B, seed + 3, maxlen, width))


@pytest.mark.parametrize("n", [0, 1, 16, 17, 48, 64])
def test_few_leaves_no_spare(n):
    """At most four leaves in a pool of just as many: the leaves ahead of the
    last one are past the pool's end."""
    keys = key_set(n, 64, 3) if n else np.zeros(0, dtype=np.uint64)
    vals = synth.values_for(keys, 3, 64)
    sa = oracle.SortedArray(keys, vals, 64)
    t = mk_tree(keys, vals, 8, max_batch=1024)
    top = np.uint64(np.iinfo(np.uint64).max)
    lo = np.concatenate([np.zeros(3, dtype=np.uint64), keys])
    hi = np.full(len(lo), top)
    mc = np.resize(np.array([100, 1, 17], dtype=np.uint32), len(lo))
    assert_range_parity(t, sa, lo, hi, mc)
