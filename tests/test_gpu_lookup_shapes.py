"""Lookup shapes the library picks by batch and tree size, at the sizes where
it changes them: one query per group up to 2^16 queries, LDS staging from
2^17, values read after the match (and streamed on trees with 256 MB of leaf
lines) above 2^16."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_lookup_parity, key_set, mk_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,slack", [(32, 0), (64, 0), (64, 1 << 20), (32, 1 << 21)])
@pytest.mark.parametrize("n", [1, 40, 60000])
def test_shape_switches(width, slack, n):
    seed = 91
    keys = key_set(n, width, seed)
    vals = synth.values_for(keys, seed, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, max_batch=4096, leaf_slack=slack or 64)
    if slack:
        assert t.stats()["leaf_cap"] * 16 * (width // 8) * 2 >= 256 << 20
    for B in ((1 << 16) - 1, 1 << 16, (1 << 16) + 1, (1 << 17) - 1, 1 << 17, (1 << 17) + 33):
        q = synth.mixed_queries(keys, B, seed + B, width)
        q[-1] = np.iinfo(keys.dtype).max
        assert_lookup_parity(t, sa, q)
    # once the tree took updates the whole value line is read with the keys
    more = key_set(50, width, seed + 1)
    t.insert(more, synth.values_for(more, 7, width))
    sa.insert(more, synth.values_for(more, 7, width))
    assert_lookup_parity(t, sa, synth.mixed_queries(sa.keys.astype(keys.dtype), (1 << 17) + 33, seed, width))
