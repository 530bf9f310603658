"""Keys laid out against a fixed sample of the sort: the positions that a hash
of index and size would sample hold keys spread over the whole range, all others
lie between two of those.  With that sample they fall into one group, which one
workgroup sorts in device memory; the sort samples elsewhere in every call."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import key_set, mk_tree
from test_gpu_lookup_rules import lookup_us

pytestmark = pytest.mark.gpu


def _hash(x):
    x = x.astype(np.uint32)
    x ^= x >> np.uint32(16)
    x *= np.uint32(0x7feb352d)
    x ^= x >> np.uint32(15)
    x *= np.uint32(0x846ca68b)
    return x ^ (x >> np.uint32(16))


@pytest.mark.parametrize("width", [32, 64])
def test_no_layout_defeats_the_sample(width):
    n, S = 1 << 18, 4096
    i = np.arange(S, dtype=np.uint64)
    a, b = i * n // S, (i + 1) * n // S
    at = a + _hash((i * 0x9E3779B9 + n) & 0xFFFFFFFF) % (b - a)
    rng = np.random.default_rng(width)
    dt = np.uint32 if width == 32 else np.uint64
    step = (1 << width) // (S + 1)
    q = (10 * step + 1 + rng.permutation(step // 2 if width == 32 else n)[:n] % (step - 2)).astype(dt)
    q[at] = (np.arange(1, S + 1, dtype=np.uint64) * step).astype(dt)[rng.permutation(S)]
    keys = np.unique(np.concatenate([q[:: 5], key_set(1000, width, 5)]))
    vals = synth.values_for(keys, 6, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8)
    us = {}
    for name, x in (("against", q), ("uniform", synth.mixed_queries(keys, n, 7, width))):
        gv, gf = t.lookup_levelwise(x)
        ov, of = sa.lookup(x)
        assert np.array_equal(gf, of) and np.array_equal(gv, ov), name
        us[name] = lookup_us(t, x, levelwise=True)
    assert us["against"] < 3 * us["uniform"], us
    t.close()
