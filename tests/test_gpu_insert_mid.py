"""Insert and delete batches of 65 to 2048 keys: one launch ranks and locates
the batch (repeats keep their own records), one workgroup of 64, 256 or 1024
threads plans it, six levels at a time.  Sizes around the workgroup sizes,
repeats, updates, dense runs, both edge keys, trees of one level and of more
than six, every LDS depth of the descent; statuses and the whole tree against
the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_export_parity, mk_tree

pytestmark = pytest.mark.gpu


def _batch(rng, base, B, dt, kind):
    top = int(np.iinfo(dt).max)
    if kind == "dense":  # one stretch: every level above it splits
        k = np.arange(B, dtype=dt) + dt(top // 3)
    else:
        k = rng.integers(0, top, B, dtype=dt)
    if kind == "one":
        k[:] = k[0]
    else:
        if len(base):
            upd = rng.random(B) < 0.25
            k[upd] = base[rng.integers(0, len(base), int(upd.sum()))]
        rep = rng.random(B) < 0.2
        k[rep] = k[rng.integers(0, B, int(rep.sum()))]
        k[:4] = [0, top, 0, top]
    return k[rng.permutation(B)]


def _drive(n, width, B, **kw):
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(B + width + n)
    keys = synth.uniform_keys(n, B, width) if n else np.zeros(0, dtype=dt)
    vals = synth.values_for(keys, B, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=4 * B + 64, max_batch=2048, **kw)
    height = t.stats()["height"]
    for kind in ("spread", "dense", "one"):
        k = _batch(rng, keys, B, dt, kind)
        v = rng.integers(0, 1 << 31, B).astype(dt)
        assert np.array_equal(t.insert(k, v), sa.insert(k, v)), kind
        assert_export_parity(t, sa)
        gone = k[rng.permutation(B)].copy()
        gone[::5] = rng.integers(0, 1 << 31, len(gone[::5])).astype(dt)
        assert np.array_equal(t.delete(gone), sa.delete(gone)), kind
        assert_export_parity(t, sa)
    t.close()
    return height


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("B", [65, 128, 129, 256, 257, 512, 513, 1000, 2047, 2048])
def test_mid_batches(B, width):
    _drive(20000, width, B)


@pytest.mark.parametrize("n", [0, 3, 200])
@pytest.mark.parametrize("B", [65, 300, 2048])
def test_small_trees(n, B):
    _drive(n, 64, B)


@pytest.mark.parametrize("B", [100, 400, 2048])
def test_more_than_six_levels(B):
    assert _drive(2500000, 64, B, fill=0.5) >= 7


@pytest.mark.parametrize("lds", [1, 3, 4])
@pytest.mark.parametrize("width", [32, 64])
def test_descent_from_lds(lds, width):
    _drive(20000, width, 700, lds_levels=lds)
