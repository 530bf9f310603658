"""The sample sort behind bulk loads and sorted batches: sizes around every
change of its shape (groups, sample runs, tiles, one or two levels) with key
sets that make its groups and bins uneven (sorted, one key repeated, few keys,
keys in runs, all-ones keys, a skewed density).  Level-wise lookups need the
stable order of (key, position); bulk loads sort straight into the leaves and
refuse repeated keys."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_export_parity, mk_tree

pytestmark = pytest.mark.gpu

SIZES = [2049, 4096, 4097, 65536, 65537, 262144, 262145, 1 << 20, (1 << 20) + 1]
KINDS = ["uniform", "sorted", "reversed", "one key", "few keys", "all ones", "runs", "skewed"]


def _draw(kind, n, dt, rng):
    top = np.iinfo(dt).max
    if kind == "uniform":
        return rng.integers(0, top, n, dtype=dt, endpoint=True)
    if kind in ("sorted", "reversed"):
        k = np.arange(n, dtype=dt) * dt(3) + dt(7)
        return k if kind == "sorted" else k[::-1].copy()
    if kind == "one key":
        return np.full(n, 12345, dtype=dt)
    if kind == "few keys":
        return rng.integers(0, 7, n).astype(dt)
    if kind == "all ones":
        return np.where(np.arange(n) % 3 == 0, dt(0), top).astype(dt)
    if kind == "runs":
        start = rng.integers(0, top - dt(300), n // 100 + 1, dtype=dt)
        return (start[:, None] + np.arange(100, dtype=dt)[None, :]).reshape(-1)[:n]
    return (rng.random(n) ** 40 * float(top) * 0.999).astype(dt)


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", SIZES)
def test_levelwise_batch_and_bulk_load(n, width):
    import paper_2604_21117_amd as g
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(n + width)
    base = np.unique(_draw("uniform", 5000, dt, rng))
    vals = base * dt(3) + dt(1)
    tree = mk_tree(base, vals, width // 8, max_batch=4096)
    for kind in KINDS:
        q = _draw(kind, n, dt, rng)
        q[::5] = base[rng.integers(0, len(base), len(q[::5]))]
        v, f = tree.lookup_levelwise(q)
        at = np.minimum(np.searchsorted(base, q), len(base) - 1)
        hit = base[at] == q
        assert np.array_equal(f, hit.astype(np.uint8)), kind
        assert np.array_equal(v, np.where(hit, vals[at], np.iinfo(dt).max)), kind
        keys = np.unique(q)
        if len(keys) < len(q):
            with pytest.raises(g.GtError) as e:
                mk_tree(q, q, width // 8, max_batch=4096)
            assert e.value.status == g.GT_ERR_DUPLICATE, kind
        keys = rng.permutation(keys)
        t = mk_tree(keys, keys ^ dt(5), width // 8, max_batch=4096, fill=[1.0, 0.75, 0.5][n % 3])
        assert_export_parity(t, oracle.SortedArray(keys, keys ^ dt(5), width))
        t.close()
    assert g.tree_device_error(tree.h) == g.GT_OK
    tree.close()


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", [3000, 70000, 300000, (1 << 20) + 77])
def test_last_writer_needs_the_stable_order(n, width):
    """Repeated keys in one insert batch: the last one's value stays."""
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(n)
    keys = rng.integers(0, n // 8, n).astype(dt) * dt(97)
    vals = np.arange(n, dtype=dt)
    tree = mk_tree(np.zeros(0, dtype=dt), np.zeros(0, dtype=dt), width // 8, leaf_slack=n // 4 + 1024, max_batch=n)
    sa = oracle.SortedArray(np.zeros(0, dtype=dt), np.zeros(0, dtype=dt), width)
    assert np.array_equal(tree.insert(keys, vals), sa.insert(keys, vals))
    assert_export_parity(tree, sa)
    tree.close()
