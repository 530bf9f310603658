"""Insert and delete batches above 2048 keys: the plan works by chunks of 2048
keys (two tiles a chunk from 2^21 keys on) and hands the upper levels to one
workgroup from a level that depends on the batch size.  Batches around those
sizes, of spread keys, dense runs (many new keys in one leaf), repeats and
updates, against the oracle after every batch."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_export_parity, mk_tree

pytestmark = pytest.mark.gpu


def _batch(rng, base, B, dt, kind):
    top = int(np.iinfo(dt).max)
    if kind == "spread":
        k = rng.integers(0, top, B, dtype=dt)
    elif kind == "runs":
        start = rng.integers(0, top - 4096, B // 700 + 1, dtype=dt)
        k = (start[:, None] + np.arange(700, dtype=dt)[None, :]).reshape(-1)[:B]
    else:  # one dense stretch, so that every level above it splits
        k = np.arange(B, dtype=dt) + dt(top // 3)
    k = k.copy()
    upd = rng.random(B) < 0.2
    k[upd] = base[rng.integers(0, len(base), int(upd.sum()))]
    rep = rng.random(B) < 0.1
    k[rep] = k[rng.integers(0, B, int(rep.sum()))]
    return k[rng.permutation(B)]


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("B", [2049, 4097, 8192, 8193, 65536, 65537])
def test_batches_around_the_plan_sizes(B, width):
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(B + width)
    keys = synth.uniform_keys(30000, B, width)
    vals = synth.values_for(keys, B, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=6 * B // 8 + 30000, max_batch=B)
    for kind in ("spread", "runs", "dense"):
        k = _batch(rng, keys, B, dt, kind)
        v = rng.integers(0, 1 << 31, B).astype(dt)
        assert np.array_equal(t.insert(k, v), sa.insert(k, v)), kind
        assert_export_parity(t, sa)
        gone = k[rng.permutation(B)][: B - B // 3].copy()
        if len(gone) > 2048:
            gone[::7] = rng.integers(0, 1 << 31, len(gone[::7])).astype(dt)
        assert np.array_equal(t.delete(gone), sa.delete(gone)), kind
        assert_export_parity(t, sa)
    t.close()


def test_two_tiles_a_chunk():
    B, width = (1 << 21) + 5, 64
    rng = np.random.default_rng(7)
    keys = synth.uniform_keys(200000, 3, width)
    vals = synth.values_for(keys, 3, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, 8, leaf_slack=B // 4, max_batch=B)
    k = np.concatenate([_batch(rng, keys, B // 2, np.uint64, "spread"), _batch(rng, keys, B - B // 2, np.uint64, "runs")])
    v = synth.values_for(k, 9, width)
    assert np.array_equal(t.insert(k, v), sa.insert(k, v))
    assert_export_parity(t, sa)
    gone = k[rng.permutation(B)]
    assert np.array_equal(t.delete(gone), sa.delete(gone))
    assert_export_parity(t, sa)
    t.close()
