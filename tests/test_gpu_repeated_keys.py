"""Batches whose keys repeat, through the device sort (above 8192 keys): the
sort deals a bin of one key by position, so its results and its time should
not depend on how often keys occur."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_export_parity, key_set, mk_tree

pytestmark = pytest.mark.gpu

N = 40000


def batch(kind, keys, B, seed):
    rng = np.random.default_rng(seed)
    if kind == "one":
        return np.repeat(keys[:1], B)
    if kind == "two":
        return keys[rng.integers(0, 2, B)]
    if kind == "hundred":
        return keys[rng.integers(0, 100, B)]
    if kind == "zipf":
        r = np.minimum(np.floor(np.exp(rng.random(B) * np.log(len(keys)))).astype(np.int64), len(keys)) - 1
        return keys[rng.permutation(len(keys))[r]]
    q = keys[rng.integers(0, len(keys), B)]
    if kind == "bursts":  # one key at both ends, nothing between
        q[:B // 5] = keys[7]
        q[-B // 5:] = keys[7]
    elif kind == "half":
        q[rng.random(B) < 0.5] = keys[3]
    elif kind == "sorted_hundred":
        q = np.sort(keys[rng.integers(0, 100, B)])
    elif kind == "runs":  # runs of consecutive keys, far apart
        q = keys[rng.integers(0, len(keys), B // 64 + 1)].repeat(64)[:B] + np.arange(B, dtype=keys.dtype) % 64
    elif kind == "uneven_runs":  # a few large bins among small ones
        q[::3] = keys[5] + (np.arange(len(q[::3])) % 40).astype(keys.dtype)
    return q


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("B", [8193, 20000, (1 << 18) + 5, 1 << 20])
def test_repeated_keys_sort_right(width, B):
    keys = key_set(N, width, 5100 + width, edges=True)
    vals = synth.values_for(keys, 3, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8)
    for i, kind in enumerate(("one", "two", "hundred", "zipf", "bursts", "half", "sorted_hundred", "runs", "uneven_runs")):
        q = batch(kind, keys, B, B + i)
        gv, gf = t.lookup_levelwise(q)
        ov, of = sa.lookup(q)
        assert np.array_equal(gf, of) and np.array_equal(gv, ov), (kind, B)
    t.close()


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("kind", ["one", "hundred", "zipf", "bursts", "half"])
def test_repeated_keys_keep_their_order(width, kind):
    """An insert takes a repeated key's last value: equal keys stay in batch
    order through the sort."""
    B = 50000
    keys = key_set(N, width, 5200 + width)
    vals = synth.values_for(keys, 3, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=1 << 13, max_batch=B)
    fresh = synth.uniform_keys(2000, 5300, width, exclude=keys)
    k = batch(kind, np.concatenate([fresh, keys[:2000]]), B, 11)
    v = synth.values_for(np.arange(B, dtype=k.dtype), 12, width)
    assert np.array_equal(t.insert(k, v), sa.insert(k, v))
    assert_export_parity(t, sa)
    t.close()


@pytest.mark.parametrize("width", [32, 64])
def test_repeated_keys_take_no_longer(width):
    """2^15 keys of which 100 differ: within 1.5 times the time of as many
    different ones (1.15 measured; 2.0 where such groups are merge-sorted)."""
    import torch
    import paper_2604_21117_amd as g
    B = 1 << 15
    keys = key_set(1 << 18, width, 5400 + width)
    t = mk_tree(keys, synth.values_for(keys, 3, width), width // 8)
    v = torch.empty(B, dtype=t.tdtype, device="cuda")
    f = torch.empty(B, dtype=torch.uint8, device="cuda")
    ws = t.levelwise_workspace(B)
    us = {}
    for kind in ("hundred", "all"):
        q = t.dev(keys[:B] if kind == "all" else batch(kind, keys, B, 1))
        torch.cuda.synchronize()  # the inputs are there before another stream reads them
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            g.tree_lookup_levelwise(t.h, q, 0, v, f, ws)
        torch.cuda.synchronize()
        gr = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gr, stream=s):
            for _ in range(20):
                g.tree_lookup_levelwise(t.h, q, 0, v, f, ws)
        gr.replay()
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            gr.replay()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        us[kind] = sorted(times)[3]
        assert bool(f.all())
    assert us["hundred"] < 1.5 * us["all"], us
    t.close()
