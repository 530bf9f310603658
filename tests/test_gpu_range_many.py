"""Range batches on either side of the sizes from which a scan takes 8 lanes
(64-bit keys above 12288 scans, 32-bit keys above 24576)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_range_parity, key_set, mk_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,B", [(64, 12288), (64, 12289), (64, 30000), (32, 24576), (32, 24577), (32, 50000)])
def test_many_scans(width, B):
    keys = key_set(50000, width, 81, edges=True)
    vals = synth.values_for(keys, 81, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=1 << 12, max_batch=1 << 14)
    rng = np.random.default_rng(B)
    k = synth.uniform_keys(9000, 82, width, exclude=keys)
    for grown in (False, True):
        if grown:
            assert np.array_equal(t.insert(k, k), sa.insert(k, k))
        lo = synth.mixed_queries(keys, B, B + grown, width)
        hi = np.where(rng.random(B) < 0.3, keys[rng.integers(0, len(keys), B)], np.iinfo(keys.dtype).max)
        assert_range_parity(t, sa, lo, hi.astype(keys.dtype), rng.integers(0, 40, B).astype(np.uint32))
    t.close()


def test_many_short_scans_of_32_bit_keys():
    """2^17 scans of one pair take well below the time of 64-bit keys, whose
    lines are twice as long (as long with 16 lanes a scan, 0.72 with 8)."""
    import torch
    import paper_2604_21117_amd as g
    B, n, us = 1 << 17, 1 << 18, {}
    for width in (32, 64):
        keys = key_set(n, width, 83)
        t = mk_tree(keys, keys, width // 8)
        lo = t.dev(keys[np.random.default_rng(84).integers(0, n, B)])
        hi, mx = torch.full_like(lo, -1), torch.ones(B, dtype=torch.int32, device="cuda")
        off = torch.arange(B, device="cuda")
        ok, ov, cnt = torch.empty_like(lo), torch.empty_like(lo), torch.empty_like(mx)
        torch.cuda.synchronize()  # the inputs are there before another stream reads them
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            g.tree_range_batch(t.h, lo, hi, mx, off, ok, ov, cnt)
        torch.cuda.synchronize()
        gr = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gr, stream=s):
            for _ in range(20):
                g.tree_range_batch(t.h, lo, hi, mx, off, ok, ov, cnt)
        gr.replay()
        times = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            gr.replay()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 50)
        us[width] = min(times)
        assert bool((ok == lo).all()) and bool((cnt == 1).all())
        t.close()
    assert us[32] < 0.9 * us[64], us
