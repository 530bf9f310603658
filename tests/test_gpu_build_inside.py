"""Where a bulk load sorts: inside its arena when nothing there has to survive,
beside it when a tree lives in any part of the arena.  A refused load in a free
arena is followed by a good one; a tree that lives in the arena, also one of
another kind or in a part of it, stays whole through a refused load and is gone
after destroy.  Sizes on each way the pairs are sorted, at two fills (leaves
that hold equally many pairs and leaves that do not), with little and with much
scratch."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_export_parity

pytestmark = pytest.mark.gpu


def _pairs(n, width, seed):
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(seed)
    k = rng.permutation(np.unique(rng.integers(0, np.iinfo(dt).max, n + n // 50 + 8, dtype=dt, endpoint=True))[:n])
    return k, k * dt(5) + dt(3)


@pytest.mark.parametrize("max_batch", [1 << 8, 1 << 18])
@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", [1, 8192, 8193, 16384, 70001, 300000, (1 << 20) + 77, 1 << 21])
def test_loads_in_a_free_arena(n, width, max_batch):
    import torch
    import paper_2604_21117_amd as g
    kb = width // 8
    for fill in (1.0, 0.7):
        keys, vals = _pairs(n, width, n + width)
        p = g.make_params(kb, max_batch=max_batch, fill=fill)
        arena = torch.empty(g.tree_arena_bytes(p, n, 16), dtype=torch.uint8, device="cuda")
        bad = keys.copy()
        bad[n // 2] = bad[0]
        for k in (keys, bad, keys[::-1], keys[np.arange(n) % 3], keys):
            distinct = len(np.unique(k)) == n
            args = (p, g.to_device(k.copy()), g.to_device(vals), arena)
            if not distinct:
                with pytest.raises(g.GtError) as e:
                    g.tree_build(*args)
                assert e.value.status == g.GT_ERR_DUPLICATE
                continue
            h = g.tree_build(*args)
            sa = oracle.SortedArray(k, vals, width)
            bits, ek, ev = oracle.check_export(g.tree_export(h), n)
            assert bits == 0 and np.array_equal(ek, sa.keys) and np.array_equal(ev, sa.vals)
            g.tree_destroy(h)


def test_trees_that_live_in_the_arena():
    import torch
    import paper_2604_21117_amd as g
    n = 40000
    keys, vals = _pairs(n, 64, 1)
    p = g.make_params(8, max_batch=1 << 16)
    arena = torch.empty(g.tree_arena_bytes(p, n, 64), dtype=torch.uint8, device="cuda")
    bad = keys.copy()
    bad[7] = bad[n - 1]
    kd, vd, bd = g.to_device(keys), g.to_device(vals), g.to_device(bad)

    def refused():
        with pytest.raises(g.GtError) as e:
            g.tree_build(p, bd, vd, arena)
        assert e.value.status == g.GT_ERR_DUPLICATE

    # a small tree in the middle, a static tree near the end
    small = arena[arena.numel() // 2 // 256 * 256:]
    k2, v2 = _pairs(300, 32, 2)
    p2 = g.make_params(4, max_batch=16)
    h = g.tree_build(p2, g.to_device(k2), g.to_device(v2), small)
    before = arena.clone()
    refused()
    assert bool((arena == before).all())
    sa2 = oracle.SortedArray(k2, v2, 32)
    bits, ek, ev = oracle.check_export(g.tree_export(h), 300)
    assert bits == 0 and np.array_equal(ek, sa2.keys) and np.array_equal(ev, sa2.vals)
    g.tree_destroy(h)
    ps = g.make_static_params(8, 32)
    k3, v3 = _pairs(500, 64, 3)
    need = g.tree_arena_bytes(ps, 500)
    at = (arena.numel() - need) // 256 * 256
    h = g.tree_build(ps, g.to_device(k3), g.to_device(v3), arena[at:at + need])
    before = arena.clone()
    refused()
    assert bool((arena == before).all())
    g.tree_destroy(h)
    # an outgrown tree: the load over it succeeds, both handles are ended
    h = g.tree_build(p, kd, vd, arena)
    h2 = g.tree_build(p, kd.flip(0), vd, arena)
    sa = oracle.SortedArray(keys[::-1], vals, 64)
    bits, ek, ev = oracle.check_export(g.tree_export(h2), n)
    assert bits == 0 and np.array_equal(ek, sa.keys) and np.array_equal(ev, sa.vals)
    g.tree_destroy(h)
    g.tree_destroy(h2)
    # a failed sort, with and without a tree in the arena
    t = g.Tree(keys, vals, 8, max_batch=1 << 14)
    before = t.arena.clone()
    old = g.set_sort_spin_limit(0)
    try:
        with pytest.raises(g.GtError) as e:
            g.tree_build(t.params, kd, vd, t.arena)
        assert e.value.status == g.GT_ERR_DEVICE
        assert bool((t.arena == before).all())
        with pytest.raises(g.GtError) as e:
            g.tree_build(p, kd, vd, arena)
        assert e.value.status == g.GT_ERR_DEVICE
    finally:
        g.set_sort_spin_limit(old)
    assert_export_parity(t, oracle.SortedArray(keys, vals, 64))
    t.close()
