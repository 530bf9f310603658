"""What a bulk load may do to its arena: nothing before its keys are known to
be good.  A load refused for a repeated key, or whose sort fails, leaves a tree
that lives in the arena as it was, byte for byte; keys and values that lie in
the arena themselves are read before the tree is written over them.  Sizes on
each way the pairs are sorted (ranked, one scatter, two)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_export_parity

pytestmark = pytest.mark.gpu

SIZES = [40, 8192, 8193, 70000, (1 << 20) + 77]


def _pairs(n, width, seed):
    dt = np.uint64 if width == 64 else np.uint32
    rng = np.random.default_rng(seed)
    k = rng.permutation(np.unique(rng.integers(0, np.iinfo(dt).max, n + n // 50 + 8, dtype=dt, endpoint=True))[:n])
    return k, k * dt(3) + dt(1)


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", SIZES)
def test_refused_load_leaves_the_arena(n, width):
    import paper_2604_21117_amd as g
    keys, vals = _pairs(n, width, n + width)
    t = g.Tree(keys, vals, width // 8, max_batch=1 << 14)
    before = t.arena.clone()
    bad = keys.copy()
    bad[n // 2] = bad[n // 3]
    few = keys[np.arange(n) % 5]
    for b in (bad, few):
        with pytest.raises(g.GtError) as e:
            g.tree_build(t.params, t.dev(b), t.dev(vals), t.arena)
        assert e.value.status == g.GT_ERR_DUPLICATE
        assert bool((t.arena == before).all())
    if n > 4096:
        old = g.set_sort_spin_limit(0)
        try:
            with pytest.raises(g.GtError) as e:
                g.tree_build(t.params, t.dev(keys[::-1]), t.dev(vals), t.arena)
            assert e.value.status == g.GT_ERR_DEVICE
        finally:
            g.set_sort_spin_limit(old)
        assert bool((t.arena == before).all())
    assert_export_parity(t, oracle.SortedArray(keys, vals, width))
    t.close()


@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("n", SIZES)
def test_keys_and_values_in_the_arena(n, width):
    import torch
    import paper_2604_21117_amd as g
    keys, vals = _pairs(n, width, n + width + 1)
    kb = width // 8
    p = g.make_params(kb, max_batch=1 << 14)
    arena = torch.empty(g.tree_arena_bytes(p, n, 64), dtype=torch.uint8, device="cuda")
    span = -(-n * kb // 256) * 256
    top = arena.numel() // 256 * 256
    sa = oracle.SortedArray(keys, vals, width)
    for at_k, at_v in ((0, span), (top - 2 * span, top - span), (top // 2 // 256 * 256, 0)):
        kd = arena[at_k:at_k + n * kb].view(g.key_dtype(kb))
        vd = arena[at_v:at_v + n * kb].view(g.key_dtype(kb))
        kd.copy_(g.to_device(keys))
        vd.copy_(g.to_device(vals))
        h = g.tree_build(p, kd, vd, arena)
        bits, ek, ev = oracle.check_export(g.tree_export(h), n)
        assert bits == 0 and np.array_equal(ek, sa.keys) and np.array_equal(ev, sa.vals), (at_k, at_v)
        g.tree_destroy(h)
