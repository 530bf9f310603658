"""The sort's paths that ordinary inputs do not reach, through the testing hooks:
the radix sort (kept for more than 2^26 keys) with its bounded look-back and
what a failure leaves, and the sort of a group in device memory."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_export_parity, key_set, mk_tree

pytestmark = pytest.mark.gpu


@pytest.fixture()
def g():
    import torch  # before the library: both then share torch's HIP runtime
    assert torch.cuda.is_available()
    import paper_2604_21117_amd as g
    top, group, spin = g.set_sample_sort_max(1 << 26), g.set_sample_sort_group(8192), g.set_sort_spin_limit(1 << 20)
    assert (top, group, spin) == (1 << 26, 8192, 1 << 20), "the defaults"
    yield g
    g.set_sample_sort_max(1 << 26)
    g.set_sample_sort_group(8192)
    g.set_sort_spin_limit(1 << 20)


def queries(keys, B, seed, width):
    """Mixed queries, a third of them one key (repeats keep their order)."""
    q = synth.mixed_queries(keys, B, seed, width)
    q[np.random.default_rng(seed).random(B) < 0.33] = keys[0]
    return q


def assert_all_paths(width, n, sizes):
    """Bulk load, level-wise lookups, insert and delete against the oracle."""
    keys = key_set(n, width, 5500 + width, edges=True)
    vals = synth.values_for(keys, 3, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=1 << 15, max_batch=1 << 17)
    assert_export_parity(t, sa)
    for B in sizes:
        q = queries(keys, B, B, width)
        gv, gf = t.lookup_levelwise(q)
        ov, of = sa.lookup(q)
        assert np.array_equal(gf, of) and np.array_equal(gv, ov), B
        if B > 1 << 17:
            continue
        k = queries(keys, B, B + 1, width)
        v = synth.values_for(np.arange(B, dtype=k.dtype), B, width)
        assert np.array_equal(t.insert(k, v), sa.insert(k, v)), B
        assert_export_parity(t, sa)
        k = queries(sa.items()[0], B, B + 2, width)
        assert np.array_equal(t.delete(k), sa.delete(k)), B
        assert_export_parity(t, sa)
    t.close()


@pytest.mark.parametrize("width", [32, 64])
def test_radix_sort(g, width):
    g.set_sample_sort_max(0)
    assert_all_paths(width, 60000, (8193, 12288, 50021, 300000))
    keys = key_set(30000, width, 5600)
    keys[29000] = keys[5]
    with pytest.raises(g.GtError) as e:
        mk_tree(keys, keys, width // 8)
    assert e.value.status == g.GT_ERR_DUPLICATE


def test_radix_sort_of_32_byte_keys(g):
    g.set_sample_sort_max(0)
    rng = np.random.default_rng(7)
    keys = rng.integers(0, 256, (20000, 32), dtype=np.uint8)
    keys[:, :9] = rng.integers(0, 256, (3, 9), dtype=np.uint8)[rng.integers(0, 3, 20000)]
    keys = np.unique(keys, axis=0)
    keys = keys[rng.permutation(len(keys))]
    vals = np.arange(len(keys), dtype=np.uint64)
    t = g.StaticTree(keys, vals, 32, 16)
    s = oracle.SortedBytes(keys, vals)
    bits, ek, ev = oracle.check_export(t.export(), len(keys))
    assert bits == 0 and np.array_equal(ek, s.keys) and np.array_equal(ev, s.vals)
    t.close()


@pytest.mark.parametrize("width", [32, 64])
def test_radix_sort_that_gives_up(g, width):
    """No look-back step: every tile of a pass but the first gives up at once.
    The load reports it, updates are refused, a lookup sets the error word."""
    keys = key_set(30000, width, 5700 + width)
    vals = synth.values_for(keys, 3, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=1 << 12, max_batch=1 << 14)
    before = t.export().copy()
    k = synth.uniform_keys(9000, 5701, width, exclude=keys)
    g.set_sample_sort_max(0)
    g.set_sort_spin_limit(0)
    for call in (lambda: mk_tree(keys, vals, width // 8), lambda: t.insert(k, k), lambda: t.delete(keys[:9000])):
        with pytest.raises(g.GtError) as e:
            call()
        assert e.value.status == g.GT_ERR_DEVICE
        assert np.array_equal(t.export(), before)
        assert g.tree_device_error(t.h) == g.GT_OK
    t.lookup_levelwise(k)
    assert g.tree_device_error(t.h) == g.GT_ERR_DEVICE
    g.set_sort_spin_limit(1 << 20)
    sa = oracle.SortedArray(keys, vals, width)
    assert np.array_equal(t.insert(k, k), sa.insert(k, k))
    assert_export_parity(t, sa)
    t.close()


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("n,group,sizes", [(30000, 100, (8193, 50021)), (300000, 1500, (300000,)),
                                           ((1 << 20) + 999, 400, ((1 << 20) + 5,))])
def test_groups_sorted_in_device_memory(g, width, n, group, sizes):
    g.set_sample_sort_group(group)
    assert_all_paths(width, n, sizes)
