"""Delete batches of 65 to 2048 keys in which keys occur many times: a key's
repeats keep records of their own, and a leaf's keys lie between them."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_export_parity, key_set, mk_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("B", [65, 300, 2048])
def test_repeats_between_the_keys_of_a_leaf(width, B):
    keys = key_set(5000, width, 91 + width, edges=True)
    vals = synth.values_for(keys, 92, width)
    sa = oracle.SortedArray(keys, vals, width)
    t = mk_tree(keys, vals, width // 8, leaf_slack=1 << 10, max_batch=1 << 12)
    order = np.sort(keys)
    absent = synth.uniform_keys(500, 93, width, exclude=keys)
    rng = np.random.default_rng(B)
    for near, heavy, few in ((40, 1, 3), (200, 2, 1), (16, 16, 40), (900, 5, 2), (1, 1, 1)):
        at = int(rng.integers(0, len(order) - 1000))
        pool = np.concatenate([order[at:at + near], absent[:few]])  # neighbours, some of them gone already
        k = pool[rng.integers(0, len(pool), B)]
        hot = rng.choice(pool, heavy)
        k = np.where(rng.random(B) < 0.8, hot[rng.integers(0, heavy, B)], k)
        assert np.array_equal(t.delete(k), sa.delete(k))
        assert_export_parity(t, sa)
    t.close()


def test_repeats_take_no_longer():
    """2048 times one key within 1.4 times the time of 2048 keys (0.9 measured;
    2.2 when every repeat was walked)."""
    import torch
    import paper_2604_21117_amd as g
    keys = key_set(1 << 20, 64, 94)
    t = mk_tree(keys, keys, 8, leaf_slack=1 << 17, max_batch=1 << 12, fill=0.75)
    st = torch.empty(2048, dtype=torch.uint8, device="cuda")
    us = {}
    for name, k in (("one", np.repeat(keys[:1], 2048)), ("all", keys[:2048])):
        k = t.dev(k)
        times = []
        for _ in range(15):
            g.tree_insert_batch(t.h, k, k, st)
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.tree_delete_batch(t.h, k, st)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1000)
        us[name] = min(times)
    assert us["one"] < 1.4 * us["all"], us
    t.close()
