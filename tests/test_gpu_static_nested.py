"""Static trees of 32-byte keys whose deciding word changes several times on
the way down: word 0 takes 3 values, word 1 five under each, word 2 seven under
each of those, word 3 differs.  Both lookup kernels, with present keys and keys
that leave the tree at any word, ranges from such keys, and the export."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _nested(n, rng):
    words = rng.integers(0, 1 << 63, (n, 4), dtype=np.uint64)
    at = np.zeros(n, dtype=np.int64)
    for w, kinds in enumerate((3, 5, 7)):
        at = at * kinds + rng.integers(0, kinds, n)
        words[:, w] = rng.integers(0, 1 << 63, 3 * 5 * 7, dtype=np.uint64)[at]
    k = np.unique(words.astype(">u8").view(np.uint8).reshape(n, 32), axis=0)
    return k[rng.permutation(len(k))]


@pytest.mark.parametrize("order", [16, 32, 64])
@pytest.mark.parametrize("n", [200, 5000, 60000])
def test_nested_prefixes(order, n):
    import paper_2604_21117_amd as g
    rng = np.random.default_rng(order + n)
    keys = _nested(n, rng)
    vals = rng.integers(0, 1 << 63, len(keys)).astype(np.uint64)
    t = g.StaticTree(keys, vals, 32, order)
    s = oracle.SortedBytes(keys, vals)
    bits, ek, ev = oracle.check_export(t.export(), len(keys))
    assert bits == 0 and np.array_equal(ek, s.keys) and np.array_equal(ev, s.vals)
    for B in (1, 3, 777, 8192):
        q = keys[rng.integers(0, len(keys), B)].copy()
        off = rng.random(B) < 0.4
        q[np.arange(B)[off], 8 * rng.integers(0, 4, B)[off] + 7] ^= 1
        gv, gf = t.lookup(q)
        ov, of = s.lookup(q)
        assert np.array_equal(gf, of) and np.array_equal(gv, ov), B
        lo, hi = q[:400], keys[rng.integers(0, len(keys), min(B, 400))]
        mc = rng.integers(0, 100, len(lo)).astype(np.uint32)
        gc, _, gk, gv = t.range(lo, hi, mc)
        oc, ooff, ok, ov = s.range(lo, hi, mc)
        assert np.array_equal(gc, oc), B
        for i in np.nonzero(oc)[0]:
            at = slice(int(ooff[i]), int(ooff[i] + oc[i]))
            assert np.array_equal(gk[at], ok[at]) and np.array_equal(gv[at], ov[at]), (B, i)
    t.close()
