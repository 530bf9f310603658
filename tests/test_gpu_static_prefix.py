"""Static trees of 32-byte keys that share prefixes, so that a node's deciding
word (the first in which its keys differ) is any of the four: one stem for all
keys, a few stems (nodes inside one and across two), stems of odd byte lengths.
Lookups of present keys, of keys one byte away and of foreign prefixes on both
lookup kernels, ranges and the export against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _keys(n, stems, length, rng):
    k = rng.integers(0, 256, (n, 32), dtype=np.uint8)
    stem = rng.integers(0, 256, (stems, 32), dtype=np.uint8)
    k[:, :length] = stem[rng.integers(0, stems, n), :length]
    k = np.unique(k, axis=0)
    return k[rng.permutation(len(k))]


@pytest.mark.parametrize("order", [16, 32, 64])
@pytest.mark.parametrize("stems,length", [(1, 8), (1, 24), (1, 28), (3, 16), (40, 17), (5, 30)])
def test_shared_prefixes(order, stems, length):
    import paper_2604_21117_amd as g
    rng = np.random.default_rng(order * 100 + stems * 40 + length)
    keys = _keys(20000 if length < 30 else 3000, stems, length, rng)
    vals = rng.integers(0, 1 << 63, len(keys)).astype(np.uint64)
    t = g.StaticTree(keys, vals, 32, order, fill=[1.0, 0.75][stems % 2])
    s = oracle.SortedBytes(keys, vals)
    bits, ek, ev = oracle.check_export(t.export(), len(keys))
    assert bits == 0 and np.array_equal(ek, s.keys) and np.array_equal(ev, s.vals)
    for B in (500, 9000, 300000):
        q = keys[rng.integers(0, len(keys), B)].copy()
        byte = rng.integers(0, 32, B)
        off = rng.random(B) < 0.5
        q[np.arange(B)[off], byte[off]] ^= rng.integers(1, 256, off.sum()).astype(np.uint8)
        q[:3] = np.array([[0] * 32, [255] * 32, [128] * 32], dtype=np.uint8)
        gv, gf = t.lookup(q)
        ov, of = s.lookup(q)
        assert np.array_equal(gf, of) and np.array_equal(gv, ov), B
    lo = q[:400]
    hi = q[400:800]
    mc = rng.integers(0, 40, 400).astype(np.uint32)
    gc, goff, gk, gv = t.range(lo, hi, mc)
    oc, ooff, ok, ov = s.range(lo, hi, mc)
    assert np.array_equal(gc, oc)
    for i in np.nonzero(oc)[0]:
        at = slice(int(ooff[i]), int(ooff[i] + oc[i]))
        assert np.array_equal(gk[at], ok[at]) and np.array_equal(gv[at], ov[at]), i
    t.close()
