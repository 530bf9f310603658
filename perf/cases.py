"""Performance cases of the batched B+-tree library.

What a program does with this library, through its public calls: point
lookups from one key to 2^20 keys (per query, level by level, through the
learned index, and on the static tree of 32-byte keys), range scans, batches
of updates (insert, read back, delete), and the cold start (bulk load, train
the learned index, first lookups).  Key widths 32 and 64 bits, 2^10 to 2^24
keys, uniform, clustered and sequential keys, uniform and skewed queries,
present and absent ones.

Inputs are made on the GPU from the seed.  Every key comes from a counter
through a bijection, so keys are distinct by construction: counters below n
are the tree's keys and the ones above are absent (or fresh) keys.
"""
import math

import numpy as np
import torch

import paper_2604_21117_amd as g

DEV = "cuda"
RUN = 64  # consecutive fresh keys of an update burst


# ------------------------------------------------------------------ cases

def listed():
    return [
        # one key, as an interactive request asks: call and launch latency
        dict(name="lookup_1", kind="lookup", width=64, n=1 << 24, dist="uniform", batch=1, hit=1.0, zipf=False),
        # the usual serving batch on the benchmark's tree
        dict(name="lookup_1024", kind="lookup", width=64, n=1 << 24, dist="uniform", batch=1024, hit=1.0, zipf=False),
        # a bulk probe (a join's build side already in the tree)
        dict(name="lookup_2p20", kind="lookup", width=64, n=1 << 24, dist="uniform", batch=1 << 20, hit=1.0,
             zipf=False),
        # 32-bit keys, ragged sizes, skewed queries of which half miss
        dict(name="lookup_u32_zipf", kind="lookup", width=32, n=3_000_017, dist="uniform", batch=100_003, hit=0.5,
             zipf=True),
        # the same serving batch through the trained learned index
        dict(name="learned_1000", kind="learned", width=64, n=1 << 24, dist="uniform", batch=1000, hit=1.0,
             zipf=False),
        # the level-by-level walk of a batch the library sorts itself
        dict(name="levelwise_50021", kind="levelwise", width=64, n=1 << 24, dist="uniform", batch=50_021, hit=0.9,
             zipf=False, presorted=False),
        # short scans: 1024 starts, 1 to 100 pairs each
        dict(name="range_1024", kind="range", width=64, n=1 << 24, dist="uniform", batch=1024, maxlen=100),
        # 32-byte keys (digests) on the static tree, bulk probe
        dict(name="static32_2p20", kind="static", key_bytes=32, order=32, n=10_000_000, prefix=False,
             batch=1 << 20, hit=0.9),
        # a handful of writes with their read-back
        dict(name="update_40", kind="update", width=64, n=1 << 24, dist="uniform", batch=40, upd=0.25, burst=0.0,
             fill=1.0),
        # the serving write batch
        dict(name="update_1000", kind="update", width=64, n=1 << 24, dist="uniform", batch=1000, upd=0.25,
             burst=0.25, fill=1.0),
        # a bulk ingest into a tree loaded with room for it, and the expiry of
        # the same keys
        dict(name="update_2p20", kind="update", width=64, n=1 << 24, dist="uniform", batch=1 << 20, upd=0.25,
             burst=0.0625, fill=0.75),
        # cold start: bulk load, train the learned index, first lookups
        dict(name="load_2p24", kind="load", width=64, n=1 << 24, dist="uniform", batch=1 << 20, hit=0.9, fill=1.0,
             learned=True),
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi], powers of two now
    and then."""
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.2:
        x = 1 << max(0, round(math.log2(max(x, 1))))
    return min(max(x, lo), hi)


def draw(rng):
    kind = rng.choice(["lookup", "lookup", "learned", "levelwise", "range", "static", "update", "update", "update",
                       "load"])
    c = {"kind": kind}
    if kind == "static":
        c["key_bytes"] = rng.choice([32, 32, 8])
        c["order"] = rng.choice([16, 32, 64] if c["key_bytes"] == 32 else [32, 64])
        c["n"] = _log(rng, 1 << 10, 10_000_000)
        c["prefix"] = rng.random() < 0.5
        c["batch"] = _log(rng, 1, 1 << 20)
        c["hit"] = rng.choice([0.5, 0.9, 1.0])
        return c
    c["width"] = rng.choice([64, 64, 32])
    c["n"] = _log(rng, 1 << 10, 1 << 24 if c["width"] == 64 else 1 << 23)
    c["dist"] = rng.choice(["uniform", "clustered"] if kind == "update" else ["uniform", "clustered", "sequential"])
    if kind in ("lookup", "learned", "levelwise"):
        c["batch"] = _log(rng, 1, 1 << 20)
        c["hit"] = rng.choice([0.5, 0.9, 1.0])
        c["zipf"] = rng.random() < 0.4
        if kind == "levelwise":
            c["presorted"] = rng.random() < 0.3
    elif kind == "range":
        c["batch"] = _log(rng, 1, 1 << 15)
        c["maxlen"] = _log(rng, 1, 400)
    elif kind == "update":
        # at most a sixteenth of the tree's keys at once
        c["n"] = max(c["n"], 1 << 14)
        c["batch"] = min(_log(rng, 1, 1 << 20), c["n"] // 16)
        c["upd"] = rng.choice([0.0, 0.25, 0.5])
        c["burst"] = 0.25 if c["batch"] <= 4096 and rng.random() < 0.5 else 0.0
        # a tree that takes bulk ingests is loaded with room for them
        c["fill"] = rng.choice([1.0, 1.0, 0.75]) if c["batch"] <= 4096 else 0.75
    else:
        c["batch"] = min(_log(rng, 1 << 10, 1 << 20), c["n"])
        c["hit"] = rng.choice([0.5, 0.9, 1.0])
        c["fill"] = rng.choice([1.0, 0.75])
        c["learned"] = rng.random() < 0.5
    return c


# ----------------------------------------------------------------- inputs

def _s64(x):
    """A 64-bit constant as torch holds it (signed)."""
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _shr(z, s):
    """Logical right shift of int64 words."""
    return (z >> s) & ((1 << (64 - s)) - 1)


def _mix64(z):
    """The splitmix64 finaliser on int64 words."""
    z = (z ^ _shr(z, 30)) * _s64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _s64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _bij(x, bits, seed):
    """A bijection of [0, 2^bits) (odd multiplications and xor-shifts), bits < 63."""
    m = (1 << bits) - 1
    h = bits // 2
    z = (x + (seed * 0x9E3779B1 + 12345)) & m
    for c in (0xBF58476D1CE4E5B9, 0x94D049BB133111EB, 0xD6E8FEB86659FD93):
        z = (z * _s64(c)) & m
        z = z ^ (z >> h)
    return z


def _keys(c, counters, seed):
    """Keys (as the bits of int64 / int32) of the given counters: the counter
    fixes all but the low six bits, which are a hash of it."""
    width, dist = c["width"], c["dist"]
    hb = width - 6
    if dist == "sequential":
        high = counters + (1 << (hb - 2))
    elif dist == "clustered":
        k = hb - 24 if width == 64 else hb - 7  # 64 clusters with gaps between them
        b = _bij(counters, 6 + k, seed)
        high = ((b >> k) << (hb - 6)) | (b & ((1 << k) - 1))
    else:
        high = _bij(counters, hb, seed)
    low = _mix64(counters ^ seed) & 63
    key = (high << 6) | low
    return key if width == 64 else key.to(torch.int32)


def _values(keys, seed):
    """value = hash(key ^ seed) at the key's width."""
    v = _mix64(keys.to(torch.int64) ^ (seed * 7919 + 1))
    return v if keys.dtype == torch.int64 else v.to(torch.int32)


def _gen(seed, purpose):
    r = torch.Generator(device=DEV)
    r.manual_seed(seed * 1000 + purpose)
    return r


def _ints(count, bound, r):
    return torch.randint(0, bound, (count,), generator=r, device=DEV, dtype=torch.int64)


def _counters(c, seed):
    """Counters of a query batch: present ones (uniform, or skewed with
    probability about 1/rank) and absent ones, mixed."""
    B, n, r = c["batch"], c["n"], _gen(seed, 1)
    if c.get("zipf"):
        u = torch.rand(B, generator=r, device=DEV, dtype=torch.float64)
        present = (torch.exp(u * math.log(n)) - 1).to(torch.int64).clamp_(0, n - 1)
    else:
        present = _ints(B, n, r)
    absent = n + _ints(B, n, r)
    pick = torch.rand(B, generator=r, device=DEV) < c["hit"]
    return torch.where(pick, present, absent)


def _base(c, seed):
    """The tree's keys and values, in random key order."""
    order = torch.arange(c["n"], device=DEV, dtype=torch.int64)
    if c["dist"] == "sequential":
        order = order[torch.randperm(c["n"], generator=_gen(seed, 2), device=DEV)]
    keys = _keys(c, order, seed)
    return keys, _values(keys, seed)


def _order(keys):
    """Keys as signed numbers in the order of the unsigned ones."""
    return keys ^ (torch.iinfo(keys.dtype).min)


def _queries(c, seed):
    q = _keys(c, _counters(c, seed), seed)
    if c.get("presorted"):
        q = _order(torch.sort(_order(q)).values)
    return q


def _found(c, seed):
    """The answers of _queries: found flags and values."""
    cnt = _counters(c, seed)
    q = _keys(c, cnt, seed)
    if c.get("presorted"):
        s, at = torch.sort(_order(q))
        q, cnt = _order(s), cnt[at]
    hit = cnt < c["n"]
    v = _values(q, seed)
    return torch.where(hit, v, torch.full_like(v, -1)), hit.to(torch.uint8)


def _update(c, seed):
    """An update batch: fresh keys (some in runs of consecutive keys) and
    present ones, shuffled; the keys to read back; the keys to delete."""
    B, n, r = c["batch"], c["n"], _gen(seed, 3)
    present = int(B * c["upd"])
    runs = int((B - present) * c["burst"]) // RUN
    single = B - present - runs * RUN
    fresh = _keys(c, n + torch.arange(single, device=DEV, dtype=torch.int64), seed)
    if runs:
        start = _keys(c, n + single + torch.arange(runs, device=DEV, dtype=torch.int64), seed) & ~(RUN - 1)
        step = torch.arange(RUN, device=DEV, dtype=start.dtype)
        fresh = torch.cat([fresh, (start[:, None] + step[None, :]).reshape(-1)])
    old = _keys(c, _ints(present, n, r), seed)
    keys = torch.cat([fresh, old])[torch.randperm(B, generator=r, device=DEV)]
    values = _values(keys, seed + 1)
    # read back: half of the batch, and as many other keys, some absent
    other = _keys(c, torch.where(torch.rand(B - B // 2, generator=r, device=DEV) < 0.9, _ints(B - B // 2, n, r),
                                 2 * n + _ints(B - B // 2, n, r)), seed)
    probe = torch.cat([keys[:B // 2], other])
    gone = fresh[torch.randperm(len(fresh), generator=r, device=DEV)]
    return keys, values, probe, gone


def _ranges(c, seed):
    """Starts at present keys, no upper bound on most and another key's on a
    quarter of them, 1 to maxlen pairs each, maxlen output places per scan."""
    B, r = c["batch"], _gen(seed, 4)
    lo = _keys(c, _ints(B, c["n"], r), seed)
    other = _order(_keys(c, _ints(B, c["n"], r), seed))
    bounded = torch.rand(B, generator=r, device=DEV) < 0.25
    hi = torch.where(bounded, torch.maximum(_order(lo), other), torch.full_like(lo, torch.iinfo(lo.dtype).max))
    hi = _order(hi)
    mx = 1 + _ints(B, c["maxlen"], r)
    off = torch.arange(B, device=DEV, dtype=torch.int64) * c["maxlen"]
    return lo, hi, mx.to(torch.int32), off, B * c["maxlen"]


def _wide_keys(c, counters, seed):
    """Keys of the static tree: (rows, 4) words of 32-byte keys or 8-byte
    keys.  One word is a bijection of the counter; with `prefix` the words
    before it come from 256 stems (a shared prefix), else from a hash."""
    if c["key_bytes"] == 8:
        return _bij(counters, 62, seed)
    unique = _bij(counters, 62, seed)
    rest = [_mix64(counters * 5 + j + seed) for j in range(3)]
    if c["prefix"]:
        stem = _mix64(counters ^ seed) & 255
        words = [_mix64(stem * 3 + 1), _mix64(stem * 3 + 2), unique, rest[0]]
    else:
        words = [unique] + rest
    return torch.stack(words, 1)


# ---------------------------------------------------- states, runs, checks

class _Tree:
    """A built tree with the arena it lives in."""

    def __init__(self, params, keys, values, arena_bytes):
        self.arena = torch.empty(arena_bytes, dtype=torch.uint8, device=DEV)
        self.h = g.tree_build(params, keys, values, self.arena)

    def __del__(self):
        if getattr(self, "h", None):
            g.tree_destroy(self.h)
            self.h = None


class _Learned:
    def __init__(self, tree):
        p = g.li_params()
        self.tree = tree
        self.arena = torch.empty(g.li_arena_bytes(tree.h, p), dtype=torch.uint8, device=DEV)
        self.h = g.li_create(tree.h, p, self.arena)

    def __del__(self):
        if getattr(self, "h", None):
            g.li_destroy(self.h)
            self.h = None


def _outputs(count, dtype):
    return torch.empty(count, dtype=dtype, device=DEV), torch.empty(count, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c, s = case, {"kind": case["kind"]}
    if c["kind"] == "static":
        order = torch.arange(c["n"], device=DEV, dtype=torch.int64)
        keys, vals = _wide_keys(c, order, seed), _mix64(order ^ (seed + 17))
        s["tree"] = g.StaticTree(keys.cpu().numpy().view(np.uint8 if c["key_bytes"] == 32 else np.uint64),
                                 vals.cpu().numpy().view(np.uint64), c["key_bytes"], c["order"])
        s.update(q=_wide_keys(c, _counters(c, seed), seed), batch=c["batch"])
        return s
    kb = c["width"] // 8
    keys, vals = _base(c, seed)
    p = g.make_params(kb, fill=c.get("fill", 1.0), max_batch=max(c["batch"], 1 << 14))
    if c["kind"] == "load":
        s.update(p=p, keys=keys, vals=vals, learned=c["learned"], q=_queries(c, seed),
                 arena=torch.empty(g.tree_arena_bytes(p, c["n"], c["n"] // 32), dtype=torch.uint8, device=DEV),
                 out=_outputs(c["batch"], keys.dtype))
        return s
    # headroom for the leaves that splits take: merged leaves are not reused,
    # and a long-running program sizes its arena for that
    slack = (6 << 20 if c["batch"] <= 4096 else 24 << 20) if c["kind"] == "update" else 0
    t = s["tree"] = _Tree(p, keys, vals, g.tree_arena_bytes(p, c["n"], slack))
    if c["kind"] == "update":
        k, v, probe, gone = _update(c, seed)
        s.update(k=k, v=v, probe=probe, gone=gone, out=_outputs(c["batch"], keys.dtype),
                 st=torch.empty(c["batch"], dtype=torch.uint8, device=DEV),
                 gst=torch.empty(len(gone), dtype=torch.uint8, device=DEV))
    elif c["kind"] == "range":
        lo, hi, mx, off, total = _ranges(c, seed)
        s.update(lo=lo, hi=hi, mx=mx, off=off, ok=torch.zeros(total, dtype=keys.dtype, device=DEV),
                 ov=torch.zeros(total, dtype=keys.dtype, device=DEV),
                 cnt=torch.empty(c["batch"], dtype=torch.int32, device=DEV))
    else:
        s.update(q=_queries(c, seed), out=_outputs(c["batch"], keys.dtype))
        if c["kind"] == "learned":
            s["li"] = _Learned(t)
            g.li_train(s["li"].h)
        elif c["kind"] == "levelwise":
            s["flags"] = g.GT_LW_PRESORTED if c["presorted"] else 0
            need = g.tree_lookup_levelwise_workspace_bytes(t.h, c["batch"], s["flags"])
            s["ws"] = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)
    return s


def run(state):
    s, kind = state, state["kind"]
    if kind == "static":
        return list(s["tree"].lookup_dev(s["q"], s["batch"]))
    if kind == "lookup":
        g.tree_lookup_batch(s["tree"].h, s["q"], *s["out"])
        return list(s["out"])
    if kind == "learned":
        g.li_lookup_batch(s["li"].h, s["q"], *s["out"])
        return list(s["out"])
    if kind == "levelwise":
        g.tree_lookup_levelwise(s["tree"].h, s["q"], s["flags"], *s["out"], s["ws"])
        return list(s["out"])
    if kind == "range":
        g.tree_range_batch(s["tree"].h, s["lo"], s["hi"], s["mx"], s["off"], s["ok"], s["ov"], s["cnt"])
        return [s["cnt"], s["ok"], s["ov"]]
    if kind == "update":
        h = s["tree"].h
        g.tree_insert_batch(h, s["k"], s["v"], s["st"])
        g.tree_lookup_batch(h, s["probe"], *s["out"])
        if s["gone"].numel():
            g.tree_delete_batch(h, s["gone"], s["gst"])
        return [s["st"], *s["out"], s["gst"]]
    h = g.tree_build(s["p"], s["keys"], s["vals"], s["arena"])
    if s["learned"]:
        p = g.li_params()
        arena = torch.empty(g.li_arena_bytes(h, p), dtype=torch.uint8, device=DEV)
        li = g.li_create(h, p, arena)
        g.li_train(li)
        g.li_lookup_batch(li, s["q"], *s["out"])
        g.li_destroy(li)
    else:
        g.tree_lookup_batch(h, s["q"], *s["out"])
    g.tree_destroy(h)
    return list(s["out"])


def exact(case, seed):
    c = case
    if c["kind"] == "static":
        cnt = _counters(c, seed)
        hit = cnt < c["n"]
        v = _mix64(cnt ^ (seed + 17))
        return [torch.where(hit, v, torch.full_like(v, -1)), hit.to(torch.uint8)]
    if c["kind"] == "update":
        base, bv = _base(c, seed)
        k, v, probe, gone = _update(c, seed)
        s, at = torch.sort(_order(base))
        present = _search(s, _order(k))[1]
        bpos, bhit = _search(s, _order(probe))
        ks, kat = torch.sort(_order(k), stable=True)
        kpos, khit = _search(ks, _order(probe))  # equal keys of a batch carry equal values
        val = torch.where(khit, v[kat[kpos]], bv[at[bpos]])
        hit = khit | bhit
        return [present.to(torch.uint8), torch.where(hit, val, torch.full_like(val, -1)), hit.to(torch.uint8),
                torch.ones(len(gone), dtype=torch.uint8, device=DEV)]
    if c["kind"] == "range":
        base, bv = _base(c, seed)
        s, at = torch.sort(_order(base))
        lo, hi, mx, off, total = _ranges(c, seed)
        first = torch.searchsorted(s, _order(lo))
        last = torch.searchsorted(s, _order(hi), right=True)
        cnt = torch.minimum(mx.to(torch.int64), (last - first).clamp(min=0))
        q = torch.arange(total, device=DEV) // c["maxlen"]
        j = torch.arange(total, device=DEV) % c["maxlen"]
        live = j < cnt[q]
        pos = (first[q] + j).clamp(max=c["n"] - 1)
        zero = torch.zeros(total, dtype=base.dtype, device=DEV)
        return [cnt.to(torch.int32), torch.where(live, _order(s[pos]), zero), torch.where(live, bv[at[pos]], zero)]
    return list(_found(c, seed))


def _search(sorted_keys, keys):
    pos = torch.searchsorted(sorted_keys, keys).clamp_(max=max(len(sorted_keys) - 1, 0))
    return pos, sorted_keys[pos] == keys


# ------------------------------------------------------------------- work

def _touched(nodes, batch):
    """Expected distinct nodes of a level that `batch` uniform keys reach."""
    return nodes * -math.expm1(batch * math.log1p(-1.0 / nodes)) if nodes > 1 else 1.0


def _descent(n, order, per_leaf, batch, key_bytes):
    """Node lines of a batch's descent, leaf key lines included."""
    total, nodes = 0.0, max(1.0, n / per_leaf)
    line = order * key_bytes
    while True:
        total += _touched(nodes, batch) * line
        if nodes <= 1:
            return total
        nodes = max(1.0, nodes / order)


def work(case):
    c, n, B = case, case["n"], case["batch"]
    if c["kind"] == "static":
        kb = c["key_bytes"]
        # an inner level needs the entries' leading words, a leaf one key
        lines = _descent(n, c["order"], c["order"] - 1, B, 8)
        return {"bytes": lines + B * (kb + 8 + 1) + B * c["hit"] * (8 + kb - 8), "flops": 0}
    kb = c["width"] // 8
    per = 16 * c.get("fill", 1.0)
    look = _descent(n, 16, per, B, kb) + B * (2 * kb + 1) + B * c.get("hit", 0.95) * kb
    if c["kind"] == "range":
        pairs = B * (c["maxlen"] + 1) / 2
        return {"bytes": _descent(n, 16, per, B, kb) + pairs * 4 * kb + B * (2 * kb + 16), "flops": 0}
    if c["kind"] == "update":
        fresh = B - int(B * c["upd"])
        leaves = _touched(max(1.0, n / per), B)
        rewrite = 4 * leaves * 16 * kb  # touched leaves' keys and values, read and written
        ins = _descent(n, 16, per, B, kb) + rewrite + B * (2 * kb + 1)
        dele = _descent(n, 16, per, fresh, kb) + rewrite + fresh * (kb + 1)
        return {"bytes": look + ins + dele, "flops": 0}
    if c["kind"] == "load":
        tree = 2 * n / c["fill"] * kb * 1.07
        return {"bytes": 2 * n * kb + tree + (n * kb if c["learned"] else 0) + look, "flops": 0}
    return {"bytes": look, "flops": 0}
