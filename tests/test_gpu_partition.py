"""The partitioned layout's three orders at sizes where a radix pass can go
wrong (tile edges, digits of one to nine bits, one pass and several), seen
through whole-slice scans, semi-joins by index on subjects and on objects, and
sort-merge joins, against the CPU oracle: results must be byte-identical."""
import numpy as np
import pytest

import oracle
from oracle import Table as OTable
from synth import Plan, pat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8193, 70001, 1600001])
@pytest.mark.parametrize("preds,step,ids", [(1, 1, 9), (5, 1, 70000), (300, 1, 600), (600, 1, 5000),
                                            (7, 100003, 2**31)])
def test_orders(ctx, n, preds, step, ids):
    rng = np.random.default_rng(n + preds)
    w = np.arange(1, preds + 1) ** -1.2
    p = 1 + step * rng.choice(preds, n, p=w / w.sum())
    pool = rng.integers(1, ids + 1, max(4, n // 3))     # values repeat, shared by s and o
    g = np.stack([rng.choice(pool, n), p, rng.choice(pool, n)], axis=1).astype(np.uint32)
    G = ctx.load(g)
    G.partition(True)
    for q in sorted(set(p.tolist()))[:4]:
        t = pat(f"?s {q} ?o")
        assert np.array_equal(ctx.scan(G, t).to_numpy(), oracle.scan(g, t).rows)
    # a small source, looked up in (predicate, subject) and (predicate, object) order
    old = ctx.get_option("semijoin_min")
    try:
        ctx.set_option("semijoin_min", 1)
        s, o = int(g[0, 0]), int(g[0, 2])
        last = int(p.max())
        for first, second, var in ((f"?x {last} {o}", "?x 1 ?y", "?x"), (f"{s} {last} ?x", "?y 1 ?x", "?x")):
            names = {}
            plan = Plan().scan(pat(first, names)).scan(pat(second, names)).join(names[var])
            pos = 0 if var == "?x" and first.startswith("?x") else 2   # where ?x stands in both
            keep = (p == last) & (g[:, 2 - pos] == (o if pos == 0 else s))
            count = dict(zip(*(x.tolist() for x in np.unique(g[p == 1][:, pos], return_counts=True))))
            size = sum(count.get(x, 0) for x in g[keep][:, pos].tolist())
            if size < 1 << 16:   # the oracle's join is single-threaded
                assert np.array_equal(ctx.query(G, plan).to_numpy(), oracle.query(g, plan).rows)
    finally:
        ctx.set_option("semijoin_min", old)
        G.free()


@pytest.mark.parametrize("n", [4097, 8192, 8193, 60001])
@pytest.mark.parametrize("bits", [5, 9, 10, 18, 32])
def test_sort_merge_join(ctx, n, bits):
    """tid_join by sort-merge: keys of one digit's width, just above it, and 32 bits."""
    rng = np.random.default_rng(n + bits)
    hi = 2**bits - 1
    keys = rng.integers(max(1, hi - 4000), hi + 1, n // 2, dtype=np.int64)
    L = np.stack([rng.choice(keys, n // 16), rng.integers(1, 50, n // 16)], axis=1).astype(np.uint32)
    R = np.stack([rng.integers(1, 50, n), rng.integers(1, hi + 1, n, dtype=np.int64)],
                 axis=1).astype(np.uint32)
    L = L[:300]
    got = ctx.join(ctx.table(L, [0, 1]), 0, ctx.table(R, [2, 0]), 1, 2).to_numpy()
    want = oracle.join(OTable(L, [0, 1]), 0, OTable(R, [2, 0]), 1, "sortmerge").rows
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n", [4095, 12289])
@pytest.mark.parametrize("preds", [15, 16])   # with 30-bit IDs: a triple is 64 bits, or 65
@pytest.mark.parametrize("side", [0, 2])
def test_orders_widest_key(ctx, n, preds, side):
    rng = np.random.default_rng(n + preds)
    top = 2**30 - 1
    g = np.stack([rng.integers(top - 999, top + 1, n), 1 + np.arange(n) % preds,
                  rng.integers(top - 999, top + 1, n)], axis=1).astype(np.uint32)
    g[:, 2 - side] = rng.permutation(n) + 1        # one position has few IDs, one the largest
    g[0] = [top, preds, top]
    G = ctx.load(g)
    G.partition(True)
    old = ctx.get_option("semijoin_min")
    try:
        ctx.set_option("semijoin_min", 1)
        for q in (1, preds):
            t = pat(f"?s {q} ?o")
            assert np.array_equal(ctx.scan(G, t).to_numpy(), oracle.scan(g, t).rows)
        x = int(g[g[:, 1] == preds][0, 2 - side])
        names = {}
        first, second = ((f"?x {preds} {x}", "?x 1 ?y") if side == 0 else
                         (f"{x} {preds} ?x", "?y 1 ?x"))
        plan = Plan().scan(pat(first, names)).scan(pat(second, names)).join(names["?x"])
        assert np.array_equal(ctx.query(G, plan).to_numpy(), oracle.query(g, plan).rows)
    finally:
        ctx.set_option("semijoin_min", old)
        G.free()
