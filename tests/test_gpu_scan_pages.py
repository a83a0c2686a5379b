"""GPU parity of the paged multi-pattern pass (more than four patterns, or
outputs too dense for one staged pass) against the CPU oracle: every table
must be byte-identical to the oracle's scan of its pattern."""
import numpy as np
import pytest

import oracle
from synth import Pattern, Plan, pat

pytestmark = pytest.mark.gpu


def graph(n, preds, seed, ids=5000):
    rng = np.random.default_rng(seed)
    w = np.arange(1, preds + 1) ** -1.1
    return np.stack([rng.integers(1, ids + 1, n), 1 + rng.choice(preds, n, p=w / w.sum()),
                     rng.integers(1, ids + 1, n)], axis=1).astype(np.uint32)


def patterns(k):
    some = [pat("?s 1 ?o"), pat("?s 2 ?o"), pat("?s 1 ?o", range_pos=2, lo=100, hi=2500),
            pat("? 3 ?"), pat("?s 1 7"), pat("?s ?p 9"), pat("?x 2 ?x"), pat("?s ?p ?o"),
            pat("11 ?p ?o"), pat("?s 4 ?o", range_pos=0, lo=50, hi=50), pat("?s 99 ?o"),
            pat("?o 1 ?s"), pat("? 1 ?o"), pat("?s ?p ?o", range_pos=2, lo=1, hi=1000),
            pat("?s 5 ?o"), pat("11 1 7")]
    return [some[(5 * j + k) % 16] for j in range(k)]


# one triple, tile edges (4096 triples), one tile to a range, several
@pytest.mark.parametrize("n", [1, 63, 4095, 4096, 4097, 8193, 70001, 2100007])
@pytest.mark.parametrize("k", [2, 4, 5, 9, 16])
def test_pages(ctx, n, k):
    g = graph(n, 6, n + k)
    G = ctx.load(g)
    ps = patterns(k)
    for p, t in zip(ps, ctx.scan_multi(G, ps)):
        want = oracle.scan(g, p)
        assert t.vars == want.vars
        assert t.nrows == want.rows.shape[0], (n, k, p)
        assert np.array_equal(t.to_numpy(), want.rows), (n, k, p)


def test_pages_all_rows(ctx):
    """Every triple matches: full pages, and pages shared by two tiles."""
    g = graph(1300003, 1, 3)
    G = ctx.load(g)
    ps = [pat("?s 1 ?o"), pat("?s ?p ?o"), pat("?s 1 ?o", range_pos=0, lo=1, hi=6000)]
    for p, t in zip(ps, ctx.scan_multi(G, ps)):
        assert np.array_equal(t.to_numpy(), oracle.scan(g, p).rows)


def test_pages_sets_and_filters(ctx):
    """Value sets (unions of scans) and semi-join filters in one paged pass."""
    g = graph(300007, 12, 5)
    G = ctx.load(g)
    plans = []
    for j in range(6):   # six fused unions: scans with a value set
        names = {}
        p = Plan()
        for q in (1 + j, 7, 8):
            p.scan(pat(f"?s {q} ?o", names))
        plans.append(p.union(3, j % 2 == 0))
    for j in range(3):   # stars whose two larger scans are filtered by the first
        names = {}
        p = Plan().scan(pat(f"?s {9 + j} {20 + j}", names)).scan(pat("?s 1 ?a", names))
        plans.append(p.join(names["?s"]).scan(pat("?s 2 ?b", names)).join(names["?s"]))
    old = ctx.get_option("semijoin_min")
    try:
        ctx.set_option("semijoin_min", 1)
        for p, t in zip(plans, ctx.query_batch(G, plans)):
            assert np.array_equal(t.to_numpy(), oracle.query(g, p).rows)
    finally:
        ctx.set_option("semijoin_min", old)


@pytest.mark.parametrize("n", [1, 4095, 4097, 300_007, 2_100_007])
@pytest.mark.parametrize("k", [4, 5, 16])
@pytest.mark.parametrize("top", [8191, 8192])      # the last ID of the LDS table, and the next
def test_predicates_alone(ctx, n, k, top):
    """Patterns that are a predicate each: rows of rare, common and absent
    predicates, and one pattern that puts no column out."""
    rng = np.random.default_rng(n + k)
    ids = np.concatenate([np.arange(1, 40), [top, top - 1]])
    w = np.arange(1, ids.size + 1) ** -1.0
    g = np.stack([rng.integers(1, 5000, n), rng.choice(ids, n, p=w / w.sum()),
                  rng.integers(1, 5000, n)], axis=1).astype(np.uint32)
    G = ctx.load(g)
    preds = [1, top, 3, 39, 777, 2] + [top - 1] + list(range(10, 19))
    ps = [pat("? 3 ?") if p == 3 else pat(f"?s {p} ?o") for p in preds[:k]]
    for p, t in zip(ps, ctx.scan_multi(G, ps)):
        want = oracle.scan(g, p)
        assert t.nrows == want.rows.shape[0], (n, k, p)
        assert np.array_equal(t.to_numpy(), want.rows), (n, k, p)
