"""GPU parity of the larger joins (hashed build sides, sorted and indexed ones
from 2^19 rows on, probe tiles of 2048 rows) of every kind against the CPU
oracle: results must be byte-identical."""
import numpy as np
import pytest

import oracle
from oracle import Table as OTable
from synth import Plan, pat

pytestmark = pytest.mark.gpu
SORTED = 1 << 19


def tables(nl, nr, keys, seed):
    """Two tables that share about one key in eight, and a hub key."""
    rng = np.random.default_rng(seed)
    lk, rk = rng.choice(keys, nl), rng.choice(keys, nr)
    lk[rng.random(nl) < .8] = keys[0] - 1 if keys[0] > 1 else keys[-1]   # most rows: no partner
    rk[rk == (keys[0] - 1 if keys[0] > 1 else keys[-1])] = keys[1]
    if nl > 100 and nr > 100:
        lk[:5] = keys[2]
        rk[rng.integers(0, nr, 300)] = keys[2]
    L = np.stack([rng.integers(1, 1000, nl), lk], axis=1).astype(np.uint32)
    R = np.stack([rk, rng.integers(1, 1000, nr)], axis=1).astype(np.uint32)
    return L, R


KEYS = {
    "dense": np.arange(2, 900001),                                     # index direct by key
    "sparse": np.arange(2, 900001) * 4001,                             # index by upper bits
    "top": 2**32 - 1 - np.arange(900000)[::-1],                        # up to 2^32 - 1
}


@pytest.mark.parametrize("keys", list(KEYS))
@pytest.mark.parametrize("nl,nr", [(4097, 2048), (2047, 4100), (2049, 30000), (70001, 70000),
                                   (SORTED + 5000, SORTED - 1), (SORTED + 5000, SORTED),
                                   (SORTED, SORTED + 2049), (3000, SORTED + 1), (0, 5000), (5000, 0)])
def test_kinds(ctx, keys, nl, nr):
    L, R = tables(nl, nr, KEYS[keys], nl + nr)
    gl, gr = ctx.table(L, [0, 1]), ctx.table(R, [1, 2])
    ol, orr = OTable(L, [0, 1]), OTable(R, [1, 2])
    assert np.array_equal(ctx.join(gl, 1, gr, 0, 1).to_numpy(),
                          oracle.join(ol, 1, orr, 0, "sortmerge").rows)
    if max(nl, nr) > 100000:
        kinds = ("full",) if keys == "sparse" else ("left",)
    else:
        kinds = ("left", "right", "full")
    for kind in kinds:
        if max(nl, nr) > 100000:      # the oracle's outer join is a nested loop: by numpy here
            got = ctx.join_outer(gl, 1, gr, 0, kind).to_numpy()
            inner = oracle.join(ol, 1, orr, 0, "sortmerge").rows
            lone = L[~np.isin(L[:, 1], R[:, 0])]
            rows = [inner, np.column_stack([lone, np.zeros(len(lone), np.uint32)])]
            if kind == "full":
                more = R[~np.isin(R[:, 0], L[:, 1])]
                rows.append(np.column_stack([np.zeros(len(more), np.uint32), more]))
            want = np.concatenate(rows)
            want = want[np.lexsort(want.T[::-1])]
        else:
            got = ctx.join_outer(gl, 1, gr, 0, kind, 1).to_numpy()
            if max(nl, nr) > 10000:
                continue
            want = oracle.join_outer(ol, 1, orr, 0, kind).rows
        assert np.array_equal(got, want), kind


@pytest.mark.parametrize("nl,nr", [(511, 255), (513, 257), (1 << 19, 1 << 14),
                                   ((1 << 19) + 1, (1 << 14) + 1)])
def test_rows_of_a_thread(ctx, nl, nr):
    """The last sizes with few rows to a thread, and the first with more."""
    L, R = tables(nl, nr, KEYS["dense"], nl + nr)
    got = ctx.join(ctx.table(L, [0, 1]), 1, ctx.table(R, [1, 2]), 0, 1).to_numpy()
    want = oracle.join(OTable(L, [0, 1]), 1, OTable(R, [1, 2]), 0, "sortmerge").rows
    assert np.array_equal(got, want)


def test_known_bounds_and_shared_variables(ctx):
    """Joins of scans (column bounds known), by index and by hash, and a
    natural join on two variables, in a batch."""
    rng = np.random.default_rng(8)
    n = 3_000_000
    g = np.stack([rng.integers(1, 4_000_000, n), rng.choice([1, 2, 3], n, p=[.55, .4, .05]),
                  rng.integers(1, 4_000_000, n)], axis=1).astype(np.uint32)
    g[::50, 0] = g[25, 0]      # a hub subject
    G = ctx.load(g)
    plans = []
    for a, b in ((1, 2), (2, 1), (1, 3)):
        names = {}
        plans.append(Plan().scan(pat(f"?x {a} ?y", names)).scan(pat(f"?y {b} ?z", names))
                     .join(names["?y"]))
    names = {}
    plans.append(Plan().scan(pat("?x 1 ?y", names)).scan(pat("?y 2 ?z", names)).join(names["?y"])
                 .scan(pat("?z 1 ?x", names)).join(names["?z"]))
    got = ctx.query_batch(G, plans)
    for p, t in zip(plans, got):
        want = oracle.query(g, p).rows
        assert np.array_equal(t.to_numpy(), want)
        assert np.array_equal(ctx.query(G, p).to_numpy(), want)
