"""The sorts of a batch round: tables of few key bits (radix passes of all their
rows together), of more bits, of several key words and of one tile, in one
batch, against numpy."""
import numpy as np
import pytest

from synth import Plan, pat

pytestmark = pytest.mark.gpu


def graph(sizes, tops, rng):
    parts = []
    for p, (n, (ts, to)) in enumerate(zip(sizes, tops), start=1):
        a = np.empty((n, 3), dtype=np.uint32)
        a[:, 0], a[:, 1], a[:, 2] = rng.integers(1, ts + 1, n), p, rng.integers(1, to + 1, n)
        parts.append(a)
    g = np.concatenate(parts)
    return g[rng.permutation(len(g))]


def plans_of(preds):
    plans, columns = [], []
    for p in preds:
        for cols in ([0], [2], [0, 2], [2, 0]):
            names = {}
            plan = Plan().scan(pat(f"?s {p} ?o", names))
            plans.append(plan.project([names["?s" if c == 0 else "?o"] for c in cols]))
            columns.append((p, cols))
    return plans, columns


SIZES = {
    "small": [1, 2, 7168, 7169, 9000],
    "middle": [100_000, 14_337, 60_001, 7168, 2],
    "large": [1_000_003, 400_000, 7169, 250_001, 3],
}


@pytest.mark.parametrize("size", list(SIZES))
@pytest.mark.parametrize("top", [1, 20, 900, 70_000, 2**31])
@pytest.mark.parametrize("partition", [False, True])
def test_batch(ctx, size, top, partition):
    rng = np.random.default_rng(top % 1000 + len(size))
    sizes = SIZES[size]
    g = graph(sizes, [(top, top)] * len(sizes), rng)
    G = ctx.load(g)
    if partition:
        G.partition()
    plans, columns = plans_of(range(1, len(sizes) + 1))
    for t, (p, cols) in zip(ctx.query_batch(G, plans), columns):
        a = g[g[:, 1] == p][:, cols]
        want = a[np.lexsort(a.T[::-1])]
        assert np.array_equal(t.to_numpy(), want), (p, cols)
    G.free()


@pytest.mark.parametrize("jobs", [2, 3, 255, 256, 257])
def test_number_of_tables(ctx, jobs):
    """The tables' order takes one bit to nine above the keys."""
    rng = np.random.default_rng(jobs)
    sizes = [7169 + 13 * (j % 50) for j in range(8)] + [200_000]
    g = graph(sizes, [(3, 60)] * len(sizes), rng)
    G = ctx.load(g)
    G.partition()
    plans, want = [], []
    for j in range(jobs):
        p = len(sizes) if j % 3 == 0 else 1 + j % len(sizes)
        names = {}
        plans.append(Plan().scan(pat(f"?s {p} ?o", names)).project([names["?o"]]))
        want.append(np.sort(g[g[:, 1] == p][:, 2]))
    for t, w in zip(ctx.query_batch(G, plans), want):
        assert np.array_equal(t.to_numpy()[:, 0], w)
    G.free()
