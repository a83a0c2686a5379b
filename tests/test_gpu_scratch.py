"""Calls that take scratch memory where it makes them faster do without it where
there is none: loads and scans of many patterns."""
import numpy as np
import pytest

import oracle
from synth import Pattern
from test_gpu_sort_memory import Budget

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spare", [0, 300_000, 600_000, 2_000_000])
def test_load(monkeypatch, spare):
    """Memory for the graph, the extreme IDs and the bins, and `spare` bytes."""
    from paper_1807_01409_amd import Context
    rng = np.random.default_rng(5)
    n, ids = 400_000, 500_000
    g = rng.integers(1, ids, (n, 3)).astype(np.uint32)
    g[: n // 2, 1] = 7
    bins = 3 * ((ids + 255) // 256) * 1024
    mem = Budget(monkeypatch)
    with Context(0, allocator="torch") as ctx:
        mem.most = mem.used + 12 * n + 64 + 24 + bins + spare
        G = ctx.load(g)
        assert mem.refused or spare == 2_000_000
        mem.most = None
        for pos in range(3):
            cum = np.concatenate([[0], np.cumsum(np.bincount(g[:, pos], minlength=ids + 2))])
            for i in np.concatenate([[1, 7, ids - 1, ids], rng.integers(1, ids, 300)]).tolist():
                assert G.count(pos, i, i + 1) == cum[i + 1] - cum[i]
                assert G.count(pos, 0, i) == cum[i]
        del G


@pytest.mark.parametrize("k", [2, 3, 9, 16])
def test_multi(monkeypatch, k):
    """Memory for the results, not for pages."""
    from paper_1807_01409_amd import Context
    rng = np.random.default_rng(k)
    n = 5_000_000
    g = rng.integers(1, 3000, (n, 3)).astype(np.uint32)
    g[:, 1] = rng.integers(1, 40, n)
    pats = [Pattern(0, 3 + j, 0, 0, -1, 1) for j in range(k)]
    mem = Budget(monkeypatch)
    with Context(0, allocator="torch") as ctx:
        G = ctx.load(g)
        cnt = np.bincount(g[:, 1], minlength=64)
        mem.most = mem.used + sum(2 * (int(cnt[3 + j]) * 4 + 256) for j in range(k)) + 1_000_000
        got = ctx.scan_multi(G, pats)
        assert mem.refused
        for p, t in zip(pats, got):
            assert np.array_equal(t.to_numpy(), oracle.scan(g, p).rows)
        del got, t, G
