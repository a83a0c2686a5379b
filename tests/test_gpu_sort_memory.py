"""Sorts with memory for row numbers (24 bytes a row beside the result) and not
for packed keys of two and more words: the rows are sorted all the same."""
import numpy as np
import pytest

from synth import Plan, pat

pytestmark = pytest.mark.gpu


class Budget:
    """Device memory of a context, at most `most` bytes of it at once."""

    def __init__(self, monkeypatch):
        import torch
        self.live, self.used, self.most, self.refused = {}, 0, None, 0
        real_alloc = torch.cuda.caching_allocator_alloc
        real_free = torch.cuda.caching_allocator_delete

        def alloc(n, *rest):
            if self.most is not None and self.used + n > self.most:
                self.refused += 1
                raise MemoryError
            p = real_alloc(n, *rest)
            self.live[p] = n
            self.used += n
            return p

        def free(p):
            self.used -= self.live.pop(p, 0)
            real_free(p)

        monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", alloc)
        monkeypatch.setattr(torch.cuda, "caching_allocator_delete", free)


@pytest.mark.parametrize("cols,words", [(3, 2), (5, 3), (7, 4)])    # 32-bit columns
@pytest.mark.parametrize("distinct", [False, True])
def test_one_table(monkeypatch, cols, words, distinct):
    from paper_1807_01409_amd import Context
    n = 1_000_000
    rng = np.random.default_rng(cols)
    rows = rng.integers(1, 1 << 32, (n, cols)).astype(np.uint32)
    rows[:, :cols - 1] = rows[rng.integers(0, 1000, n), :cols - 1]
    rows[n // 2:] = rows[:n - n // 2]
    want = rows[np.lexsort(rows.T[::-1])]
    if distinct:
        want = want[np.concatenate([[True], (want[1:] != want[:-1]).any(axis=1)])]
    mem = Budget(monkeypatch)
    with Context(0, allocator="torch") as ctx:
        t = ctx.table(rows, list(range(cols)))
        table = 4 * n * cols
        beside = max(24 * n, table if distinct else 0) + 4_000_000
        assert beside < 16 * words * n
        mem.most = mem.used + table + beside
        got = ctx.sort(t, distinct).to_numpy()
        assert mem.refused
        assert np.array_equal(got, want)
        del t


def test_batch(monkeypatch):
    from paper_1807_01409_amd import Context
    n, plans = 1_000_000, 3
    rng = np.random.default_rng(1)
    g = rng.integers(1, 1 << 32, (n, 3)).astype(np.uint32)
    want = g[np.lexsort(g.T[::-1])]
    mem = Budget(monkeypatch)
    with Context(0, allocator="torch") as ctx:
        G = ctx.load(g)
        p = [Plan().scan(pat("?s ?p ?o", {}))] * plans
        mem.most = mem.used + (plans + 1) * 12 * n + 24 * n + 4_000_000
        got = ctx.query_batch(G, p)
        assert mem.refused
        for t in got:
            assert np.array_equal(t.to_numpy(), want)
        del got, t, G
