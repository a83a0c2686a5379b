"""A batch whose sorts take more than one chunk of key buffers (4 GiB): the rows
of every plan, and the memory, which holds one chunk at a time."""
import numpy as np
import pytest

from synth import Plan, pat

pytestmark = pytest.mark.gpu

CHUNK = 4 << 30
ROWS = 4_000_000


@pytest.mark.parametrize("top,words,plans", [(1 << 20, 1, 200), (1 << 31, 2, 100)])
def test_chunks(top, words, plans):
    import torch
    from paper_1807_01409_amd import Context
    rng = np.random.default_rng(words)
    pred = 3 if words == 1 else top + 3
    g = np.empty((ROWS, 3), dtype=np.uint32)
    g[:, 0], g[:, 1], g[:, 2] = rng.integers(1, top, ROWS), pred, rng.integers(1, top, ROWS)
    key = np.sort(g[:, 0].astype(np.uint64) << np.uint64(32) | g[:, 2])
    want = [torch.from_numpy(x.astype(np.uint32).view(np.int32)).cuda()
            for x in (key >> np.uint64(32), np.full(ROWS, pred), key & np.uint64(0xFFFFFFFF))]
    with Context(0, allocator="torch") as ctx:
        G = ctx.load(g)
        # one key word: two columns; two: three columns of 32 bits
        p = [Plan().scan(pat(f"?s {pred} ?o" if words == 1 else "?s ?p ?o", {}))] * plans
        columns = words + 1
        assert plans * ROWS * 16 * words > 2 * CHUNK
        ctx.query(G, p[0]).free()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        got = ctx.query_batch(G, p)
        ctx.synchronize()
        used = torch.cuda.max_memory_allocated() - before
        # the results and the one scan behind them, a chunk, and small buffers
        assert used < (plans + 1) * columns * ROWS * 4 + CHUNK + (1 << 29), used
        cols = [want[0], want[2]] if words == 1 else want
        for t in got:
            assert t.nrows == ROWS
            for c in range(columns):
                assert torch.equal(column(torch, t.column_ptr(c)), cols[c])
        del got


def column(torch, ptr):
    """A table's device column as a tensor."""
    class Column:
        __cuda_array_interface__ = {"shape": (ROWS,), "typestr": "<i4", "data": (ptr, False),
                                    "version": 2}
    return torch.as_tensor(Column(), device="cuda")
