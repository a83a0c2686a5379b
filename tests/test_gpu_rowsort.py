"""GPU parity of the packed-key row sort (one to four key words, one tile,
several tiles and merge levels, and the wider rows left to the radix sort)
against the CPU oracle: results must be byte-identical."""
import numpy as np
import pytest

import oracle
from oracle import Table as OTable

pytestmark = pytest.mark.gpu

MAX = 2**32 - 1
# column bounds: the key of 1, 2, 3, 4 and 5 words (the last one is too wide)
SCHEMAS = {
    "1 word, one column": [50],
    "1 word, a zero column": [1000, 0, 7],
    "1 word, all 64 bits": [MAX, MAX],
    "2 words, a column across them": [2**25, 2**25, 2**25],
    "2 words, all 128 bits": [MAX] * 4,
    "3 words": [2**25] * 7,
    "4 words": [2**31 - 1] * 8,
    "5 words": [MAX] * 9,
}


@pytest.mark.parametrize("n", [2, 7, 8, 447, 1791, 1792, 1793, 3584, 3585, 7168, 7169, 14336, 14337,
                               30011])
@pytest.mark.parametrize("schema", list(SCHEMAS))
def test_row_sort(ctx, schema, n):
    hi = SCHEMAS[schema]
    rng = np.random.default_rng(n + len(hi))
    rows = np.stack([rng.integers(0, h + 1, n, dtype=np.int64) for h in hi], axis=1)
    rows[0] = hi                       # the bounds are reached
    if n > 20:                         # repeated rows, the largest key among them
        rows[n // 2:n // 2 + n // 8] = hi
        rows[n // 8:n // 4] = rows[1]
        rows[-3:] = 0
    rows = rows.astype(np.uint32)
    t, ot = ctx.table(rows, list(range(len(hi)))), OTable(rows, list(range(len(hi))))
    got = ctx.sort(t, False)
    assert got.nrows == n
    assert np.array_equal(got.to_numpy(), oracle.sort_rows(ot).rows)
    assert np.array_equal(ctx.sort(t, True).to_numpy(), oracle.distinct(ot).rows)


@pytest.mark.parametrize("n", [14335, 14336, 14337, 14592, 114688, 114689])
@pytest.mark.parametrize("schema", ["1 word, one column", "1 word, all 64 bits",
                                    "2 words, a column across them", "3 words", "4 words"])
@pytest.mark.parametrize("kind", ["random", "sorted", "reversed", "apart", "one"])
def test_rank_merge(ctx, schema, n, kind):
    """Runs that interleave, follow one another (their parts of another run are
    empty or, out of order, all of it, more than fits LDS) or are all equal."""
    hi = np.array(SCHEMAS[schema], dtype=np.int64)
    rng = np.random.default_rng(n)
    u = rng.random(n)
    if kind == "sorted":
        u = np.sort(u)
    elif kind == "reversed":
        u = np.sort(u)[::-1]
    elif kind == "apart":   # a run of large rows among runs of small ones
        u = np.where((np.arange(n) // 1792) % 8 == 3, 0.9 + u / 20, u / 1000)
        u[::256] = 1.0
    elif kind == "one":
        u[:] = 0.5
    rows = np.minimum((u[:, None] * (hi + 1)).astype(np.int64), hi)
    rows[0] = hi
    rows = rows.astype(np.uint32)
    t, ot = ctx.table(rows, list(range(len(hi)))), OTable(rows, list(range(len(hi))))
    assert np.array_equal(ctx.sort(t, False).to_numpy(), oracle.sort_rows(ot).rows)
    assert np.array_equal(ctx.sort(t, True).to_numpy(), oracle.distinct(ot).rows)


@pytest.mark.parametrize("n", [114689, 116480, 116481, 229377, 300007])
@pytest.mark.parametrize("schema", ["1 word, all 64 bits", "2 words, a column across them",
                                    "3 words", "4 words"])
@pytest.mark.parametrize("rows_each", [1.0, 2.5, 3000])
def test_distinct_of_merged(ctx, schema, n, rows_each):
    """DISTINCT in the last merge level: equal rows within a tile, over tile
    edges and over several tiles."""
    hi = np.array(SCHEMAS[schema], dtype=np.int64)
    rng = np.random.default_rng(n)
    pool = rng.integers(0, hi + 1, (max(1, int(n / rows_each)), hi.size), dtype=np.int64)
    rows = pool[rng.integers(0, len(pool), n)] if rows_each > 1 else pool
    rows[0] = hi
    rows = rows.astype(np.uint32)
    t, ot = ctx.table(rows, list(range(len(hi)))), OTable(rows, list(range(len(hi))))
    assert np.array_equal(ctx.sort(t, True).to_numpy(), oracle.distinct(ot).rows)


@pytest.mark.parametrize("dedupe", [False, True])
def test_union_of_many(ctx, dedupe):
    """More columns than one launch copies; empty tables; variables that only some have."""
    rng = np.random.default_rng(5)
    ts, ots = [], []
    for j in range(90):
        vs = [[0, 1], [1, 2], [2], [0, 1, 2]][j % 4]
        rows = rng.integers(1, 50, (int(rng.integers(0, 3)) * j * 7 % 1100, len(vs)),
                            dtype=np.int64).astype(np.uint32)
        ts.append(ctx.table(rows, vs))
        ots.append(OTable(rows, vs))
    got, want = ctx.union(ts, dedupe), oracle.union(ots, dedupe)
    assert np.array_equal(got.to_numpy(), want.rows)


@pytest.mark.parametrize("n,hi", [
    ((1 << 19) - 1, [2**15 - 1, 2**15 - 1]),   # the last size that is merged
    (1 << 19, [2**15 - 1, 2**15 - 1]),         # three radix passes
    (1 << 19, [1]),                            # one bit
    (600_011, [2**20 - 1, 0, 2**20 - 1]),      # four passes of ten bits
    ((3 << 20) + 5, [2**23 - 1, 2**23 - 1]),   # five passes
])
@pytest.mark.parametrize("repeat", [False, True])
def test_radix_of_packed_rows(ctx, n, hi, repeat):
    rng = np.random.default_rng(n)
    rows = np.stack([rng.integers(0, h + 1, n, dtype=np.int64) for h in hi], axis=1)
    if repeat:
        rows = rows[rng.integers(0, n // 3, n)]
    rows[-1] = hi
    rows = rows.astype(np.uint32)
    key = np.zeros(n, dtype=np.uint64)
    for c, h in enumerate(hi):
        key = key << np.uint64(int(h).bit_length()) | rows[:, c].astype(np.uint64)
    order = np.argsort(key, kind="stable")
    t = ctx.table(rows, list(range(len(hi))))
    assert np.array_equal(ctx.sort(t, False).to_numpy(), rows[order])
    first = np.concatenate([[True], key[order][1:] != key[order][:-1]])
    assert np.array_equal(ctx.sort(t, True).to_numpy(), rows[order][first])
