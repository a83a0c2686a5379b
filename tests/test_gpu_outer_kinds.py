"""Outer joins of every kind above 10,000 rows, over several probe tiles, hashed
and sorted build sides, against numpy."""
import numpy as np
import pytest

import oracle
from oracle import Table as OTable
from test_gpu_big_join import KEYS, SORTED, tables

pytestmark = pytest.mark.gpu


def expected(L, R, kind):
    """Rows over L's columns, then R's without its key, in lexicographic order."""
    inner = oracle.join(OTable(L, [0, 1]), 1, OTable(R, [1, 2]), 0, "sortmerge").rows
    rows = [inner]
    if kind in ("left", "full"):
        lone = L[~np.isin(L[:, 1], R[:, 0])]
        rows.append(np.column_stack([lone, np.zeros(len(lone), np.uint32)]))
    if kind in ("right", "full"):
        lone = R[~np.isin(R[:, 0], L[:, 1])]
        rows.append(np.column_stack([np.zeros(len(lone), np.uint32), lone]))
    want = np.concatenate(rows)
    return want[np.lexsort(want.T[::-1])]


@pytest.mark.parametrize("kind", ["left", "right", "full"])
@pytest.mark.parametrize("keys", list(KEYS))
@pytest.mark.parametrize("nl,nr", [(2049, 30_000), (30_000, 2049), (70_001, 70_000),
                                   (3000, SORTED + 1), (SORTED + 1, 3000),
                                   (SORTED + 2049, SORTED)])
@pytest.mark.parametrize("algo", [0, 1, 2])
def test_kind(ctx, keys, nl, nr, kind, algo):
    L, R = tables(nl, nr, KEYS[keys], nl + nr)
    got = ctx.join_outer(ctx.table(L, [0, 1]), 1, ctx.table(R, [1, 2]), 0, kind, algo)
    assert np.array_equal(got.to_numpy(), expected(L, R, kind))
