"""Sorts of tables whose rows have few key bits, one or two radix passes, on both
sides of the sizes where those are taken: against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def table(rng, n, cols, top, kind):
    a = rng.integers(0 if kind == "zeros" else 1, top + 1, (n, cols)).astype(np.uint32)
    if kind == "one":
        a[:] = top
    a[n // 2] = top
    return a


@pytest.mark.parametrize("n", [1792, 1793, 4000, 7168, 7169, 8960, 16_001, 114_688, 114_689, 200_003, 524_288])
@pytest.mark.parametrize("cols,top", [(1, 1), (1, 1023), (1, 1024), (2, 31), (2, 1023), (3, 127),
                                      (10, 1)])
@pytest.mark.parametrize("kind", ["any", "zeros", "one"])
def test_sort(ctx, n, cols, top, kind):
    rng = np.random.default_rng(n + cols + top)
    a = table(rng, n, cols, top, kind)
    want = a[np.lexsort(a.T[::-1])]
    t = ctx.table(a, list(range(cols)))
    assert np.array_equal(ctx.sort(t).to_numpy(), want)
    keep = np.concatenate([[True], (want[1:] != want[:-1]).any(axis=1)])
    assert np.array_equal(ctx.sort(t, True).to_numpy(), want[keep])
