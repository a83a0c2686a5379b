"""Load-time ID counts on both sides of the line (1024 blocks of 256 IDs in all)
up to which the bins are summed on the host: every ID, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ids", [(256 * 1022 - 1, 255, 1), (256 * 1022, 255, 1), (255, 256 * 1023, 3),
                                 (120_000, 50, 160_000), (40_000, 40_000, 40_000)])
@pytest.mark.parametrize("where", ["host", "device"])
def test_counts(ctx, ids, where):
    import torch
    rng = np.random.default_rng(sum(ids))
    n = 250_000
    g = np.empty((n, 3), dtype=np.uint32)
    for x, top in enumerate(ids):
        g[:, x] = rng.integers(1, top + 1, n)
        for j, c in enumerate((253, 254, 255, 256, 700, 30_000)):   # counts around a byte's end
            at = min(top, 255 + j)
            g[rng.integers(0, n, c), x] = at
        g[0, x], g[-1, x] = top, 1
    source = g
    if where == "device":
        source = torch.from_numpy(g.view(np.int32)).cuda()
        torch.cuda.synchronize()
    G = ctx.load(source)
    for x, top in enumerate(ids):
        cum = np.concatenate([[0], np.cumsum(np.bincount(g[:, x], minlength=top + 2))])
        asks = np.unique(np.concatenate([np.arange(0, min(top, 700) + 2), [top, top + 1],
                                         rng.integers(0, top + 2, 3000)]))
        for i in asks.tolist():
            assert G.count(x, i, i + 1) == cum[min(i + 1, top + 2)] - cum[i], (x, i)
            assert G.count(x, 0, i) == cum[i], (x, i)
    G.free()
