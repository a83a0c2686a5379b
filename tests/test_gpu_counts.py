"""The load-time ID counts (one byte an ID, a list of the counts of 255 and
more, 64 IDs to a block) against numpy: every single ID, and ranges that start
and end inside blocks and past the largest ID."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ids", [1, 62, 63, 64, 65, 127, 128, 300])
@pytest.mark.parametrize("hubs", [False, True])
def test_counts(ctx, ids, hubs):
    rng = np.random.default_rng(ids + hubs)
    # counts around the byte's limit, some IDs absent; with hubs whole blocks of them
    cnt = rng.choice([0, 1, 2, 253, 254, 255, 256, 700], ids,
                     p=[.3, .3, .2, .04, .04, .04, .04, .04])
    if hubs:
        cnt[: max(1, ids // 2)] += 255
    cnt[-1] = max(cnt[-1], 1)
    col = rng.permutation(np.repeat(np.arange(1, ids + 1), cnt))
    n = col.size
    other = rng.integers(1, 40, n)
    for pos in range(3):
        g = np.stack([other] * 3, axis=1).astype(np.uint32)
        g[:, pos] = col
        G = ctx.load(g)
        cum = np.concatenate([[0, 0], np.cumsum(cnt)])   # cum[i]: IDs below i
        for i in range(ids + 1):
            assert G.count(pos, i, i + 1) == cum[i + 1] - cum[i], (pos, i)
        for _ in range(40):
            lo, hi = (int(x) for x in rng.integers(0, ids + 70, 2))
            want = cum[min(hi, ids + 1)] - cum[min(lo, ids + 1)] if hi > lo else 0
            assert G.count(pos, lo, hi) == want, (pos, lo, hi)
        G.free()
