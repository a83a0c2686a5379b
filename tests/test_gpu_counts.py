"""The load-time ID counts (one byte an ID, a list of the counts of 255 and
more, in blocks) against numpy: every single ID, and ranges that start
and end inside blocks and past the largest ID."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ids", [1, 63, 64, 65, 128, 254, 255, 256, 257, 300, 511, 512, 600])
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


@pytest.mark.parametrize("n,ids", [
    ((1 << 18) - 1, (40, 8192, 8191)),                 # the last size counted with atomics
    (1 << 18, (8190, 8191, 8192)),                     # IDs counted in LDS at every position
    (1 << 18, (8192, 100, 32766)),                     # one bucket, nearly full
    (1 << 18, (32767, 32768, 65535)),                  # one bucket full, two buckets
    (300_001, (1_000_003, 90_000, 5)),                 # three kinds at once
    (4096 * 77 + 1, (70_000, 12, (1 << 24) - 1)),      # as many buckets as there may be
    (270_000, (1 << 24, 3, 50)),                       # one more
    (2 * (1 << 22), (1 << 24, 3, 50)),                 # in two passes
    (3 * (1 << 22) + 1, (40_000_000, 9000, 20_000_000)),    # three passes, one and two
    (3_000_000, (200_000, 50, 600_000)),
])
@pytest.mark.parametrize("hub", [0.0, 0.7])
def test_counts_split(ctx, n, ids, hub):
    import torch
    rng = np.random.default_rng(n)
    g = np.empty((n, 3), dtype=np.uint32)
    for x in range(3):
        g[:, x] = rng.integers(1, ids[x] + 1, n)
        if hub:     # most triples have one ID, the last of a bucket if there is one
            g[rng.random(n) < hub, x] = min(ids[x], 32767)
        g[0, x], g[-1, x] = ids[x], 1
    t = torch.from_numpy(g.view(np.int32)).cuda()
    torch.cuda.synchronize()
    G = ctx.load(t)
    for x in range(3):
        cum = np.concatenate([[0], np.cumsum(np.bincount(g[:, x], minlength=ids[x] + 1))])
        near = [v for b in range(0, ids[x] + 1, 32768) for v in (b - 1, b, b + 1)]
        pick = np.concatenate([[1, ids[x]], near, rng.integers(1, ids[x] + 1, 300)])
        for v in pick[(pick >= 1) & (pick <= ids[x])]:
            assert G.count(x, int(v), int(v) + 1) == cum[v + 1] - cum[v], (x, v)
        for lo, hi in rng.integers(1, ids[x] + 2, (100, 2)):
            want = cum[hi] - cum[lo] if hi > lo else 0
            assert G.count(x, int(lo), int(hi)) == want, (x, lo, hi)
    G.free()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 1023, 1024, 262143, 800_001, 800_002, 800_003])
@pytest.mark.parametrize("skip", [0, 1, 4])     # triples before: 12 bytes off, and 48
def test_device_triples(ctx, n, skip):
    """Triples copied from device memory: every row, the largest IDs, and ID 0
    refused at either end."""
    import torch
    from paper_1807_01409_amd import TidError
    rng = np.random.default_rng(n)
    g = rng.integers(1, 5000, (n + skip, 3)).astype(np.uint32)
    top = 70_000 + np.arange(3)
    for x in range(3):
        g[skip + (n - 1) * (x + 1) // 3, x] = top[x]
    t = torch.from_numpy(g.view(np.int32)).cuda()[skip:]
    torch.cuda.synchronize()
    G = ctx.load(t)
    from synth import pat
    assert np.array_equal(ctx.scan(G, pat("?s ?p ?o")).to_numpy(), g[skip:])
    for x in range(3):
        assert G.count(x, int(top[x]), int(top[x]) + 1) == 1
        assert G.count(x, 1, 1 << 20) == n
    G.free()
    for row, col in ((0, 0), (n - 1, 2), (n - 1, 1)):
        bad = t.clone()
        bad[row, col] = 0
        torch.cuda.synchronize()
        with pytest.raises(TidError):
            ctx.load(bad)
