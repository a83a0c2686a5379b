"""Dictionary encoding of byte strings on the device: lengths around the
eight-byte words that the kernels read, any alignment, strings that differ in
one byte, one term in every place of a wave, the string whose FNV-1a hash is 0,
offsets that are not aligned, rows over the input's own memory, and offsets
that fall or pass the bytes."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ZERO = bytes([0xd5, 0x6b, 0xb9, 0x53, 0x42, 0x87, 0x08, 0x36])  # FNV-1a, 64 bits: 0


def terms_of(kind, n, rng):
    if kind == "lengths":     # 0 to 24 bytes, one of three last bytes
        return [bytes(rng.integers(65, 67, int(k), dtype=np.uint8)) + bytes([c])
                for k, c in zip(rng.integers(0, 24, 3 * n), rng.integers(0, 3, 3 * n))] + [b""]
    if kind == "one":
        return [b"the same term"]
    if kind == "distinct":
        return [b"%d" % (7 * i) for i in range(3 * n)]
    return [ZERO, b"", b"a", ZERO + b"x"]


def call_encode(ctx, torch, blob, off, n, rows):
    """blob, off, rows: device tensors"""
    out = ctypes.c_void_p()
    st = ctx._lib.tid_encode(ctx.ptr, ctypes.c_void_p(blob.data_ptr()), blob.numel(),
                             ctypes.c_void_p(off.data_ptr()), n, 1,
                             ctypes.c_void_p(rows.data_ptr()), ctypes.byref(out))
    return st, out


@pytest.mark.parametrize("kind,n", [("lengths", 1), ("lengths", 21), ("lengths", 5000),
                                    ("one", 22), ("one", 30_000), ("distinct", 86),
                                    ("distinct", 50_000), ("zero", 700)])
@pytest.mark.parametrize("place", ["apart", "unaligned", "over"])
def test_encode_bytes(ctx, kind, n, place):
    import torch
    from paper_1807_01409_amd.tid import Dict
    rng = np.random.default_rng(n)
    pool = terms_of(kind, n, rng)
    pick = (np.arange(3 * n) if kind == "distinct" else rng.integers(0, len(pool), 3 * n))
    terms = [pool[i] for i in pick]
    off = np.zeros(3 * n + 1, dtype=np.uint64)
    off[1:] = np.cumsum([len(t) for t in terms])
    blob = np.frombuffer(b"".join(terms) + b"tail", dtype=np.uint8)[:max(1, int(off[-1]))].copy()
    dev = torch.from_numpy(blob).cuda()
    if place == "unaligned":
        mem = torch.zeros(8 * (3 * n + 1) + 4, dtype=torch.uint8, device="cuda")
        o = mem[4:]
        o.copy_(torch.from_numpy(off.view(np.uint8)))
    else:
        o = torch.from_numpy(off.view(np.int64)).cuda()
    rows = (o.view(torch.int32) if place == "over"
            else torch.zeros(3 * n, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    st, h = call_encode(ctx, torch, dev, o, n, rows)
    assert st == 0
    d = Dict(ctx, h)
    ids = {}
    want = [ids.setdefault(t, len(ids) + 1) for t in terms]
    got = rows[:3 * n].cpu().numpy().view(np.uint32)
    assert np.array_equal(got, np.array(want, dtype=np.uint32))
    assert d.info() == (len(ids), sum(map(len, ids)))
    back = np.arange(1, len(ids) + 1, dtype=np.uint32)
    at = np.zeros(len(ids) + 1, dtype=np.uint64)
    text = np.zeros(sum(map(len, ids)) + 1, dtype=np.uint8)
    st = ctx._lib.tid_decode(ctx.ptr, d._p, back.ctypes.data_as(ctypes.c_void_p), len(ids), 0,
                             at.ctypes.data_as(ctypes.c_void_p),
                             text.ctypes.data_as(ctypes.c_void_p), text.size)
    assert st == 0
    raw = text.tobytes()
    assert [raw[int(a):int(b)] for a, b in zip(at, at[1:])] == list(ids)


@pytest.mark.parametrize("where", [0, 63, 299])
@pytest.mark.parametrize("how", ["fall", "past"])
def test_bad_offsets(ctx, how, where):
    import torch
    n = 100
    off = np.arange(301, dtype=np.int64) * 2
    if how == "fall":
        off[where + 1] = off[where] - 1 if where else -1  # as unsigned: past every byte
        off[where + 1:where + 2] = np.maximum(off[where + 1], 0) if where else 0
        off[where] += 1
    else:
        off[where + 1:] += 10_000
    blob = torch.zeros(600, dtype=torch.uint8, device="cuda")
    rows = torch.zeros(300, dtype=torch.int32, device="cuda")
    o = torch.from_numpy(off).cuda()
    torch.cuda.synchronize()
    st, _ = call_encode(ctx, torch, blob, o, n, rows)
    assert st == -1
    text = ctx._lib.tid_last_error(ctx.ptr).decode()
    assert ("fall" if how == "fall" else "past") in text
    st, _ = call_encode(ctx, torch, blob, torch.arange(0, 602, 2, device="cuda"), n, rows)
    assert st == 0      # the flags of a refused call do not outlive it
