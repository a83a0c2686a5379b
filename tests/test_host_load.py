"""What a load queues (on the host code alone, stand_in.py)."""
import pytest

import stand_in

LOAD = """
ctx = context()
n = {n}
word("read_word", ctypes.c_uint32).value = {ids}     # smallest and largest ID, and every count
word("host_word").value = 0
host = (ctypes.c_uint32 * (3 * n))()
g = ctypes.c_void_p()
done = len(kernels())
st = lib.tid_load(ctx, {source}, n, {device}, ctypes.byref(g))
out = dict(st=st, error=error(ctx), queued=kernels()[done:])
"""


@pytest.mark.parametrize("device", [0, 1])
@pytest.mark.parametrize("ids,packed", [(3, False), (5000, False), (87_000, False),
                                        (87_500, True), (200_000, True)])
def test_small_tables_of_counts_are_not_packed(tmp_path, device, ids, packed):
    """Up to 1024 blocks of 256 IDs (three positions) the bins go to the host as
    they are: one copy, after the extreme IDs'."""
    source = "device(12 * n)" if device else "host"
    out = stand_in.run(tmp_path, LOAD.format(n=1000, ids=ids, device=device, source=source))
    assert out["st"] == 0, out["error"]
    q = out["queued"]
    assert any("pack_counts" in k for k in q) == packed, q
    assert q.count("copy down") == (4 if packed else 2), q
    if not packed:
        assert sum(k not in ("copy up", "copy down") for k in q) == 3, q
    if not device:      # host triples are copied before anything is launched
        assert q[0] == "copy up", q


def test_counts_without_memory_to_pack_them(tmp_path):
    code = LOAD.format(n=1000, ids=2_000_000, device=1, source="source").replace(
        "done =", """source = device(12 * n)
bins = 3 * ((2000001 + 255) // 256) * 1024
word("most_bytes").value = word("live_bytes").value + (1 << 25) + 65536 * 2   # the bins' block
done =""")
    out = stand_in.run(tmp_path, code)
    assert out["st"] == 0, out["error"]
    assert not any("pack_counts" in k for k in out["queued"])
