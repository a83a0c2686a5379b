"""Which sort a table takes, by its rows and key bits (on the host code alone,
stand_in.py)."""
import pytest

import stand_in


def sorts(queued):
    kinds = set()
    for k in queued:
        for kind in ("row_tile_sort", "row_rank_merge", "row_merge", "radix_scatter"):
            if kind in k:
                kinds.add(kind)
    return kinds


@pytest.mark.parametrize("top,cols,rows,kinds", [
    (63, 1, 1792, {"row_tile_sort"}),                              # one small tile
    (63, 1, 1793, {"radix_scatter"}),                              # one pass
    (63, 1, 7169, {"radix_scatter"}),
    (31, 2, 300_000, {"radix_scatter"}),
    (1023, 2, 114_688, {"row_tile_sort", "row_rank_merge"}),       # two
    (1023, 2, 114_689, {"radix_scatter"}),
    (1023, 3, 300_000, {"row_tile_sort", "row_merge"}),            # three
    (1023, 3, 1 << 19, {"radix_scatter"}),
    ((1 << 32) - 1, 3, 1 << 19, {"row_tile_sort", "row_merge"}),   # two key words
])
@pytest.mark.parametrize("distinct", [0, 1])
def test_route(tmp_path, top, cols, rows, kinds, distinct):
    out = stand_in.run(tmp_path, f"""
ctx = context()
word("read_word", ctypes.c_uint32).value = {top}     # every column's maximum
t = table(ctx, {rows}, {cols})
r = ctypes.c_void_p()
done = len(kernels())
st = lib.tid_sort(ctx, t, {distinct}, ctypes.byref(r))
out = dict(st=st, error=error(ctx), queued=kernels()[done:])
""")
    assert out["st"] == 0, out["error"]
    if distinct and rows <= 7168:       # one large tile
        kinds = {"row_tile_sort"}
    assert sorts(out["queued"]) == kinds


@pytest.mark.parametrize("plans,columns,passes", [(2, 2, 0), (2, 1, 2), (64, 1, 3)])
def test_route_of_a_round(tmp_path, plans, columns, passes):
    """A round's tables of 300,000 rows with columns of 17 bits: radix passes over
    all their rows, or six merge levels."""
    out = stand_in.run(tmp_path, f"""
from types import SimpleNamespace as NS
from paper_1807_01409_amd import tid
ctx = context()
n = 1 << 20
word("read_word", ctypes.c_uint32).value = 100_000   # the largest ID
word("host_word").value = 300_000                    # every scan's rows
g = ctypes.c_void_p()
assert lib.tid_load(ctx, device(12 * n), n, 1, ctypes.byref(g)) == 0
p = NS(s=0, p=1, o=0, vs=0, vp=-1, vo=1, range_pos=-1, lo=0, hi=0)
ops = [1, 0, 5, {columns}, 1, 0][:4 + {columns}]     # SCAN, PROJECT
block = tid._Plans([NS(patterns=[p], ops=ops)] * {plans})
outs = (ctypes.c_void_p * {plans})()
done = len(kernels())
st = lib.tid_query_batch(ctx, g, ctypes.cast(block.pointers(),
                         ctypes.POINTER(ctypes.POINTER(L.tid_plan))), {plans}, outs)
out = dict(st=st, error=error(ctx), queued=kernels()[done:])
""")
    assert out["st"] == 0, out["error"]
    q = out["queued"]
    assert any("row_merge_many" in k for k in q) == (not passes), q
    assert any("rows_to_words_many" in k for k in q) == bool(passes), q
    assert sum("radix_scatter" in k for k in q) == passes, q
