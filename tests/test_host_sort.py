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
