"""Sizes that the library refuses, on the host code alone (stand_in.py: no GPU,
no memory behind the tables)."""
import pytest

import stand_in

MOST_BUILD = 1 << 30    # rows of a join's build side


@pytest.mark.parametrize("call", ["inner", "left", "right", "full"])
@pytest.mark.parametrize("extra", [0, 1, (1 << 32) - 1 - MOST_BUILD])
def test_hash_join_build_side(tmp_path, call, extra):
    """A hash join's build side (the smaller side of an inner join, the other
    side of a one-sided one) has at most 2^30 rows."""
    out = stand_in.run(tmp_path, f"""
ctx = context()
most = {MOST_BUILD} + {extra}
small = most if "{call}" == "inner" else 1000
swap = "{call}" == "right"
l = table(ctx, most if swap else small, 1, 0)
r = table(ctx, small if swap else most, 1, 0)
t = ctypes.c_void_p()
if "{call}" == "inner":
    st = lib.tid_join(ctx, l, 0, r, 0, 1, ctypes.byref(t))
else:
    kind = ["inner", "left", "right", "full"].index("{call}")
    st = lib.tid_join_outer(ctx, l, 0, r, 0, kind, 1, ctypes.byref(t))
out = dict(st=st, error=error(ctx), kernels=kernels())
""")
    if extra:
        assert (out["st"], "build side" in out["error"]) == (-4, True), out["error"]
        assert not [k for k in out["kernels"] if "index_runs" in k]
    else:
        assert out["st"] == 0, out["error"]


def test_full_join_without_right_rows(tmp_path):
    """No R row can be without a partner: nothing is built over L, of any size."""
    out = stand_in.run(tmp_path, f"""
ctx = context()
l, r = table(ctx, {MOST_BUILD} + 1), table(ctx, 0)
t = ctypes.c_void_p()
out = dict(st=lib.tid_join_outer(ctx, l, 0, r, 0, 3, 1, ctypes.byref(t)), error=error(ctx),
           kernels=kernels())
""")
    assert out["st"] == 0, out["error"]
    assert not [k for k in out["kernels"] if "index_runs" in k or "big_insert" in k]
