"""Host tables that a join copies to the device are left as they are until the
stream has been waited for (on the host code alone, stand_in.py)."""
import pytest

import stand_in


@pytest.mark.parametrize("kind", ["inner", "left", "right", "full"])
@pytest.mark.parametrize("rows", [500, 600_000])      # a hashed and a sorted build side
def test_join_tables_outlive_their_copies(tmp_path, kind, rows):
    out = stand_in.run(tmp_path, f"""
word("host_word").value = 5000       # every count and total that the host reads
ctx = context()
l, r = table(ctx, {rows} + 7, 2, 0), table(ctx, {rows}, 2, 1)
kind = ["inner", "left", "right", "full"].index("{kind}")
st = 0
for _ in range(3):
    t = ctypes.c_void_p()
    st = st or lib.tid_join_outer(ctx, l, 1, r, 0, kind, 1, ctypes.byref(t))
st = st or lib.tid_ctx_synchronize(ctx)
out = dict(st=st, error=error(ctx), copies=word("copies").value, changed=word("changed").value,
           kernels=kernels())
""")
    assert out["st"] == 0, out["error"]
    assert any("big_expand" in k for k in out["kernels"]) and out["copies"] >= 6
    assert out["changed"] == 0
