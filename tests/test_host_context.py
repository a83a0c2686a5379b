"""What a context allocates (on the host code alone, stand_in.py)."""
import stand_in


def test_one_pinned_block_until_something_is_read(tmp_path):
    """The error flags and the first tables' count words are one allocation: each
    costs more than a small call."""
    out = stand_in.run(tmp_path, """
ctx = context()
made = word("pinned").value
ts = [table(ctx, 5, 2) for _ in range(100)]
out = dict(made=made, tables=word("pinned").value, copies=word("copies").value)
""")
    assert (out["made"], out["tables"]) == (1, 1)
