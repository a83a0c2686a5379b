"""A term of 2^32 bytes or more is refused: lengths are kept as 32-bit words."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

WIDE = 1 << 32


@pytest.mark.parametrize("where", [0, 1, 2])
def test_long_term(ctx, where):
    import torch
    blob = torch.zeros(WIDE + 64, dtype=torch.uint8, device="cuda")
    ends = [0, 5, 9, 12]
    off = [e if i <= where else e + WIDE for i, e in enumerate(ends)]
    o = torch.tensor(off, dtype=torch.int64, device="cuda")
    rows = torch.zeros(3, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    out = ctypes.c_void_p()
    st = ctx._lib.tid_encode(ctx.ptr, ctypes.c_void_p(blob.data_ptr()), blob.numel(),
                             ctypes.c_void_p(o.data_ptr()), 1, 1,
                             ctypes.c_void_p(rows.data_ptr()), ctypes.byref(out))
    text = ctx._lib.tid_last_error(ctx.ptr).decode()
    assert st == -4 and "2^32 bytes" in text, (st, text)
    assert out.value is None


@pytest.mark.parametrize("at", [(1 << 64) - 1, (1 << 64) - 4, (1 << 63) + 7])
def test_offset_that_wraps(ctx, at):
    """An offset so large that the difference to the next one wraps to a small length."""
    import torch
    blob = torch.zeros(64, dtype=torch.uint8, device="cuda")
    o = torch.tensor([at - (1 << 64), 5, 9, 12], dtype=torch.int64, device="cuda")
    rows = torch.zeros(3, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    out = ctypes.c_void_p()
    st = ctx._lib.tid_encode(ctx.ptr, ctypes.c_void_p(blob.data_ptr()), blob.numel(),
                             ctypes.c_void_p(o.data_ptr()), 1, 1,
                             ctypes.c_void_p(rows.data_ptr()), ctypes.byref(out))
    text = ctx._lib.tid_last_error(ctx.ptr).decode()
    assert st == -1 and "fall" in text, (st, text)
