"""The C structures that the binding packs for plans hold what the plans say."""
import ctypes
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1807_01409_amd import _lib as L
from paper_1807_01409_amd import tid

FIELDS = [n for n, _ in L.tid_pattern._fields_]


def pattern(*v):
    return SimpleNamespace(**dict(zip(FIELDS, v)))


@pytest.mark.parametrize("n", [0, 1, 3])
def test_plans(n):
    plans = [SimpleNamespace(patterns=[pattern(i, j, 2 ** 32 - 1, -1, j, 3, -1, 0, 7)
                                       for j in range(i)],
                             ops=list(range(2 * i))) for i in range(n)]
    block = tid._Plans(plans)
    at = ctypes.cast(block.pointers(), ctypes.POINTER(ctypes.POINTER(L.tid_plan)))
    for i, p in enumerate(plans):
        c = at[i].contents
        assert (c.n_patterns, c.n_ops) == (len(p.patterns), len(p.ops))
        assert [c.ops[j] for j in range(c.n_ops)] == p.ops
        for j, q in enumerate(p.patterns):
            assert [getattr(c.patterns[j], f) for f in FIELDS] == [getattr(q, f) for f in FIELDS]


@pytest.mark.parametrize("v", [
    (np.int64(5), 1, 0, -1, 0, np.int32(1), -1, 0, 0),
    (5, 2 ** 32 + 7, -1, 2 ** 32 - 1, 0, 1, -1, 0, 0),      # wraps at 32 bits
    (5.0, "6", 0, -1, 0, 1, -1, 0.0, 0),                    # what int() takes
])
def test_converted_fields(v):
    got = L.tid_pattern.from_buffer_copy(tid._pattern_bytes(pattern(*v)))
    for f, x, (_, t) in zip(FIELDS, v, L.tid_pattern._fields_):
        assert getattr(got, f) == t(int(x)).value


@pytest.mark.parametrize("ops", [[], [3, 2 ** 32 - 1], [-1, 4], np.array([5, 6]), (7.0, 8)])
def test_ops(ops):
    want = np.asarray(ops, dtype=np.int64).astype(np.uint32)
    assert tid._ops_bytes(ops) == want.tobytes()
