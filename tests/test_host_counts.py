"""The load-time ID counts as the host builds them (csrc/idcounts.hpp), and a
circular server's view of 2^32 triples or more, whose sums take 64 bits."""
import os
import subprocess

import numpy as np
import pytest

import stand_in

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "idcounts.hpp"
#include <cstdio>
// bins of `blocks` blocks on stdin, then pairs (first block, ID): the IDs below
int main(int argc, char **argv) {
    uint64_t blocks = strtoull(argv[1], nullptr, 10), q[2];
    std::vector<uint32_t> bins(blocks * tid::IdCounts::kBlock);
    if (fread(bins.data(), 4, bins.size(), stdin) != bins.size()) return 1;
    tid::IdCounts c;
    c.mem = tid::counts_of_bins(bins.data(), blocks);
    while (fread(q, 8, 2, stdin) == 2) {
        c.first = q[0];
        c.ids = (blocks - q[0]) * tid::IdCounts::kBlock;
        c.total = c.mem->rows[blocks] - c.mem->rows[c.first];
        printf("%llu\n", (unsigned long long)c.below(q[1]));
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("counts")
    (d / "counts.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-include", "cstdlib", "-I",
                    os.path.join(ROOT, "paper_1807_01409_amd", "csrc"), str(d / "counts.cpp"),
                    "-o", str(d / "counts")], check=True)
    return str(d / "counts")


@pytest.mark.parametrize("blocks", [1, 2, 5])
@pytest.mark.parametrize("most", [256, 1 << 16, (1 << 32) - 1])
def test_counts_of_bins(program, blocks, most):
    rng = np.random.default_rng(blocks + most)
    bins = rng.integers(0, 300, 256 * blocks).astype(np.uint32)
    bins[rng.integers(0, bins.size, 40)] = rng.integers(most // 2, most, 40, endpoint=True)
    bins[[0, -1]] = 0, most       # several bins near 2^32 in a block
    asks = [(f, i) for f in range(blocks) for i in range(256 * (blocks - f) + 3)]
    got = subprocess.run([program, str(blocks)],
                         input=bins.tobytes() + np.array(asks, dtype=np.uint64).tobytes(),
                         capture_output=True, check=True).stdout.split()
    cum = np.concatenate([[0], np.cumsum(bins.astype(np.uint64))])
    want = [int(cum[min(256 * f + i, bins.size)] - cum[256 * f]) for f, i in asks]
    assert [int(x) for x in got] == want


@pytest.mark.parametrize("chunks,on_device", [(1, False), (2, True)])
def test_large_views_are_summed_on_the_host(tmp_path, chunks, on_device):
    """A view of 2^32 triples or more does not go through the 32-bit block sums
    of the device."""
    out = stand_in.run(tmp_path, f"""
ctx = context()
n = (1 << 32) + 4096
word("read_word", ctypes.c_uint32).value = 300000  # smallest and largest ID, and every count
g, s = ctypes.c_void_p(), ctypes.c_void_p()
assert lib.tid_load(ctx, device(12 * n), n, 1, ctypes.byref(g)) == 0
st = lib.tid_serve_open(ctx, g, {chunks}, 1, ctypes.byref(s))
out = dict(st=st, error=error(ctx), kernels=kernels())
""")
    assert out["st"] == 0, out["error"]
    assert any("hist3_kernel" in k for k in out["kernels"])
    assert any("pack_counts" in k for k in out["kernels"]) == on_device
