"""What the many-row prefill kernels and their launchers compute from sizes
alone, on the CPU."""
import ctypes
import os

import pytest

from tests import wide_host

pytestmark = pytest.mark.skipif(not os.path.exists(wide_host.CLANG), reason="ROCm compilers not installed")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return wide_host.load(tmp_path_factory.mktemp("wide_host"))


@pytest.mark.timeout(60)
def test_k_walk_ends_and_keeps_the_summation_order(host):
    """For every tile count from one up, the staged kernels walk K in the order
    of the 16-row kernels' sums: wavefront w = 0..7 takes the tiles w, w + 16, ...
    in one accumulator and w + 8, w + 24, ... in another; after the last tile
    the walk stays past the end (classes past the last tile are empty)."""
    for kt in range(1, 1001):
        want = [t for w in range(8) for c in (w, w + 8) for t in range(c, kt, 16)]
        assert sorted(want) == list(range(kt))
        got = (ctypes.c_int * (kt + 1))()
        host.walk(kt, got)
        assert list(got)[:kt] == want, kt
        assert got[kt] >= kt, kt
