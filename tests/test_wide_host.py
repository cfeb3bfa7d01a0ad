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


@pytest.mark.parametrize("nkv", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 16, 20, 32, 40])
def test_attention_blocks_fill_every_xcd(host, nkv):
    """A prefill attention launch covers every KV head's row blocks once, the
    longest first, and gives the eight XCDs (block number modulo 8) equally many;
    1, 2, 4 or 8 heads keep to 8 / heads XCDs each."""
    for n_rb in (1, 2, 3, 7, 8, 16, 33, 128):
        n = nkv * n_rb
        out = (ctypes.c_int * (2 * n))()
        host.attn_blocks(nkv, n_rb, out)
        pairs = list(zip(out[0::2], out[1::2]))
        assert sorted(pairs) == [(h, r) for h in range(nkv) for r in range(n_rb)]
        per_xcd = [len(pairs[x::8]) for x in range(8)]
        assert max(per_xcd) - min(per_xcd) <= 1
        for h in range(nkv):
            assert [r for k, r in pairs if k == h] == list(range(n_rb))[::-1]
            if nkv in (1, 2, 4, 8):
                xcds = {b % 8 for b, (k, _) in enumerate(pairs) if k == h}
                assert len(xcds) == min(n_rb, 8 // nkv)
