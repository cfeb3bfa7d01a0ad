"""The allocation-free sampling entry point (lede_op_sample_noalloc) through the
C ABI: its draws against the oracle's probabilities, with rows of up to and past
the 32768 tokens that are read once; and, bit-exact, against lede_op_sample row
by row: two calls in a row on the same device array, the second with fewer and
shorter rows, and a call with a row stride past the row length."""
import ctypes

import numpy as np
import pytest

import lede_inputs as li
from oracle import model as om
from tests.parity import CDF_EPS, draw_consistent, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _rows(n, V, seed, scale=3.0):
    z = li.normal(seed, 70, n * V, scale, "f32").reshape(n, V)
    return torch.from_numpy(z).to("cuda")


def _reference(z, T, u):
    from paper_2606_03113_amd import op_sample
    return [op_sample(z[r], T, float(u[r])) for r in range(z.shape[0])]


def test_noalloc_sampling_matches_allocating_entry_point():
    from paper_2606_03113_amd import op_sample_noalloc
    for n, V, T, seed in ((20, 32000, 0.6, 1), (5, 1000, 0.05, 2)):
        say("noalloc sampling rows=%d V=%d T=%g" % (n, V, T))
        z = _rows(n, V, seed)
        u = li.uniform01(seed, 71, n)
        got = op_sample_noalloc(z, T, u)
        assert got == _reference(z, T, u)


@pytest.mark.parametrize("n,V", [(32, 16), (32, 1025), (20, 32768), (20, 32769), (7, 50257), (3, 128256), (2, 300000)])
def test_noalloc_sampling_is_inverse_cdf(n, V):
    from paper_2606_03113_amd import op_sample_noalloc
    say("noalloc sampling, oracle probabilities, rows=%d V=%d" % (n, V))
    z = _rows(n, V, 5, 1.0)
    u = li.uniform01(5, 74, n)
    got = op_sample_noalloc(z, 0.6, u)
    for r in range(n):
        p = om.probs_at(z[r].cpu().numpy().astype(np.float64), 0.6)
        assert draw_consistent(p, got[r], float(np.float32(u[r])), CDF_EPS), r


def test_noalloc_row_stride_and_limits():
    from paper_2606_03113_amd import load, op_sample_noalloc
    from paper_2606_03113_amd.lede import LEDE_E_ARG
    L = load()
    n, V, ld = 32, 1025, 1031
    say("noalloc sampling rows=%d V=%d ld=%d" % (n, V, ld))
    zf = _rows(n, ld, 3)
    u = li.uniform01(3, 72, n)
    out = np.zeros(n, dtype=np.int32)
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    up = u.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
    op = out.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    assert L.lede_op_sample_noalloc(zf.data_ptr(), n, ld, V, 0.6, up, op, s) == 0
    assert out.tolist() == _reference(zf[:, :V].contiguous(), 0.6, u)
    # more rows than the static key array holds, a stride below the row length,
    # a bad temperature or uniform: refused before anything runs
    u33 = np.full(33, 0.5, dtype=np.float32)
    assert L.lede_op_sample_noalloc(zf.data_ptr(), 33, ld, V, 0.6, u33.ctypes.data_as(ctypes.POINTER(ctypes.c_float)),
                                    op, s) == LEDE_E_ARG
    assert L.lede_op_sample_noalloc(zf.data_ptr(), n, V - 1, V, 0.6, up, op, s) == LEDE_E_ARG
    assert L.lede_op_sample_noalloc(zf.data_ptr(), n, ld, V, 0.0, up, op, s) == LEDE_E_ARG
    bad = u.copy()
    bad[3] = 1.0
    assert L.lede_op_sample_noalloc(zf.data_ptr(), n, ld, V, 0.6, bad.ctypes.data_as(ctypes.POINTER(ctypes.c_float)),
                                    op, s) == LEDE_E_ARG
    # the array still serves a smaller call afterwards
    z2 = _rows(2, 64, 4)
    u2 = li.uniform01(4, 73, 2)
    assert op_sample_noalloc(z2, 1.0, u2) == _reference(z2, 1.0, u2)
