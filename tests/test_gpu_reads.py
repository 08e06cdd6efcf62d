"""Reads of the state and the pass sums, through the stack (small jobs) and the
pinned buffer, against the copies a saved state holds; parts left out; a
batch's against an integrator's of the same job."""
import ctypes as C

import numpy as np
import pytest

import workloads as W
from gpu_util import mcv

pytestmark = pytest.mark.gpu


# d, K, n: below, around (16 KB of edges) and above the pinned buffer's bound
@pytest.mark.parametrize("d,K,n", [(1, 1, 5), (3, 13, 50), (4, 13, 51), (10, 32, 100)])
def test_reads_match_saved_state(d, K, n):
    p = W.gauss_mixture(d, K, n, 5)
    h = mcv().Integrator(p, max_iterations=4)
    h.sample_iteration(20_000)
    h.refine()
    h.sample_iteration(20_000)
    blob = np.frombuffer(h.save_state(), np.float64)[16:]
    ne, nh = K * d * (n + 1), K * d * n
    at = np.cumsum([0, ne, K, 4 * 5, nh, K * 8, K, K + 1])
    part = [blob[a:b] for a, b in zip(at[:-1], at[1:])]
    e, a, nc = h.get_state()
    hist, stats = h.pass_stats()
    assert np.array_equal(e.ravel(), part[0]) and np.array_equal(a, part[1])
    assert np.array_equal(h.history, part[2].reshape(4, 5)[:2])
    assert np.array_equal(hist.ravel(), part[3])
    assert np.array_equal(stats, part[4].reshape(K, 8)[:, :7])
    assert np.array_equal(nc[:K], part[5].view(np.int64)) and nc[K] == part[6].view(np.int64)[K]
    only = np.full(K, -1.0)
    assert mcv().lib().mcv_get_state(h._h, None, only.ctypes.data_as(C.POINTER(C.c_double)), None) == 0
    assert np.array_equal(only, a)

    b = mcv().Batch([p, p], [20_000, 30_000], max_iterations=4)
    b.iterate()
    b.iterate(what=0)
    be, ba, bnc = b.get_state(0)
    assert np.array_equal(bnc, nc) and b.history(0).shape == (2, 5)
    assert np.allclose(be, e, rtol=1e-9, atol=1e-12) and np.allclose(ba, a, rtol=1e-9)
    assert b.result(0)["n_iter"] == 2
    # the weighted mean of one row, (E / s^2) / (1 / s^2): three roundings
    row = b.history(0)[1, 0]
    assert abs(b.result(0, 1)["integral"] - row) <= 3 * 2.0**-53 * 2 * abs(row)
    b.close()
    h.close()
