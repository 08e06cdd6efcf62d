"""Refinement with one wavefront per axis (sets of more than 2048 axes) against
the 256-thread workgroups of a single job, at bins below, at and beyond a
wavefront, and the queues' dealing of such sets' units: each job's state after
two iterations is the single job's (sums of other units: 1e-9)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import mcv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(5, 0), (64, 0), (65, 0), (256, 0), (50, 0)])
def test_many_axes_refine_like_one_job(n, prec):
    M = mcv()
    ps = [W.gauss_mixture(d, 16, n, 3 + i).with_(precision=prec)
          for i, d in enumerate([4, 3, 5, 4] * 9 + [2, 7])]
    assert max(p.n_channels * p.dim for p in ps) * len(ps) > 2048
    N = [4000 + 300 * i for i in range(len(ps))]
    b = M.Batch(ps, N, max_iterations=4)
    for _ in range(2):
        b.iterate()
    for i in (0, 2, len(ps) - 1):
        h = M.Integrator(ps[i], max_iterations=4)
        for _ in range(2):
            h.sample_iteration(N[i])
            h.refine()
        e, a, _ = b.get_state(i)
        es, as_, _ = h.get_state()
        assert np.allclose(e, es, rtol=1e-9, atol=1e-12) and np.allclose(a, as_, rtol=1e-9)
        h.close()
    b.close()
