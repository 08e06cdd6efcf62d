"""Batched FP64 passes of channels with one or two Breit-Wigner axes, the
others flat: the pair channels' own path, which a set takes when all its units
are resident at once, against the general path of a larger set.  The first
pass of a job is the same bit for bit in both (its estimate, error and largest
weight hold every call's f and g): dimensions of every kernel body, hint cells
of 256 and 512, crowded cells, and channels of the other kinds beside them."""
import numpy as np
import pytest

import workloads as W
from gpu_util import mcv

pytestmark = pytest.mark.gpu

TUNE = {"block": 256, "unit_calls": 256, "launch_bound": 256, "term_bound": 0}


def _job(d, K, n, seed):
    rng = np.random.default_rng(seed)
    p = W.gauss_mixture(d, K, n, seed)
    kind = np.zeros((K, d), np.int32)
    width = np.exp(rng.uniform(np.log(1e-5), np.log(0.1), (K, d)))
    for c in range(K):
        axes = rng.permutation(d)
        if c % 8 == 7:  # a Gaussian axis, or Breit-Wigner ones on all
            kind[c] = W.BW if c % 16 == 15 else W.FLAT
            kind[c, axes[0]] = W.GAUSS if c % 16 == 7 else kind[c, axes[0]]
        else:
            kind[c, axes[:1 + c % 2]] = W.BW
    return p.with_(peak_kind=kind, chan_kind=kind.copy(), peak_width=width, chan_width=width.copy())


@pytest.mark.parametrize("term_bound", [0, 1])
def test_first_pass_is_the_same_in_any_set(term_bound):
    jobs = [_job(d, 3 + 2 * d, 100 if d % 3 == 0 else 33, d) for d in range(1, 13)]
    calls = [3000 + 77 * d for d in range(1, 13)]
    tune = dict(TUNE, term_bound=term_bound)
    small = mcv().Batch(jobs, calls, tuning=tune, max_iterations=2)
    assert small.info()["units"] <= 1024  # 16 wavefronts on each of 256 CUs
    large = mcv().Batch(jobs + [_job(2, 4, 20, 99)], calls + [400_000], tuning=tune, max_iterations=2)
    assert large.info()["units"] > 1024
    for b in (small, large):
        b.iterate()
    for i in range(len(jobs)):
        x, y = small.history(i)[0], large.history(i)[0]
        assert np.isfinite(x).all() and x[4] == 0
        np.testing.assert_array_equal(x, y, err_msg="d = %d" % jobs[i].dim)
    small.close()
    large.close()
