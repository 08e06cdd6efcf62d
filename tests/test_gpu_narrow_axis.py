"""A Gaussian axis so narrow that the squared distance from its centre leaves
the FP64 range: its density kernel is 0 on the other channels' calls, whose
weights stay finite."""
import numpy as np
import pytest

import workloads as W
from gpu_util import mcv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rng,strat", [(0, 0), (1, 0), (0, 2)])
def test_calls_of_other_channels_stay_finite(rng, strat):
    p = W.gauss_mixture(3, 4, 20, 8, anisotropic=True).with_(rng=rng, strat=strat)
    width = p.chan_width.copy()
    width[2, 1] = 1e-160
    p = p.with_(chan_width=width, peak_width=width.copy())
    gpu = mcv().Integrator(p)
    gpu.sample_iteration(20_000)
    stats = gpu.channel_stats
    others = [0, 1, 3]
    assert np.all(stats[others, 3] == 0) and np.all(np.isfinite(stats[others, :3]))
    assert np.all(stats[others, 0] > 0)
    direct = gpu.trace(20_000, 0, 0, 17_000)
    assert np.all(np.isfinite(direct["w"][np.isin(direct["chan"], others)]))
