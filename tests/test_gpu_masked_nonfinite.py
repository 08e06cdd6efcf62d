"""The FP32 pass with channel masks on calls that have no point: a width beyond
the FP32 range gives NaN on its axis for every call of its channel, so that no
bound of the product holds.  Channels short of a whole tile of 32, narrow
enough for masks: the pass
counts those calls as non-finite, and the others as they are without them."""
import numpy as np
import pytest

import workloads as W
from gpu_util import mcv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K", [(4, 12), (5, 31), (9, 14), (10, 33), (12, 40), (16, 15)])
def test_calls_without_a_point_are_counted(d, K):
    p = W.gauss_mixture(d, K, 20, d + K, sigma_range=(0.01, 0.03)).with_(precision=W.FP32_MIXED)
    width = p.chan_width.copy()
    width[K - 1, 0] = 1e39
    gpu = mcv().Integrator(p.with_(chan_width=width))
    N = 30_000
    out = []
    for _ in range(2):
        gpu.sample_iteration(N)
        stats, alloc = gpu.channel_stats, gpu.alloc
        assert stats[K - 1, 3] == alloc[K - 1]
        assert np.all(stats[:K - 1, 3] <= alloc[:K - 1]) and gpu.history[-1][4] == stats[:, 3].sum()
        out.append(stats)
    traced = gpu.trace(N, 1, 0, int(gpu.alloc[:-1].sum()))
    bad = np.bincount(traced["chan"][~np.isfinite(traced["w"])], minlength=K)
    assert out[1][K - 1, 3] == bad[K - 1]
    # (the direct evaluation also multiplies the channel's infinite norm by
    # kernels of 0, which the pass leaves out)
    assert np.all(out[1][:, 3] <= bad)
