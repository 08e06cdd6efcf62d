"""Stratified passes with more work units than boxes: many channels of one box
each beside one of 2^d boxes.  Units without a box write no partial sums, and
none may be read for them: the sums of a pass after another one, whose partial
sums are still in the buffers, are the oracle's."""
import os

import numpy as np
import pytest

import workloads as W
from gpu_util import inject, pair, rel

pytestmark = pytest.mark.gpu

THREADS = min(16, os.cpu_count() or 1)


def test_units_without_boxes_add_nothing():
    d, K = 9, 450
    p = W.gauss_mixture(d, K, 8, 4).with_(strat=2)
    calls = np.array([38_000.0] + [1022.0] * (K - 1))
    N = int(calls.sum())
    gpu, orc = pair(p)
    # a short pass leaves sums in the slots of most units, then the other one
    # has 512 boxes of channel 0 and one of each other channel, fewer than its
    # rounds of 256 boxes of two calls
    for n in (10_000, N):
        inject(gpu, orc, alpha=calls / N)
        gpu.sample_iteration(n)
        orc.sample_iteration(n, THREADS)
        np.testing.assert_array_equal(gpu.alloc, orc.alloc)
    assert orc.alloc[0] % 512 == 0 and 512 + K - 1 < N // 512
    sg, so = gpu.channel_stats, orc.channel_stats
    assert rel(sg[:, :3], so[:, :3]) < 1e-11
    assert rel(gpu.hist.sum(2), orc.hist.sum(2)) < 1e-11
    assert rel(gpu.history[1][0], orc.history[1][0]) < 1e-11
    assert rel(gpu.history[1][1], orc.history[1][1]) < 1e-9
