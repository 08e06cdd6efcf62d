"""The FP32 pass with channel masks (mcv_mask.h, PendingTerms) against the pass
without, bit for bit.  A job of four channels, three of them Gaussian, has no
masks; 16 more channels, narrow Gaussians in corners that take half of the
calls, give the same job masks (most pairs of its channels are then far apart).
The first four channels make the same calls with half the weights, and on calls
away from the corners the others' density kernels are exactly 0: f is the same, g is halved exactly and w doubled.
The Gaussians overlap, so that a channel wrongly left out shows: dimensions at
and below the kernels' buckets, in both forms of the mask."""
import math

import numpy as np
import pytest

import workloads as W
from gpu_util import mcv, random_edges

pytestmark = pytest.mark.gpu

N = 20_000
NARROW = 2e-3
# 0.03 or 0.97 on each of the first four axes
CORNERS = 0.03 + 0.94 * ((np.arange(16)[:, None] >> np.arange(4)) & 1)


def _problems(d, sigma, seed, shape):
    rng = np.random.default_rng(seed)
    kind = np.full((20, d), W.GAUSS, np.int32)
    loc = np.full((20, d), 0.97)
    loc[4:, :4] = CORNERS
    width = np.full((20, d), NARROW)
    loc[0] = rng.uniform(0.3, 0.5, d)
    for c in (1, 2):
        loc[c] = loc[0] + rng.uniform(-1, 1, d) * sigma / math.sqrt(d)
    width[:3] = sigma * (rng.uniform(0.9, 1.1, (3, 1)) if shape == "iso" else rng.uniform(0.7, 1.4, (3, d)))
    if shape == "product":  # a Breit-Wigner axis beside the Gaussian ones
        kind[:3, 1] = W.BW
    kind[3] = W.FLAT
    kind[3, 0], loc[3, 0], width[3, 0] = W.BW, 0.4, 0.05
    a = W.Problem(d, 20, kind[:4], loc[:4], width[:4], np.full(4, 0.25), kind[:4].copy(), loc[:4].copy(),
                  width[:4].copy(), seed=seed, precision=W.FP32_MIXED)
    return a, a.with_(chan_kind=kind, chan_loc=loc, chan_width=width)


def _own_share(p, c, x):
    """Channel c's share of g at x on equidistant grids and equal weights."""
    q = np.ones((p.n_channels, len(x)))
    for i in range(p.n_channels):
        for k in range(p.dim):
            if p.chan_kind[i, k] != W.FLAT:
                m, s = p.chan_loc[i, k], p.chan_width[i, k]
                if p.chan_kind[i, k] == W.GAUSS:
                    z = 0.5 * (math.erf((1 - m) / s / math.sqrt(2)) + math.erf(m / s / math.sqrt(2)))
                    q[i] *= np.exp(-0.5 * ((x[:, k] - m) / s) ** 2) / (s * math.sqrt(2 * math.pi) * z)
                else:
                    th = math.atan((1 - m) / (s / 2)) + math.atan(m / (s / 2))
                    q[i] *= (s / 2) / ((x[:, k] - m) ** 2 + (s / 2) ** 2) / th
    return q[c, np.arange(len(x))] / q.sum(0)


@pytest.mark.parametrize("rng", [0, 1])
@pytest.mark.parametrize("sigma", [0.03, 0.1])
@pytest.mark.parametrize("d,shape", [(d, s) for d in range(4, 17) for s in ("iso", "aniso", "product")
                                     if d < 8 or s != "product"])  # beyond, no mask bounds products
def test_masks_leave_every_bit(d, shape, sigma, rng):
    pa, pb = (p.with_(rng=rng) for p in _problems(d, sigma, 100 * d + len(shape), shape))
    a, b = mcv().Integrator(pa), mcv().Integrator(pb)
    for grids in ("flat", "random"):
        if grids == "random":
            e = random_edges(np.random.default_rng(d), 20, d, 20, fp32=True, spread=1.0)
            a.set_state_for_test(e[:4], None)
            b.set_state_for_test(e, None)
        b.set_state_for_test(None, np.array([1 / 8] * 4 + [1 / 32] * 16))
        ta, tb = a.sample_trace(N, 3, 0, N), b.sample_trace(2 * N, 3, 0, N)
        point = a.trace(N, 3, 0, N)
        near = np.abs(point["p"][:, None, :4] - CORNERS) < 40 * NARROW
        away = ~near.all(2).any(1)
        assert away.mean() > 0.99
        if grids == "flat":
            # the other channels matter where a Gaussian's calls fall
            share = _own_share(pa, point["chan"], point["p"])[point["chan"] < 3]
            assert np.mean(share < 0.9) > 0.3
        for k, s in (("f", 1.0), ("g", 0.5), ("w", 2.0)):
            x, y = ta[k][away] * s, tb[k][away]
            assert np.all(np.isfinite(x)), k
            wrong = np.flatnonzero(x != y)
            assert len(wrong) == 0, (grids, k, len(wrong), x[wrong[:3]], y[wrong[:3]])
    a.close()
    b.close()
