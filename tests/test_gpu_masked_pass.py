"""The FP32 pass with channel masks and put-off lookups (mcv_mask.h,
PendingTerms) against the direct evaluation of every channel term in the trace
kernel, at the edges of its forms: kernel buckets and dimensions below them,
channels below, at and beyond whole tiles of 32, channels that the mask cannot
bound, peaks without a channel, narrow widths beyond the FP16 range, negative
peaks, and enough overlapping channels to fill the 64-entry queue.  Both sides
are FP32 at the same point and differ by the order of their sums: K + 2d + 20
roundings of 2^-24 of the terms' magnitudes."""
import numpy as np
import pytest

import workloads as W
from gpu_util import mcv, random_alpha, random_edges

pytestmark = pytest.mark.gpu


def _problem(shape, d, K, seed):
    rng = np.random.default_rng(seed)
    if shape == "product":  # Gaussian, Breit-Wigner and flat axes in one channel
        p = W.gauss_mixture(d, K, 50, seed, anisotropic=True)
        kind = rng.integers(0, 3, (K, d)).astype(np.int32)
        kind[:, 0] = W.GAUSS
        return p.with_(peak_kind=kind, chan_kind=kind.copy())
    if shape == "wide":  # every channel counts nearly everywhere
        return W.gauss_mixture(d, K, 20, seed, sigma_range=(0.3, 0.6))
    if shape == "narrow":  # beyond the FP16 range of the coefficients for some
        return W.gauss_mixture(d, K, 50, seed, sigma_range=(5e-5, 0.1))
    if shape == "orphans":  # more peaks than channels
        p = W.gauss_mixture(d, K + 5, 33, seed, anisotropic=True)
        return p.with_(chan_kind=p.chan_kind[:K], chan_loc=p.chan_loc[:K], chan_width=p.chan_width[:K])
    if shape == "negative":
        p = W.gauss_mixture(d, K, 40, seed)
        w = p.peak_weight.copy()
        w[::3] *= -0.2
        return p.with_(peak_weight=w)
    return W.gauss_mixture(d, K, 100, seed, sigma_range=(0.01, 0.1), anisotropic=shape == "aniso")


@pytest.mark.parametrize("shape,d,K", [
    ("iso", 4, 4), ("aniso", 5, 31), ("aniso", 6, 32), ("aniso", 7, 33), ("iso", 8, 64),
    ("aniso", 9, 65), ("iso", 10, 97), ("aniso", 12, 12), ("iso", 13, 20), ("aniso", 16, 40),
    ("product", 5, 20), ("product", 7, 40), ("wide", 4, 40), ("wide", 10, 70), ("narrow", 6, 24),
    ("narrow", 10, 24), ("orphans", 6, 9), ("negative", 7, 12)])
def test_masked_pass_equals_direct_evaluation(shape, d, K):
    p = _problem(shape, d, K, 1000 * d + K).with_(precision=W.FP32_MIXED)
    gpu = mcv().Integrator(p)
    rng = np.random.default_rng(d + K)
    gpu.set_state_for_test(random_edges(rng, K, d, p.n_bins, fp32=True, spread=2.0), random_alpha(rng, K))
    N, count = 40_000 + 11 * K, 2000
    tol = (K + 2 * d + 20) * 2.0 ** -24
    for first in (0, N // 2, N - count):
        timed, direct = gpu.sample_trace(N, 5, first, count), gpu.trace(N, 5, first, count)
        a, b = timed["g"], direct["g"]
        # where ten widths of 5e-5 take the FP32 normalisation beyond its range,
        # inf * 0 and the order of the factors decide what is finite on either
        # side: there is nothing to compare
        ok = np.isfinite(b) & (b != 0) & np.isfinite(a) & (a != 0)
        if shape != "narrow":
            assert np.all(ok == (np.isfinite(b) & (b != 0)))
        assert ok.mean() > (0.2 if shape == "narrow" else 0.9)
        assert np.max(np.abs(a[ok] - b[ok]) / b[ok]) < tol
        fa, fb = timed["f"][ok], direct["f"][ok]
        if shape == "negative":  # the terms cancel: against their magnitudes
            q = p.with_(peak_weight=np.abs(p.peak_weight))
            h = mcv().Integrator(q)
            h.set_state_for_test(*gpu.get_state()[:2])
            scale = h.trace(N, 5, first, count)["f"][ok]
        else:
            scale = np.abs(fb)
        assert np.max(np.abs(fa - fb) / scale) < tol


@pytest.mark.parametrize("precision", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("N", [40, 255, 256, 257, 65_537, 262_144, 1_000_003])
def test_units_and_sums_cover_every_call(N, precision):
    """The split of a pass into units and the chunked sums: per-bin sums,
    S2 and the history agree with each other whatever the split (each axis'
    bins of channel c add up to S2_c; orders of summation: N roundings)."""
    p = W.mixed_problem(4, 3, 1, 20, seed=5, precision=precision)
    gpu = mcv().Integrator(p)
    gpu.sample_iteration(N)
    hist, st = gpu.pass_stats()
    e = gpu.history[0]
    assert e[2] == gpu.alloc[-1] == gpu.alloc[:-1].sum() and e[4] == 0
    for k in range(p.dim):
        np.testing.assert_allclose(hist[:, k].sum(1), st[:, 1], rtol=N * 2.0 ** -53 + 1e-14)
    np.testing.assert_allclose(e[0], st[:, 0].sum() / e[2], rtol=1e-14)
    assert e[3] == st[:, 2].max()
