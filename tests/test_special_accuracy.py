"""The tangent of the channel maps as mcv_device.h has it (compiled for the
CPU, see test_special_ends.py) against mpmath.  Bound: 1/2 ulp of the final
sum, and the parts that carry no remainder: the polynomial rests of sine and
cosine, at most 0.1 and 0.42 of their sums (pi / 4), a rounding and a half each
of their own unit; 1 ulp in all, and 0.3 on average for rounding errors that
are independent."""
import mpmath as mp
import numpy as np

from test_special_ends import build


def _ulps(got, want):
    return float(abs(mp.mpf(got) - want) / mp.mpf(float(np.spacing(abs(float(want))))))


def test_tangent(tmp_path):
    lib = build(tmp_path)
    mp.mp.dps = 45
    rng = np.random.default_rng(6)
    half = np.pi / 2
    for lo, hi in ((0.0, 0.7), (0.7, 0.87), (0.87, half)):
        a = rng.uniform(lo, hi, 3000) * rng.choice([-1, 1], 3000)
        e = np.array([_ulps(lib.t_tan(float(v)), mp.tan(mp.mpf(float(v)))) for v in a])
        assert e.max() < 1.0 and e.mean() < 0.3, (lo, hi)
    ends = np.concatenate([half - np.exp(rng.uniform(-36, 0, 1000)), np.exp(rng.uniform(-60, 0, 1000)), [half, -half]])
    for v in ends:
        assert _ulps(lib.t_tan(float(v)), mp.tan(mp.mpf(float(v)))) < 1.0, v
    assert lib.t_tan(0.0) == 0.0 and lib.t_tan(1e-310) == 1e-310 and np.isnan(lib.t_tan(float("nan")))
