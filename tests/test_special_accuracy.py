"""The tangent and erfcinv of the channel maps and the far tail of the FP32
erfcinv as mcv_device.h has them (compiled for the CPU, see test_special_ends.py) against
mpmath.  Tangent: 1/2 ulp of the final
sum, and the parts that carry no remainder: the polynomial rests of sine and
cosine, at most 0.1 and 0.42 of their sums (pi / 4), a rounding and a half each
of their own unit; 1 ulp in all, and 0.3 on average for rounding errors that
are independent.  Far tail: 1/2 ulp of the final
sum, and t (|t| <= 1, in a term of at most 0.42 of the result) with two
roundings and the slope with one: 1.2 ulp, 0.4 on average.  FP64 erfcinv: the
errors of the library's erfcinv on the card, measured at the same ranges."""
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


def test_fp32_far_tail(tmp_path):
    lib = build(tmp_path)
    mp.mp.dps = 30
    rng = np.random.default_rng(7)
    y = np.exp(rng.uniform(np.log(1e-44), np.log(7.4e-9), 2000)).astype(np.float32)
    e = []
    for v in y[y > 0]:
        m = mp.mpf(float(v))
        z = mp.sqrt(-mp.log(m))
        for _ in range(60):  # Halley's rule on erfc(z) = y
            u = (mp.erfc(z) - m) / (-2 / mp.sqrt(mp.pi) * mp.exp(-z * z))
            step = u / (1 + z * u)
            z -= step
            if abs(step) < mp.mpf(10) ** -25:
                break
        e.append(float(abs(mp.mpf(lib.t_far(float(v))) - z) / mp.mpf(float(np.spacing(np.float32(float(z)))))))
    assert max(e) < 1.2 and np.mean(e) < 0.4
    assert lib.t_far(0.0) == np.inf and np.isnan(lib.t_far(float("nan")))


def test_erfcinv(tmp_path):
    lib = build(tmp_path)
    mp.mp.dps = 45
    rng = np.random.default_rng(8)
    # mean and largest error of the library's function, ulp
    for lo, hi, mean in ((0.5, 1.0, 0.478), (0.05, 0.5, 0.496), (2.4e-4, 0.05, 0.410), (1e-12, 2.4e-4, 0.465),
                         (1e-300, 1e-12, 0.505)):
        y = rng.uniform(lo, hi, 1500) if hi / lo < 20 else np.exp(rng.uniform(np.log(lo), np.log(hi), 1500))
        e = []
        for v in y:
            m = mp.mpf(float(v))
            if v > 0.01:
                z = mp.erfinv(1 - m)
            else:
                z = mp.sqrt(-mp.log(m))
                for _ in range(60):
                    u = (mp.erfc(z) - m) / (-2 / mp.sqrt(mp.pi) * mp.exp(-z * z))
                    step = u / (1 + z * u)
                    z -= step
                    if abs(step) < mp.mpf(10) ** -40 * z:
                        break
            e.append(_ulps(lib.t_erfcinv(float(v)), z))
        assert max(e) < 2.32 and np.mean(e) < mean, (lo, hi, max(e), np.mean(e))
