"""The special functions of the channel maps in mcv_device.h: their
coefficients are the ones fp64_fit.py computes, and the same evaluation in
numpy (plain multiplies and adds where the kernel fuses them) stays within a
few roundings of mpmath.  Bounds: a Horner chain on [-1, 1] whose partial sums
stay below a few times its value, a logarithm and three more operations: 12
roundings of 2^-53; the FP32 ones 12 of 2^-24."""
import os
import re
import sys

import mpmath as mp
import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_09711_amd", "csrc")
SRC = open(os.path.join(CSRC, "mcv_device.h")).read()
NUM = r"-?\d[\d.]*(?:e[+-]\d+)?"


@pytest.fixture(scope="module")
def fits():
    sys.path.insert(0, CSRC)
    try:
        import fp64_fit
    finally:
        sys.path.pop(0)
    return fp64_fit, {k: ([float(v) for v in c], cut) for k, (c, cut) in fp64_fit.fits().items()}


def _table(name):
    body = SRC[SRC.index(name):]
    body = body[body.index("= {") + 3:body.index("};")]
    return [float(v) for v in re.findall(NUM, re.sub(r"//[^\n]*", "", body))]


def _chain(fn):
    body = SRC[SRC.index(fn):]
    body = body[:body.index("\n}\n")]
    first = re.search(r"float P = (%s)f" % NUM, body).group(1)
    return [float(first)] + [float(v) for v in re.findall(r"P = fmaf\(P, \w, (%s)f\)" % NUM, body)]


def test_source_holds_the_fitted_coefficients(fits):
    mod, f = fits
    for name, cut in (("central", 1e-16), ("log", 1e-18), ("sin", 1e-17), ("cos", 1e-17), ("exp2", 1e-17),
                      ("piece0", 1e-16), ("piece1", 1e-16), ("piece2", 1e-16), ("far", 1e-8)):
        assert f[name][1] < cut, name
    assert _table("kErfcinvTab[") == f["log"][0] + f["central"][0]
    assert _table("kSinCosTab[") == f["sin"][0] + f["cos"][0]
    assert _table("kExp2Tab[") == f["exp2"][0]
    pieces = _table("kErfcinvPiece[3]")
    n = len(f["piece0"][0]) + 2
    for i, (a, b) in enumerate(mod.PIECES):
        row = pieces[i * n:(i + 1) * n]
        s, e = float(mp.sqrt(a)), float(mp.sqrt(b))
        assert abs(row[0] - (s + e) / 2) < 1e-14 and abs(row[1] - 2 / (e - s)) < 1e-14
        assert row[2:] == f["piece%d" % i][0]
    np.testing.assert_allclose(_chain("float erfcinv_far("), f["far"][0], rtol=1e-9)


def _horner(c, t):
    P = np.full_like(t, c[0])
    for v in c[1:]:
        P = P * t + v
    return P


def _erfcinv(y, f, mod):
    q = y * (2.0 - y)
    m, e = np.frexp(q)
    low = m < np.sqrt(0.5)
    m, e = np.where(low, 2 * m, m), np.where(low, e - 1, e)
    s = (m - 1.0) / (m + 1.0)
    z = s * s
    w = -(s * (z * _horner(f["log"][0], z) + 2 / np.log(2.0)) + e)
    P = _horner(f["central"][0], w * (2.0 / mod.W1) - 1.0)
    for i, (a, b) in enumerate(mod.PIECES):
        sa, sb = np.sqrt(a), np.sqrt(b)
        Pi = _horner(f["piece%d" % i][0], (np.sqrt(np.maximum(w, 0.0)) - (sa + sb) / 2) * (2 / (sb - sa)))
        P = np.where(w > a if i else w > mod.W1, Pi, P)
    return (1.0 - y) * P


def test_erfcinv_against_mpmath(fits):
    mod, f = fits
    rng = np.random.default_rng(3)
    y = np.concatenate([rng.uniform(0, 1, 400), np.exp(rng.uniform(np.log(1e-300), 0, 400)),
                        1 - np.exp(rng.uniform(np.log(1e-12), 0, 100)), [1.0, 0.5, 2.4e-4, 1e-308]])
    y = y[(y > 0) & (y <= 1)]
    got = _erfcinv(y, f, mod)
    mp.mp.dps = 40
    for v, g in zip(y, got):
        x = 1 - mp.mpf(float(v))
        if v > 0.01:
            want = mp.erfinv(x)
        else:
            want = mod.p_of_w(-mp.log(mp.mpf(float(v)) * (2 - mp.mpf(float(v))), 2)) * x
        tol = 12 * 2.0 ** -53 * max(abs(float(want)), 0.0)
        assert abs(g - float(want)) <= tol + 1e-300, (v, g, want)


def test_exp2_and_tan_against_mpmath(fits):
    _, f = fits
    rng = np.random.default_rng(4)
    x = -np.exp(rng.uniform(np.log(1e-6), np.log(1000), 300))
    n = np.rint(x)
    got = np.ldexp(_horner(f["exp2"][0], x - n), n.astype(int))
    for v, g in zip(x, got):
        want = float(mp.mpf(2) ** mp.mpf(float(v)))
        assert abs(g - want) <= 12 * 2.0 ** -53 * want
    a = np.concatenate([rng.uniform(0, np.pi / 2, 300), np.pi / 2 - np.exp(rng.uniform(-25, 0, 100))])
    near = a > 0.78539816339744830962
    r = np.where(near, (1.57079632679489655800 - a) + 6.12323399573676603587e-17, a)
    s, c = r * _horner(f["sin"][0], r * r), _horner(f["cos"][0], r * r)
    got = np.where(near, c / s, s / c)
    for v, g in zip(a, got):
        want = float(mp.tan(mp.mpf(float(v))))
        assert abs(g - want) <= 12 * 2.0 ** -53 * abs(want)


def test_fp32_far_tail(fits):
    mod, _ = fits
    f32 = np.float32
    rng = np.random.default_rng(5)
    y = np.exp(rng.uniform(np.log(1e-44), np.log(7.4e-9), 200)).astype(f32)
    y = y[y > 0]
    w = (f32(63) - np.log2(y.astype(np.float64) * 2.0 ** 64)).astype(f32)
    sa, sb = np.sqrt(mod.FAR[0]), np.sqrt(mod.FAR[1])
    t = ((np.sqrt(w) - f32((sa + sb) / 2)) * f32(2 / (sb - sa))).astype(f32)
    P = np.full_like(t, f32(_chain("float erfcinv_far(")[0]))
    for v in _chain("float erfcinv_far(")[1:]:
        P = (P * t + f32(v)).astype(f32)
    for v, g in zip(y, P):
        want = float(mod.p_of_w(-mp.log(mp.mpf(float(v)) * 2, 2)))
        assert abs(g - want) <= 12 * 2.0 ** -24 * want
