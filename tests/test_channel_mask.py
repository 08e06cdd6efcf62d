"""The bound that leaves channels out of the FP32 pass (mcv_mask.h): whenever
the FP16 product of a call's features and a channel's coefficients passes the
channel's threshold, the channel's exact exponent S_c(p) plus the call's e does
reach the skip exponent E it stands for.  The kernel's steps in numpy: features
rounded toward zero to FP16, coefficients to the nearest, FP32 sums; both forms
(every axis, and the smallest ga for all)."""
import numpy as np
import pytest

EXP_SCALE = np.sqrt(np.log2(np.e) / 2)


def _rtz16(x):
    h = x.astype(np.float16)
    over = np.abs(h.astype(np.float64)) > np.abs(x)
    return np.where(over, np.nextafter(h, np.float16(0)), h)


def _coefficients(loc, width, general):
    """As k_setup_mask: scaled coefficients (linear, squares), offset and scale."""
    ga = EXP_SCALE / width
    if not general:
        ga = np.full_like(ga, ga.min())
    g = ga * (0.5 - loc)
    A, B = ga * ga, 2 * ga * g
    big = max(A.max(), np.abs(B).max())
    s = max(0, int(np.ceil(np.log2(big))) - 10)
    while big > 2.0 ** (10 + s):
        s += 1
    sc = 2.0 ** -s
    d = len(loc)
    eps = 2.0 ** -9 * np.sum(0.25 * A + 0.5 * np.abs(B) + g * g) + \
        2.0 ** -14 * np.sum(A + np.abs(B)) + 2 * d * 2.0 ** -14 / sc + 0.5
    return (B * sc).astype(np.float16), (A * sc).astype(np.float16), \
        np.float32(eps - np.sum(g * g) + 1.0), np.float32(sc), s


@pytest.mark.parametrize("general", [True, False])
@pytest.mark.parametrize("d", [1, 3, 7, 10, 16])
def test_passing_the_threshold_proves_the_exponent(d, general):
    rng = np.random.default_rng(100 * d + general)
    ruled_out = 0
    for _ in range(300):
        loc = rng.uniform(0.0, 1.0, d)
        width = np.exp(rng.uniform(np.log(3e-4), np.log(0.5), d))
        lin, sq, off, sc, s = _coefficients(loc, width, general)
        if s > 14:
            continue
        # points near the channel's skip surface and anywhere
        far = rng.uniform(0, 1, (200, d))
        near = loc + width * rng.normal(size=(200, d)) * np.exp(rng.uniform(0, 3, (200, 1)))
        p = np.clip(np.concatenate([far, near]), 0, 1).astype(np.float32)
        e = rng.integers(-126, 60, 400)
        E = float(rng.integers(-60, 200))
        thr = np.float32((np.float32(E) + off) * sc)
        q = p - np.float32(0.5)
        D = np.zeros(400, np.float32)
        qsum = np.zeros(400, np.float32)
        for k in range(d):
            D += _rtz16(q[:, k]).astype(np.float32) * np.float32(lin[k])
            if general:
                D += _rtz16(q[:, k] * q[:, k]).astype(np.float32) * np.float32(sq[k])
            else:
                qsum += q[:, k] * q[:, k]
        if not general:
            D += _rtz16(qsum).astype(np.float32) * np.float32(sq[0])
        D += e.astype(np.float32) * sc
        out = D >= thr
        ruled_out += int(out.sum())
        S = np.sum((EXP_SCALE * (p.astype(np.float64) - loc) / width) ** 2, axis=1)
        assert np.all(S[out] * (1 - 2.0 ** -20) + e[out] >= E)
    assert ruled_out > 1000  # the bound does rule channels out
