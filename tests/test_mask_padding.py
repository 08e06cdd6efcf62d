"""The features of a call for the channel masks, as mcv_mask.h forms them
(its own code, compiled for the CPU), in dimensions at and below the kernels'
buckets: an axis beyond d holds 0 and adds nothing, so that passing a
channel's threshold proves the exponent over the d axes.  The product's steps
as in test_channel_mask.py."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from test_channel_mask import EXP_SCALE, _coefficients, _rtz16

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_09711_amd", "csrc")
BUCKETS = [2, 4, 6, 8, 10, 12, 16]
PRELUDE = """
#include <cmath>
#define __device__
#define __forceinline__ inline
"""
CALL = """
template <int MAXD, bool EXACT>
static void fill(const float* p, int n, int d, const float* ee, float* out) {
  constexpr int N = 16 * mask_form(MAXD, EXACT).steps;
  for (int i = 0; i < n; ++i) {
    float q[MAXD];
    for (int k = 0; k < MAXD; ++k) q[k] = k < d ? p[i * d + k] : 0.0f;
    float x[N];
    mask_features<MAXD, EXACT>(q, d, ee[i], x);
    for (int k = 0; k < N; ++k) out[i * N + k] = x[k];
  }
}
extern "C" void form(int d, int* f) {
  const MaskForm m = mask_form_of(d);
  f[0] = m.axes; f[1] = m.q2; f[2] = m.e; f[3] = m.steps;
}
extern "C" int features(int d, const float* p, int n, const float* ee, float* out) {
  %s
  return 1;
}
""" % "\n  ".join("if (d <= %d) { if (d == %d) fill<%d, true>(p, n, d, ee, out); "
                  "else fill<%d, false>(p, n, d, ee, out); return 0; }" % ((b,) * 4) for b in BUCKETS)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    src = open(os.path.join(CSRC, "mcv_mask.h")).read()
    forms = src[src.index("struct MaskForm"):src.index("// The features of one call")]
    body = src[src.index("template <int MAXD, bool EXACT, typename T, int N>"):src.index("// Bit j: channel")]
    d = tmp_path_factory.mktemp("mask")
    (d / "m.cpp").write_text(PRELUDE + forms + body + CALL)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wno-unknown-pragmas", "-o",
                           str(d / "m.so"), str(d / "m.cpp")])
    return ctypes.CDLL(str(d / "m.so"))


def _fp(a):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_float))


@pytest.mark.parametrize("d", [4, 5, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16])
def test_axes_beyond_the_dimension_add_nothing(lib, d):
    form = (ctypes.c_int * 4)()
    lib.form(d, form)
    axes, q2, e_at, steps = form
    general = axes > 0
    rng = np.random.default_rng(d)
    ruled_out = 0
    for _ in range(100):
        loc = rng.uniform(0.2, 0.8, d)
        width = np.exp(rng.uniform(np.log(0.02), np.log(0.2), d))
        lin, sq, off, sc, s = _coefficients(loc, width, general)
        assert s <= 14
        p = np.concatenate([rng.uniform(0, 1, (200, d)),
                            loc + width * rng.normal(size=(200, d)) * np.exp(rng.uniform(-1, 2, (200, 1)))])
        p = np.ascontiguousarray(np.clip(p, 0, 1).astype(np.float32))
        e = rng.integers(-126, 60, 400)
        ee = e.astype(np.float32)
        x = np.zeros((400, 16 * steps), np.float32)
        assert lib.features(d, _fp(p), 400, _fp(ee), _fp(x)) == 0
        coef = np.zeros(16 * steps, np.float16)
        coef[:d] = lin
        coef[q2:q2 + (d if general else 1)] = sq[:d if general else 1]
        coef[e_at] = sc
        D = np.zeros(400, np.float32)
        for k in range(16 * steps):
            D += _rtz16(x[:, k]).astype(np.float32) * np.float32(coef[k])
        E = float(rng.integers(-60, 200))
        out = D >= np.float32((np.float32(E) + off) * sc)
        ruled_out += int(out.sum())
        S = np.sum((EXP_SCALE * (p.astype(np.float64) - loc) / width) ** 2, axis=1)
        assert np.all(S[out] * (1 - 2.0 ** -20) + e[out] >= E)
    assert ruled_out > 1000
