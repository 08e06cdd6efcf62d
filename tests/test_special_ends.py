"""The FP64 special functions of the channel maps as mcv_device.h has them, its
own code compiled for the CPU (with fused multiply-adds, and a reciprocal of
2^-24 for the hardware's): the ends of their ranges."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_09711_amd", "csrc")
PRELUDE = """
#include <cmath>
#include <cstdint>
using std::fma; using std::fmax; using std::isfinite;
#define __device__
#define __forceinline__ inline
#define __noinline__
#define asm
#define volatile(...)
template <typename T> using CP = const T*;
template <typename T> static CP<T> cp(const T* p) { return p; }
static double amd_mant(double x) { int e; return std::frexp(x, &e); }
static int amd_exp(double x) { int e; std::frexp(x, &e); return std::isfinite(x) ? e : 0; }
static float amd_mantf(float x) { int e; return std::frexp(x, &e); }
static int amd_expf(float x) { int e; std::frexp(x, &e); return e; }
#define __builtin_amdgcn_frexp_mant amd_mant
#define __builtin_amdgcn_frexp_exp amd_exp
#define __builtin_amdgcn_frexp_mantf amd_mantf
#define __builtin_amdgcn_frexp_expf amd_expf
#define __builtin_amdgcn_ldexp std::ldexp
#define __builtin_amdgcn_rcp(x) ((double)(float)(1.0 / (x)) * (1.0 + 0x1p-24))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_logf(x) std::log2((float)(x))
#define __builtin_amdgcn_exp2f(x) std::exp2((float)(x))
"""
CALL = """
extern "C" {
double t_exp2(double x) { return m_exp2(x); }
double t_tan(double x) { return m_tan(x); }
double t_erfcinv(double x) { return m_erfcinv(x); }
float t_far(float x) { return erfcinv_far(x); }
}
"""


def build(folder):
    src = open(os.path.join(CSRC, "mcv_device.h")).read()
    body = src[src.index("// Coefficients of the FP64 special functions"):src.index("constexpr double kSqrt2")]
    (folder / "s.cpp").write_text(PRELUDE + body + CALL)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-w",
                           "-Wno-unknown-pragmas", "-o", str(folder / "s.so"), str(folder / "s.cpp")])
    lib = ctypes.CDLL(str(folder / "s.so"))
    for name in ("t_exp2", "t_tan", "t_erfcinv"):
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = ctypes.c_double, [ctypes.c_double]
    lib.t_far.restype, lib.t_far.argtypes = ctypes.c_float, [ctypes.c_float]
    return lib


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return build(tmp_path_factory.mktemp("special"))


def test_exp2_below_the_exponent_range_is_zero(lib):
    for x in (-math.inf, -1.8e308, -1e300, -1e17, -4097.0, -4096.0, -1080.0):
        assert lib.t_exp2(x) == 0.0, x
    assert math.isnan(lib.t_exp2(math.nan))
    assert lib.t_exp2(0.0) == 1.0 and lib.t_exp2(-1074.0) == 2.0 ** -1074


def test_erfcinv_ends(lib):
    assert lib.t_erfcinv(1.0) == 0.0
    assert math.isnan(lib.t_erfcinv(math.nan))
    # the smallest arguments that a map can form, against their asymptotic value
    for y in (5e-324, 1e-310, 2.2250738585072014e-308):
        x = lib.t_erfcinv(y)
        assert abs(math.erfc(x) - y) <= 1e-12 * y + 5e-324
    assert np.all(np.diff([lib.t_erfcinv(v) for v in np.exp(np.linspace(-740, 0, 2000))]) < 0)
