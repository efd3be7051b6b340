"""The remainder that brackets stage times, bit for bit the C library's fmod: quotients
that round up or down to the next whole number, negative and zero dividends, dividends
below the divisor, an infinite divisor, and quotients past 2^51."""

import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1707_05163_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("fmod")
    src = d / "f.cpp"
    src.write_text('#include "lp_fmod.h"\n'
                   'extern "C" double f(double a, double p) { return exact_fmod(a, p); }\n')
    out = d / "f.so"
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(out)],
                   check=True)
    f = ctypes.CDLL(str(out)).f
    f.restype = ctypes.c_double
    f.argtypes = [ctypes.c_double, ctypes.c_double]
    return f


def _same(f, a, p):
    want, got = math.fmod(a, p), f(a, p)
    assert want == got and math.copysign(1.0, want) == math.copysign(1.0, got), (a, p, want, got)


def test_random_quotients(lib):
    g = np.random.default_rng(1)
    for _ in range(20000):
        p = float(np.exp(g.uniform(-20, 20)))
        _same(lib, float(g.normal()) * p * float(np.exp(g.uniform(-5, 40))), p)


@pytest.mark.parametrize("p", [0.1, 1.0 / 3.0, 86400.1, 87000.0, 2592000.0, 1e-300, 1e300,
                               5e-324, 2.2250738585072014e-308])
def test_beside_whole_multiples(lib, p):
    for k in [1, 2, 3, 7, 10, 12345, 2**31 - 1, 2**50 - 1, 2**50, 2**51, 2**52 + 1]:
        a = k * p
        if math.isinf(a):
            continue
        for b in (a, math.nextafter(a, math.inf), math.nextafter(a, -math.inf)):
            if not math.isinf(b):
                _same(lib, b, p)
                _same(lib, -b, p)


def test_zeros_and_infinite_divisor(lib):
    for p in (1.0, 87000.0, math.inf):
        for a in (0.0, 5e-324, 0.5, 86400.0, 1e300):
            if p == math.inf or a < 1e15:
                _same(lib, a, p)
                _same(lib, -a, p)
    assert math.isnan(lib(math.nan, 2.0)) and math.isnan(lib(math.inf, 2.0))
