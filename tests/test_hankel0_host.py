"""hankel0 of csrc/bessel.hpp (the Hankel function of the 2D field kernels) on
the host, over the arguments the kernels meet and at the edges of its three
intervals, against an 80-bit evaluation (scipy's j0 and y0 carry an absolute
error of a few 1e-16, which is 1e-14 of |H0| at the largest arguments).
Tolerance: 2e-15 |H0| for the polynomials plus 2 ulp of the argument in the
phase."""
import ctypes
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2604_15796_amd" / "csrc"


def _reference(x):
    """H0^(1) in long double: the power series below 1, above it
    (2 / (pi sqrt x)) e^{i (x - pi/4)} times the integral over s > 0 of
    sqrt 2 exp(-s^2) (1 + i s^2 / 2x)^(-1/2) by the trapezoidal rule (step h:
    error exp(-2 pi sqrt(x) / h))."""
    x = x.astype(np.longdouble)
    pi, euler = np.longdouble("3.14159265358979323846264338"), np.longdouble("0.57721566490153286060651209")
    v, h = np.maximum(x, 1), np.longdouble("0.15")
    acc = np.full(x.shape, 0.5, dtype=np.clongdouble)
    for k in range(1, 45):
        s2 = (k * h) ** 2
        acc += np.exp(-s2) / np.sqrt(1 + 1j * (s2 / (2 * v)))
    big = 2 * h * np.sqrt(np.longdouble(2)) / (pi * np.sqrt(v)) * np.exp(1j * (v - pi / 4)) * acc
    v = np.minimum(x, 1)
    q, t, har = -v * v / 4, np.ones_like(v), np.longdouble(0)
    j0, tail = np.ones_like(v), np.zeros_like(v)
    for n in range(1, 14):
        t, har = t * q / n**2, har + np.longdouble(1) / n
        j0, tail = j0 + t, tail - har * t
    return np.where(x < 1, j0 + 2j / pi * ((np.log(v / 2) + euler) * j0 + tail), big)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_hankel0_matches_80_bit_evaluation(tmp_path):
    src = tmp_path / "h.cpp"
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("#define __host__\n#define __device__\n")
    src.write_text('#include "bessel.hpp"\n'
                   'extern "C" void h0(int n, const double* x, double* j, double* y) {\n'
                   '  for (int i = 0; i < n; ++i) fwi::hankel0(x[i], j + i, y + i);\n}\n')
    so = tmp_path / "h.so"
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", f"-I{tmp_path}", f"-I{CSRC}", str(src), "-o",
                    str(so)], check=True, timeout=300)
    edges = [e * (1 + d) for e in (4.0, 8.0, 25.0) for d in (-1e-12, -2.3e-16, 0.0, 2.3e-16, 1e-12)]
    x = np.concatenate([np.logspace(-6, 3.2, 200001), np.linspace(1e-3, 30, 100001), edges])
    j, y = np.empty_like(x), np.empty_like(x)
    dp = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    ctypes.CDLL(str(so)).h0(len(x), dp(x), dp(j), dp(y))
    ref = _reference(x)
    err = np.abs(j + 1j * y - ref) / np.abs(ref)
    assert np.all(err < 2e-15 + 2 * np.spacing(x)), (x[np.argmax(err)], err.max())
