"""The slope bound of the search with weight samples (CPU), the functions that ship (mist_bounds.h):
Algorithm 1's time, with both host streams longer by the same length, never grows by less than the least
slope over the orders in which the streams may finish; over the orders that start with GPU-GPU (and
compute after it) when they do so at the start."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import oracle as O
from paper_2503_19050_amd import build as B
from paper_2503_19050_amd import workloads as W

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")

LOWERED = 1.0 - 2.0 ** -30  # the kernel lowers every bound by this factor

SOURCE = r"""
#include "mist_bounds.h"
extern "C" void slopes(const double* phi, double* out) { mist::host_slopes((const double(*)[4])phi, out); }
extern "C" double any_length(double T, double sl, double h) { return mist::any_length(T, sl, h); }
extern "C" double largest() { return mist::kSlopeFactors; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bounds")
    (d / "b.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(B.CSRC), str(d / "b.cpp"), "-o", str(d / "b.so")], check=True)
    L = ctypes.CDLL(str(d / "b.so"))
    L.any_length.argtypes = [ctypes.c_double] * 3
    L.any_length.restype = L.largest.restype = ctypes.c_double
    return L


def _slopes(lib, phi):
    p = np.ascontiguousarray(phi, dtype=np.float64)
    out = np.zeros(3)
    D = ctypes.POINTER(ctypes.c_double)
    lib.slopes(p.ctypes.data_as(D), out.ctypes.data_as(D))
    return out


def _first(x, phi):
    """Which of the slopes holds: 0, 1 (GPU-GPU finishes first) or 2 (and compute after it)."""
    s = x * phi[15]
    if not 0.0 < s[1] < min(s[0], s[2], s[3]):
        return 0
    y = (s - s[1]) * (1.0 / phi[15]) * phi[13]
    return 2 if y[0] < min(y[2], y[3]) else 1


@pytest.mark.parametrize("hi", [1.0, 1.5, 50.0])
def test_time_grows_at_least_with_the_slope(hi, lib):
    rng = np.random.default_rng(int(hi * 10))
    for case in range(300):
        phi = np.array(W.hw_sample(case)["phi"]) if hi == 1.5 else 1.0 + (hi - 1.0) * rng.random((16, 4))
        x = rng.choice([0.0, 1.0], 4, p=[0.1, 0.9]) * 10.0 ** rng.uniform(-2, 2, 4)
        x[0] = max(x[0], 0.01)
        slopes = _slopes(lib, phi)
        assert slopes[0] <= slopes[1] <= slopes[2]
        slope = slopes[_first(x, phi)]
        T0 = O.interference(x, phi)
        for length in 10.0 ** rng.uniform(-3, 3, 8):
            T = O.interference(x + np.array([0.0, 0.0, length, length]), phi)
            assert (T0 + slope * length) * LOWERED <= T
            assert lib.any_length(T0, slope, max(x[2], x[3])) * LOWERED <= T


@pytest.mark.parametrize("exponent", [6, 8, 12, 16])
def test_the_bound_holds_for_rounded_times(exponent, lib):
    """Factors up to 2^exponent and streams whose scaled times nearly meet, where a round leaves little
    but rounding noise and the later ones scale it.  Factors above the largest that the slopes are for have
    no slope (-inf), and the maxima that the kernel takes are left with their other bounds."""
    rng = np.random.default_rng(exponent)
    for case in range(3000):
        phi = 2.0 ** (exponent * (rng.random((16, 4)) if case % 2 else rng.integers(0, 2, (16, 4))))
        phi[15, 0] = 2.0 ** exponent
        near = rng.choice([0.0, 1e-15, 1e-12, 1e-6, 0.1], 4) * rng.random(4)
        x = 2.0 ** rng.uniform(0, 3) / phi[15] * (1.0 + near)
        slopes = _slopes(lib, phi)
        if 2.0 ** exponent > lib.largest():
            assert np.all(slopes == -np.inf)
        slope = slopes[_first(x, phi)]
        T0 = O.interference(x, phi)
        for length in x[2] * 10.0 ** rng.uniform(-17, 1, 6):
            T = O.interference(x + np.array([0.0, 0.0, length, length]), phi)
            floor = max(x[0], x[1], x[2] + length, x[3] + length)
            for bound in (T0 + slope * length, lib.any_length(T0, slope, max(x[2], x[3]))):
                assert np.fmax(bound, floor) * LOWERED <= T
