"""The two forms of c2p_setup (pb_c2p.h, compiled for the host) bracket the
root alike: the one that takes the square root only where s - E can be
positive must find the same lower end, bit for bit, as the one that always
takes it, and the same cells admissible.  Values next to the boundary s = E,
extreme scales, zeros, infinities and NaN, as arguments of the function."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_19273_amd", "csrc")

SRC = """
#define __device__
#define __forceinline__ inline
#include <cmath>
using std::isfinite;
static inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }
static inline double __builtin_amdgcn_rsq(double x) { return 1.0 / std::sqrt(x); }
#include "pb_c2p.h"
extern "C" void setup(int n, const double *D, const double *S, const double *tau, double *lo, double *hi, int *ok)
{
    for (int i = 0; i < n; ++i) {
        const pb::C2pIn a = pb::c2p_setup<true>(D[i], S[i], 0.0, 0.0, tau[i], 5.0 / 3.0);
        const pb::C2pIn b = pb::c2p_setup<false>(D[i], S[i], 0.0, 0.0, tau[i], 5.0 / 3.0);
        lo[i] = a.lo; lo[n + i] = b.lo;
        hi[i] = a.hi; hi[n + i] = b.hi;
        ok[i] = a.ok; ok[n + i] = b.ok;
    }
}
"""


@pytest.fixture(scope="module")
def setup(tmp_path_factory):
    d = tmp_path_factory.mktemp("c2p")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#pragma once\n")   # the header needs nothing of it on the host
    (d / "t.cpp").write_text(SRC)
    so = str(d / "t.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I", str(d), "-I", CSRC,
                           "-o", so, str(d / "t.cpp")])
    f = C.CDLL(so).setup
    f.argtypes = [C.c_int] + [C.c_void_p] * 6

    def call(D, S, tau):
        n = len(D)
        D, S, tau = (np.ascontiguousarray(v, np.float64) for v in (D, S, tau))
        lo, hi, ok = np.empty((2, n)), np.empty((2, n)), np.empty((2, n), np.int32)
        f(n, *(v.ctypes.data for v in (D, S, tau, lo, hi, ok)))
        return lo, hi, ok

    return call


def test_both_forms_bracket_alike(setup):
    rng = np.random.default_rng(5)
    n = 20000
    # E over the whole range of binary64 and near one; s within 120 roundings
    # of E and, a quarter of them, up to a tenth away
    E = np.concatenate([10.0 ** rng.uniform(-300, 150, n), rng.uniform(0.5, 2, n)])
    D = E * 10.0 ** rng.uniform(-12, -0.01, E.size)
    tau = E - D
    with np.errstate(all="ignore"):
        S = (tau + D) * (1.0 + rng.integers(-120, 121, E.size) * 2.0**-53)
        S = np.where(rng.random(E.size) < 0.25, S * rng.uniform(0.9, 1.1, E.size), S)
        sp = np.array([0.0, -0.0, 5e-324, 1e-160, 1.0, -1.0, 1e154, 1e200, np.inf, -np.inf, np.nan])
        a, b, c = (v.ravel() for v in np.meshgrid(sp, sp, sp))
        D, S, tau = np.concatenate([D, a]), np.concatenate([S, b]), np.concatenate([tau, c])
        lo, hi, ok = setup(D, S, tau)
    np.testing.assert_array_equal(lo[0], lo[1])
    np.testing.assert_array_equal(hi[0], hi[1])
    np.testing.assert_array_equal(ok[0], ok[1])
    # both sides of the boundary were met, next to it and away from it
    near = np.abs(S[:2 * n] - E) < 1e-13 * E
    assert np.sum(near & (lo[0][:2 * n] > 0)) > 1000 and np.sum(near & (lo[0][:2 * n] == 0)) > 1000
    assert np.sum(~near & (lo[0][:2 * n] > 0)) > 1000 and np.any(ok[0]) and not np.all(ok[0])
