"""The double mode's exponential (exp64.hpp) compiled for the CPU, whose fused
multiply-adds round as the device's do, against 80-bit arithmetic: no larger an
error than the device library's exp, measured over the same ranges (0.861 ulp at
most, 0.2577 in the mean)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r'''
#define __device__
#define __forceinline__ inline
#include "exp64.hpp"
extern "C" void run(const double* d, double* o, long n) { for (long i = 0; i < n; ++i) o[i] = pf::exp_nonpos(d[i]); }
'''


@pytest.fixture(scope="module")
def exp_nonpos(tmp_path_factory):
    d = tmp_path_factory.mktemp("exp64")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2308_00763_amd", "csrc"), str(d / "shim.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)

    def run(x):
        x = np.ascontiguousarray(x, dtype=np.float64)
        out = np.empty_like(x)
        lib.run(ctypes.c_void_p(x.ctypes.data), ctypes.c_void_p(out.ctypes.data), ctypes.c_long(x.size))
        return out
    return run


@pytest.mark.parametrize("lo", [-0.35, -1.0, -23.0, -100.0, -708.0, -745.2])
def test_error_within_the_librarys(exp_nonpos, lo):
    hi = -708.0 if lo < -708 else 0.0  # the subnormal results by themselves
    d = np.random.default_rng(7).uniform(lo, hi, 1 << 20)
    ref = np.exp(d.astype(np.longdouble))
    err = np.abs((exp_nonpos(d).astype(np.longdouble) - ref) / np.spacing(ref.astype(np.float64)))
    print(f"[exp64] {lo}..{hi} max {float(err.max()):.4f} mean {float(err.mean()):.4f}")
    assert err.max() <= 0.861 and err.mean() <= 0.2577


def test_ends(exp_nonpos):
    x = np.array([0.0, -0.0, -1e-320, -745.13, -745.14, -800.0, -801.0, -1e300, -np.inf])
    want = np.array([1.0, 1.0, 1.0, 5e-324, 0.0, 0.0, 0.0, 0.0, 0.0])
    assert np.array_equal(exp_nonpos(x), want)
    assert np.isnan(exp_nonpos(np.array([np.nan])))[0]
