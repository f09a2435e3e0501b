"""The FP64 exponentials of the cells outside the temperature tables, compiled
for the host, against the C library over their whole range."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2607_01338_amd import build

SRC = """
#include "rare_exp.h"
extern "C" void exps(const double* x, double* e, double* m, long n) {
  for (long i = 0; i < n; ++i) {
    e[i] = iris::exp_rare(x[i]);
    m[i] = iris::expm1_rare(x[i]);
  }
}
"""


@pytest.fixture(scope="module")
def exps(tmp_path_factory):
    d = tmp_path_factory.mktemp("rare_exp")
    src, lib = str(d / "exps.hip"), str(d / "libexps.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([build.HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-shared", "-fPIC",
                    "-I", build.CSRC, src, "-o", lib], check=True, capture_output=True,
                   env=dict(os.environ, HIP_PLATFORM="amd"))
    fn = ctypes.CDLL(lib).exps
    fn.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long]

    def call(x):
        x = np.ascontiguousarray(x, dtype=np.float64)
        e, m = np.empty_like(x), np.empty_like(x)
        fn(x.ctypes.data, e.ctypes.data, m.ctypes.data, x.size)
        return e, m

    return call


def test_whole_range(exps):
    rng = np.random.default_rng(1)
    x = np.concatenate([rng.uniform(-2000, 2000, 100000), rng.uniform(700, 720, 20000),
                        rng.uniform(-760, -700, 20000), np.linspace(44, 46, 4001),
                        rng.uniform(-2, 2, 20000), 10.0 ** rng.uniform(-300, 0, 5000),
                        -(10.0 ** rng.uniform(-300, 0, 5000)),
                        np.nextafter(np.log(np.finfo(float).max), [0.0, np.inf])])
    e, m = exps(x)
    with np.errstate(over="ignore", under="ignore"):
        re, rm = np.exp(x), np.expm1(x)
    # A few ulp: half an ulp each for the reduced argument, the last two steps
    # of the series and the sums; a subnormal result to its last bit. The
    # smallest x that overflows may lie a few ulp of the result off.
    edge = np.abs(x - np.log(np.finfo(float).max)) < 1e-12
    for got, ref in ((e, re), (m, rm)):
        assert not np.any(np.isnan(got))
        big = np.isinf(ref) & ~edge
        assert np.all(got[big] == np.inf)
        fin = np.isfinite(ref) & ~edge
        tol = 4 * np.finfo(float).eps * np.abs(ref[fin]) + 5e-324
        assert np.all(np.abs(got[fin] - ref[fin]) <= tol)


def test_special_values(exps):
    e, m = exps([np.inf, -np.inf, np.nan, 0.0])
    assert e[0] == np.inf and e[1] == 0.0 and np.isnan(e[2]) and e[3] == 1.0
    assert m[0] == np.inf and m[1] == -1.0 and np.isnan(m[2]) and m[3] == 0.0
