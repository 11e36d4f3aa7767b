"""The reciprocal of a Gauss-Jordan pivot, compiled from its source for the
host with a hardware-like estimate (1 / d off by up to 2^-23 of itself): both
quotients have the bits of the divisions, at any scale of the pivot."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_11058_amd", "csrc", "gj.hip")

HOST = """
#include <cmath>
#include <cstdint>
using std::fma;
#define __device__
struct double2 { double x, y; };
static double2 make_double2(double x, double y) { return {x, y}; }
static double off;
static double estimate(double d) { return (1.0 / d) * (1.0 + off); }
%s
extern "C" void run(long n, const double* p, const double* e, double* out) {
  for (long i = 0; i < n; ++i) {
    off = e[i];
    const double2 r = gj_recip({p[2 * i], p[2 * i + 1]});
    out[2 * i] = r.x;
    out[2 * i + 1] = r.y;
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_bits_of_the_divisions(tmp_path):
    src = open(SRC).read()
    body = re.search(r"__device__ inline double2 gj_recip\(.*?\n}\n", src, re.S).group(0)
    cpp = tmp_path / "recip.cpp"
    cpp.write_text(HOST % body.replace("__builtin_amdgcn_rcp(", "estimate("))
    so = str(tmp_path / "recip.so")
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-shared", "-fPIC", str(cpp), "-o", so], check=True)
    rng = np.random.default_rng(3)
    n = 400_000
    p = rng.uniform(-2, 2, (n, 2)) * 2.0 ** rng.integers(-40, 41, (n, 2)) * 2.0 ** rng.integers(-400, 401, (n, 1))
    p[:50, 0] = 0.0
    p[50:100, 1] = 0.0
    e = rng.uniform(-2.0 ** -23, 2.0 ** -23, n)
    out = np.empty((n, 2))
    ctypes.CDLL(so).run(ctypes.c_long(n), *[ctypes.c_void_p(a.ctypes.data) for a in (p, e, out)])
    d = p[:, 0] * p[:, 0] + p[:, 1] * p[:, 1]
    for got, want in ((out[:, 0], p[:, 0] / d), (out[:, 1], -p[:, 1] / d)):
        # (a quotient below the normal range is rounded there; the residual is not exact any more)
        big = np.abs(want) > 1e-290
        assert np.count_nonzero((got != want) & big) == 0
