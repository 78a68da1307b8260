"""Sine and cosine of the continuous wave's phase (host build of the kernels'
function, no GPU) against references whose reduction uses 1400 bits of pi: every
binade from 2^-40 to the largest double, the doubles next to multiples of pi/2
among them, and infinities and NaN.

Bar: 4 units of 2^-53 absolute.  The remainder carries one rounding (1 unit) and
n 2^-109, the series truncates below half a unit and rounds twice."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_06834_amd", "csrc")
BITS = 1400

SOURCE = """
#include "phase_dev.h"
extern "C" void phase(int far, int n, const double *x, double *s, double *c) {
  for (int i = 0; i < n; ++i)
    if (far) pt::sincos_phase<true>(x[i], s[i], c[i]);
    else pt::sincos_phase<false>(x[i], s[i], c[i]);
}
"""


def arctan_inverse(q, one):
    total, term, k, sign = 0, one // q, 1, 1
    while term:
        total += sign * (term // k)
        term //= q * q
        k, sign = k + 2, -sign
    return total


ONE = 1 << BITS
PI = 4 * (4 * arctan_inverse(5, ONE) - arctan_inverse(239, ONE))   # pi 2^BITS


def reference(x):
    m, e = math.frexp(x)
    v = int(m * (1 << 53))
    e += BITS - 53
    v = v << e if e >= 0 else v >> -e           # x 2^BITS (exact, or far below the bar)
    n = (2 * v + PI // 2) // PI                 # nearest multiple of pi/2
    r = (2 * v - n * PI) / (2 * ONE)            # (true division of integers: correctly rounded)
    s, c = math.sin(r), math.cos(r)
    return [(s, c), (c, -s), (-s, -c), (-c, s)][n & 3]


@pytest.fixture(scope="module")
def phase(tmp_path_factory):
    from paper_2607_06834_amd import build as b
    d = tmp_path_factory.mktemp("phase")
    (d / "host.hip").write_text(SOURCE)
    subprocess.run([b.HIPCC, *b.FLAGS, "-shared", str(d / "host.hip"), "-o", str(d / "host.so")], check=True,
                   capture_output=True)
    lib = ctypes.CDLL(str(d / "host.so"))

    def call(x, far):
        x = np.ascontiguousarray(x, np.float64)
        s, c = np.empty_like(x), np.empty_like(x)
        p = [a.ctypes.data_as(ctypes.c_void_p) for a in (x, s, c)]
        lib.phase(int(far), x.size, *p)
        return s, c
    return call


def arguments(lo, hi):
    rng = np.random.default_rng(7)
    x = [0.0]
    for e in range(lo, hi):
        x += list(np.ldexp(rng.uniform(1.0, 2.0, 24), e))
        x += [math.ldexp(1.0, e), math.ldexp(2.0 - 2.0 ** -52, e)]
        if e >= 1:                              # the nearest to multiples of pi/2
            for u in rng.integers(1 << 52, 1 << 53, 8):
                n = (2 * int(u) << BITS + e) // (PI << 53)
                x.append(n * PI / (2 * ONE))
    if hi > 900:
        x.append(math.ldexp(6381956970095103.0, 797))   # 2^-61 from one
    x = np.array(x)
    return np.concatenate([x, -x])


def check(got, x):
    ref = np.array([reference(float(v)) for v in x])
    err = np.maximum(np.abs(got[0] - ref[:, 0]), np.abs(got[1] - ref[:, 1]))
    assert err.max() <= 4 * 2.0 ** -53, (x[err.argmax()], err.max())


def test_short_reduction(phase):
    x = arguments(-40, 45)
    check(phase(x, False), x)
    check(phase(x, True), x)


def test_any_argument(phase):
    x = arguments(45, 1024)
    check(phase(x, True), x)
    s, c = phase([np.inf, -np.inf, np.nan], True)
    assert np.all(np.isnan(s)) and np.all(np.isnan(c))
