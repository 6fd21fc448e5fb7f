"""quotient() and rounded_root() give n / d and sqrtf(x) to the last bit over the
ranges the minimisers use them in, from any estimate within an ulp; a divisor
of all ones (2 - 2^-23 times a power of two) wants the correctly rounded one.
Compiled for the host."""
import ctypes as ct
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "%s/paper_1311_4527_amd/csrc/prox.h"
#include <cmath>
using namespace twa;
static float nudge(float v, int by) {
    for (; by > 0; --by) v = nextafterf(v, INFINITY);
    for (; by < 0; ++by) v = nextafterf(v, 0.f);
    return v;
}
extern "C" long check_div(long n, const float *a, const float *d, int by) {
    long bad = 0;
    for (long k = 0; k < n; ++k)
        bad += quotient(a[k], d[k], refined_rcp(d[k], nudge(1.f / d[k], by))) != a[k] / d[k];
    return bad;
}
extern "C" long check_root(long n, const float *x, int by) {
    long bad = 0;
    for (long k = 0; k < n; ++k) bad += rounded_root(x[k], nudge(sqrtf(x[k]), by)) != sqrtf(x[k]);
    return bad;
}
"""


@pytest.fixture(scope="module")
def lib():
    d = tempfile.mkdtemp(prefix="twa_quot_")
    src, so = os.path.join(d, "q.hip"), os.path.join(d, "q.so")
    with open(src, "w") as f:
        f.write(SRC % ROOT)
    subprocess.run(["hipcc", "-O2", "-mfma", "-ffp-contract=on", "-fPIC", "-shared", "-std=c++17", "--offload-host-only",
                    "-o", so, src], check=True)
    so = ct.CDLL(so)
    so.check_div.restype = so.check_root.restype = ct.c_long
    return so


def _p(a):
    return a.ctypes.data_as(ct.c_void_p)


def _floats(rng, n, lo, hi):
    m = 1 + rng.integers(0, 1 << 23, n) / float(1 << 23)
    edge = rng.random(n) < 0.2  # mantissas next to a power of two
    m = np.where(edge, 1 + rng.integers(0, 4, n) / float(1 << 23), m)
    m = np.where(rng.random(n) < 0.1, 2 - rng.integers(1, 4, n) / float(1 << 23), m)
    return (m * 2.0 ** rng.integers(lo, hi, n)).astype(np.float32)


@pytest.mark.parametrize("by", [-1, 0, 1])
def test_quotients(lib, by):
    rng = np.random.default_rng(3 + by)
    n = 4_000_000
    for (alo, ahi), (dlo, dhi) in (((-2, 2), (-2, 2)), ((-83, 41), (-13, 30)), ((-23, 41), (-13, 71)), ((0, 1), (-41, 2))):
        a = _floats(rng, n, alo, ahi) * rng.choice(np.float32([-1, 1]), n)
        d = _floats(rng, n, dlo, dhi)
        if by:
            ones = (d.view(np.uint32) & 0x7FFFFF) == 0x7FFFFF
            d[ones] = np.float32(1.5)
        assert lib.check_div(ct.c_long(n), _p(a), _p(d), ct.c_int(by)) == 0


@pytest.mark.parametrize("by", [-1, 0, 1])
def test_roots(lib, by):
    x = _floats(np.random.default_rng(13 + by), 8_000_000, -84, 4)
    assert lib.check_root(ct.c_long(x.size), _p(x), ct.c_int(by)) == 0
