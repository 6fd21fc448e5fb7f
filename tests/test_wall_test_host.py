"""The wall factors' activity test with its early answer for far pairs
(segseg_below) gives, bit for bit, segseg_sq(...) < r * r, compiled for the
host: random pairs, pairs at the radius within a few roundings, collinear and
parallel ones, degenerate segments, large coordinates, non-finite ends."""
import ctypes as ct
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "%s/paper_1311_4527_amd/csrc/prox.h"
using namespace twa;
extern "C" long run(long n, const float *v, const float *r, long *far) {
    long bad = 0;
    *far = 0;
    for (long k = 0; k < n; ++k) {
        const float *q = v + 8 * k;
        f2 p0 = mk(q[0], q[1]), p1 = mk(q[2], q[3]), q0 = mk(q[4], q[5]), q1 = mk(q[6], q[7]);
        const bool want = segseg_sq(p0, p1, q0, q1) < r[k] * r[k];
        bad += segseg_below(p0, p1, q0, q1, r[k]) != want;
        *far += !want;
    }
    return bad;
}
"""


@pytest.fixture(scope="module")
def lib():
    d = tempfile.mkdtemp(prefix="twa_wall_")
    src, so = os.path.join(d, "w.hip"), os.path.join(d, "w.so")
    with open(src, "w") as f:
        f.write(SRC % ROOT)
    subprocess.run(["hipcc", "-O2", "-ffp-contract=on", "-fPIC", "-shared", "-std=c++17", "--offload-host-only", "-o",
                    so, src], check=True)
    return ct.CDLL(so)


def _check(lib, v, r):
    v = np.ascontiguousarray(v, dtype=np.float32)
    r = np.ascontiguousarray(np.broadcast_to(np.asarray(r, dtype=np.float32), v.shape[0]))
    far = ct.c_long()
    lib.run.restype = ct.c_long
    bad = lib.run(ct.c_long(v.shape[0]), v.ctypes.data_as(ct.c_void_p), r.ctypes.data_as(ct.c_void_p), ct.byref(far))
    assert bad == 0
    return far.value / v.shape[0]


def test_random_pairs(lib):
    rng = np.random.default_rng(0)
    n = 400_000
    c = rng.uniform(0, 1, (n, 2, 2))
    d = rng.normal(0, 1, (n, 2, 2)) * rng.choice([0.01, 0.05, 0.3], (n, 2, 1))
    v = np.concatenate([c[:, 0] - d[:, 0], c[:, 0] + d[:, 0], c[:, 1] - d[:, 1], c[:, 1] + d[:, 1]], 1)
    assert _check(lib, v, 0.01) > 0.5
    _check(lib, v, 0.2)
    _check(lib, v * 1000.0 + 5000.0, 3.0)
    _check(lib, v * 1e-6, 1e-8)


def test_at_the_radius(lib):
    """Ends at the distance r from the other segment, to a few roundings."""
    rng = np.random.default_rng(1)
    n = 200_000
    a, b = rng.uniform(-1, 1, (n, 2)), rng.uniform(-1, 1, (n, 2))
    r = rng.choice([1e-4, 0.01, 0.3], n)
    t = rng.uniform(-0.3, 1.3, (n, 1))
    w = b - a
    nrm = np.stack([-w[:, 1], w[:, 0]], 1) / np.linalg.norm(w, axis=1)[:, None]
    k = 1.0 + rng.integers(-40, 41, n) * 6e-8
    foot = a + np.clip(t, 0, 1) * w
    away = np.where((t < 0) | (t > 1), (a + t * w - foot) / np.maximum(np.linalg.norm(a + t * w - foot, axis=1), 1e-9)[:, None], nrm)
    p = foot + away * (r * k)[:, None]
    p2 = p + away * rng.uniform(0, 0.5, (n, 1)) + nrm * 1e-3 * rng.normal(size=(n, 1))
    v = np.concatenate([p, p2, a, b], 1)
    _check(lib, v, r)
    _check(lib, v[:, [4, 5, 6, 7, 0, 1, 2, 3]], r)


def test_collinear_degenerate_and_non_finite(lib):
    rng = np.random.default_rng(2)
    n = 100_000
    a, u = rng.uniform(-1, 1, (n, 2)), rng.normal(size=(n, 2))
    t = np.sort(rng.uniform(-1, 1, (n, 4)), 1)[:, rng.permutation(4)]
    v = np.concatenate([a + t[:, [k]] * u for k in range(4)], 1)          # collinear up to rounding
    for r in (1e-5, 0.01, 0.2):
        _check(lib, v, r)
    g = rng.integers(-3, 4, (n, 8)).astype(np.float64) / 4                # exact collinearity, shared points
    for r in (0.05, 0.25, 0.5):
        _check(lib, g, r)
    point = v.copy()
    point[:, 6:8] = point[:, 4:6]                                         # a wall of no length
    _check(lib, point, 0.05)
    point[:, 2:4] = point[:, 0:2]
    _check(lib, point, 0.05)
    tiny = v.copy()
    tiny[:, 6:8] = tiny[:, 4:6] * (1 + 1e-7)
    _check(lib, tiny, 0.05)
    odd = v.copy()
    odd[np.arange(n), rng.integers(0, 4, n)] = rng.choice([np.nan, np.inf, -np.inf, 1e30], n)
    _check(lib, odd, 0.05)
