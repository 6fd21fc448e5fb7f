"""The cyclic walk of a batch's groups names every pair of agents exactly once,
as its items cut it (compiled for the host)."""
import ctypes as ct
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "%s/paper_1311_4527_amd/csrc/pairs.h"
using namespace twa;
extern "C" void run(int p, int *count) {
    const int blocks = (p + 63) / 64, items = cyclic_items(p), spans = blocks ? items / blocks : 0;
    for (int m = 0; m < items; ++m)
        for (int r = 0; r < kGroupSpan; ++r)
            for (int lane = 0; lane < 64; ++lane) {
                int i = 0, j = 0;
                if (group_pair(p, m / spans, 1 + m %% spans * kGroupSpan + r, lane, &i, &j)) {
                    if (i < 0 || j <= i || j >= p) count[0] = -1000000;
                    else ++count[i * p + j];
                }
            }
}
"""


@pytest.fixture(scope="module")
def lib():
    d = tempfile.mkdtemp(prefix="twa_pairs_")
    src, so = os.path.join(d, "p.hip"), os.path.join(d, "p.so")
    with open(src, "w") as f:
        f.write(SRC % ROOT)
    subprocess.run(["hipcc", "-O2", "-fPIC", "-shared", "-std=c++17", "--offload-host-only", "-o", so, src], check=True)
    return ct.CDLL(so)


def test_every_pair_once(lib):
    for p in list(range(1, 140)) + [191, 192, 193, 256, 300]:
        count = np.zeros((p, p), dtype=np.int32)
        lib.run(ct.c_int(p), count.ctypes.data_as(ct.c_void_p))
        assert (count == np.triu(np.ones((p, p), np.int32), 1)).all(), p
