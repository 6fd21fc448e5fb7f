"""The walks of the persistent batch over the rows of the pair triangle name every
chunk exactly once (compiled for the host)."""
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
extern "C" int rows(int p, int *count) { // the pairs of every task's rows
    for (int w = 0; w < bits_walk(p); ++w) {
        int i0 = -1, J = -1;
        bits_task(p, w, &i0, &J);
        if (i0 < 0 || i0 >= p - 1 || J < 0 || J > (p - 1) >> 6) return 1;
        for (int i = i0; i < i0 + kRows && i < p - 1; ++i)
            for (int j = 64 * J; j < 64 * J + 64; ++j)
                if (J >= ((i + 1) >> 6) && j > i && j < p) ++count[i * p + j];
    }
    return 0;
}
extern "C" int chunks(int p, int *count) {
    for (int w = 0; w < pair_chunks(p); ++w) {
        int i = -1, j0 = -1;
        pair_chunk(p, w, &i, &j0);
        if (i < 0 || j0 <= i || j0 >= p) return 1;
        for (int j = j0; j < j0 + 64 && j < p; ++j) ++count[i * p + j];
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lib():
    d = tempfile.mkdtemp(prefix="twa_walk_")
    src, so = os.path.join(d, "p.hip"), os.path.join(d, "p.so")
    with open(src, "w") as f:
        f.write(SRC % ROOT)
    subprocess.run(["hipcc", "-O2", "-fPIC", "-shared", "-std=c++17", "--offload-host-only", "-o", so, src], check=True)
    return ct.CDLL(so)


@pytest.mark.parametrize("walk", ["rows", "chunks"])
def test_every_pair_once(lib, walk):
    for p in list(range(2, 140)) + [191, 192, 193, 194, 256, 300]:
        count = np.zeros((p, p), dtype=np.int32)
        assert getattr(lib, walk)(ct.c_int(p), count.ctypes.data_as(ct.c_void_p)) == 0
        assert (count == np.triu(np.ones((p, p), np.int32), 1)).all(), p
