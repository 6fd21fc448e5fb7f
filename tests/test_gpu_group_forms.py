"""Which instances run in a group, and in how many shares, depends on the form;
with the most shares of each form the state equals that of plain launches."""
import ctypes as ct

import pytest

from tests.test_gpu_group import _box, _plain, _same, F_ADMM, F_DENSE

pytestmark = pytest.mark.gpu


def _shares(S):
    from paper_1311_4527_amd import twa as T
    size, shares = ct.c_int(), ct.c_int()
    st = T.load_library().twa_debug_group_members(S.h, 0, ct.byref(size), ct.byref(shares))
    assert st in (T.TWA_OK, T.TWA_E_STATE)
    return shares.value if st == T.TWA_OK else 0


@pytest.mark.parametrize("flags,p,eta,walls,shares", [
    (0, 60, 8, 0, 32), (0, 100, 16, 0, 64), (0, 200, 16, 7, 128), (0, 290, 17, 0, 0),
    (F_DENSE, 60, 8, 0, 32), (F_DENSE, 90, 10, 0, 64), (F_DENSE, 160, 16, 0, 128), (F_DENSE, 200, 16, 0, 0),
    (F_ADMM, 40, 8, 0, 32), (F_ADMM, 60, 8, 5, 64), (F_ADMM, 100, 8, 0, 128), (F_ADMM, 40, 8, 60, 128),
    (F_ADMM, 100, 16, 0, 0),
    # many nodes of few agents
    (0, 20, 150, 0, 32), (0, 20, 200, 0, 0), (0, 64, 70, 0, 64), (0, 64, 80, 0, 0), (F_DENSE, 8, 200, 0, 32),
    (F_DENSE, 8, 250, 0, 0), (F_ADMM, 5, 500, 0, 32), (F_ADMM, 5, 700, 0, 0),
])
def test_shares_by_form(flags, p, eta, walls, shares):
    from paper_1311_4527_amd.twa import Solver
    inst = _box(p, eta, walls)
    A, B = Solver.from_instance(inst, flags=flags), Solver.from_instance(inst, flags=flags)
    assert _shares(A) == shares
    A.twa_iterate(14)
    _plain(B, 14)
    _same(A, B)
    A.close(), B.close()
