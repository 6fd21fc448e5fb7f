"""Which batches run in groups at block 0, and with how many members each: a large
instance among more than the card holds at once keeps its shares; batches that
the phased launches run faster keep those.  The state is that of plain launches."""
import ctypes as ct

import pytest

from paper_1311_4527_amd import instances as I
from tests.test_gpu_group import _box, _plain, _same, F_ADMM, F_DENSE

pytestmark = pytest.mark.gpu


def _members(B, i):
    """Workgroups that ran instance i in the last launch (0: phased)."""
    from paper_1311_4527_amd import twa as T
    size, shares = ct.c_int(), ct.c_int()
    S = B.twa_batch_solver(i)
    st = T.load_library().twa_debug_group_members(S.h, 0, ct.byref(size), ct.byref(shares))
    assert st in (T.TWA_OK, T.TWA_E_STATE)
    return size.value if st == T.TWA_OK else 0


def _check(B, insts, which, k, flags=0):
    from paper_1311_4527_amd.twa import Solver
    for i in which:
        S = Solver.from_instance(insts[i], flags=flags)
        _plain(S, k)
        _same(B.twa_batch_solver(i), S)
        S.close()


def test_large_instance_among_many():
    from paper_1311_4527_amd.twa import Batch
    small = [I.circle_swap(6, 0.05, 2, seed=k) for k in range(7)]
    insts = [small[k % 7] for k in range(850)]
    insts[400] = _box(128, 8, 2)
    B = Batch(insts)
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(12)
    assert _members(B, 400) > 30 and _members(B, 3) == 1
    _check(B, insts, (0, 399, 400, 849), 12)
    B.close()


@pytest.mark.parametrize("n,p,eta,flags,groups", [
    (1, 128, 8, 0, True), (1, 200, 16, 0, False), (4, 200, 16, 0, True), (8, 440, 8, 0, False),
    (4, 70, 64, 0, False), (8, 70, 64, 0, True), (3, 30, 4, F_DENSE, False), (3, 30, 4, F_ADMM, False),
])
def test_groups_by_size(n, p, eta, flags, groups):
    from paper_1311_4527_amd.twa import Batch
    one = _box(p, eta, 0)
    B = Batch([one] * n, flags=flags)
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(8)
    assert (_members(B, 0) > 0) == groups
    _check(B, [one] * n, {0, n - 1}, 8, flags)
    B.close()
