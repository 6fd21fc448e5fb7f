"""Calls of few iterations: where a group's launch costs more than it saves, the
plain and phased launches run; any mix of calls gives the plain state."""
import ctypes as ct

import pytest

from tests.test_gpu_group import _box, _plain, _same, F_DENSE

pytestmark = pytest.mark.gpu


def _members(S):
    """Workgroups of the last group launch (0: none yet)."""
    from paper_1311_4527_amd import twa as T
    size, shares = ct.c_int(), ct.c_int()
    assert T.load_library().twa_debug_group_members(S.h, 0, ct.byref(size), ct.byref(shares)) == T.TWA_OK
    return size.value


@pytest.mark.parametrize("p,eta,flags,least", [(60, 8, 0, 1), (100, 16, 0, 2), (200, 16, 0, 2), (140, 16, F_DENSE, 6)])
def test_group_from_so_many_iterations_on(p, eta, flags, least):
    from paper_1311_4527_amd.twa import Solver
    inst = _box(p, eta, 0)
    A, B = Solver.from_instance(inst, flags=flags), Solver.from_instance(inst, flags=flags)
    A.twa_iterate(1)
    ran = 1
    for k in range(1, least):
        A.twa_iterate(k)
        ran += k
        assert _members(A) == 0
    for k in (least, 1, least + 3, 1, 1):
        A.twa_iterate(k)
        ran += k
        assert _members(A) > 0
    _plain(B, ran - ran % 2)
    if ran % 2:
        B.twa_iterate_timed(1)
    _same(A, B)
    A.close(), B.close()


def test_batch_of_single_iterations():
    from paper_1311_4527_amd.twa import Batch, Solver
    insts = [_box(60, 5, 2), _box(9, 3, 9), _box(66, 4, 0, dim=3)]
    B = Batch(insts)
    B.twa_batch_config(0, 1)
    for _ in range(3):
        B.twa_batch_iterate(1)
    assert _members(B.twa_batch_solver(0)) == 0
    B.twa_batch_iterate(2)
    assert _members(B.twa_batch_solver(0)) > 0
    for k in (1, 5, 1, 1):
        B.twa_batch_iterate(k)
    for i, inst in enumerate(insts):
        S = Solver.from_instance(inst)
        _plain(S, 12)
        S.twa_iterate_timed(1)
        _same(B.twa_batch_solver(i), S)
        S.close()
    B.close()
