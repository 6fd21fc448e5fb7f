"""Mid-sized instances: steady untimed iterations run in a group of resident
workgroups, all iterations of a call in one launch.  The per-factor code and
the exact sums are the plain kernels', so the state after any mix of such calls
and plain iterations equals, bit for bit, the state after plain iterations
alone (twa_iterate_timed launches its last two iterations on their own, so
calls of two timed iterations run plain throughout)."""
import pytest

from paper_1311_4527_amd import instances as I

pytestmark = pytest.mark.gpu

F_DENSE, F_ADMM, F_NONE, F_MAXVEL, F_MINVEL, F_VO = 1, 4, 8, 16, 32, 64


def _box(p, eta, walls, dim=2, seed=11):
    return I.random_box(p, 0.01, eta, n_walls=walls, dim=dim, sigma=1e-3, seed=seed, alpha=0.1, C=1.0 / (p * eta))


def _swap(p, eta, dim=2, seed=12):
    return I.circle_swap(p, min(0.05, 2.0 / p), eta, dim=dim, seed=seed, alpha=0.1, C=1.0 / (p * eta))


CASES = {
    "swap18_eta4": lambda: _swap(18, 4),              # 612 collision factors: just past the one-workgroup path
    "swap26_odd_eta": lambda: _swap(26, 5, dim=3),    # a last item of one interval
    "box9_walls": lambda: _box(9, 3, 9),              # 243 wall factors: a ragged last unit, shares without any
    "box65_rows_of_64": lambda: _box(65, 6, 3),       # a row of exactly one chunk
    "box66_3d": lambda: _box(66, 7, 0, dim=3),        # a row one pair past a chunk
    "swap100": lambda: _swap(100, 8),                 # several thousand active at the start: queues past a wave
    "box128_64_shares": lambda: _box(128, 12, 5),
    "box200_128_shares": lambda: _box(200, 16, 7),
    "pair_long": lambda: I.circle_swap(2, 0.05, 3000, seed=4),  # 3000 columns of one pair
}


def _state(S):
    import torch
    z, u, lr, it = S.twa_get_state()
    torch.cuda.synchronize()
    return z.cpu(), u.cpu(), lr.cpu(), it


def _plain(S, k):
    for _ in range(k // 2):
        S.twa_iterate_timed(2)


def _same(A, B):
    import torch
    a, b = _state(A), _state(B)
    assert a[3] == b[3]
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y)
    sa, sb = A.twa_get_stats(), B.twa_get_stats()
    sa.pop("graph_iterations"), sb.pop("graph_iterations")
    assert sa == sb


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("flags", [0, F_DENSE])
def test_group_equals_plain(case, flags):
    from paper_1311_4527_amd.twa import Solver
    inst = CASES[case]()
    A, B = Solver.from_instance(inst, flags=flags), Solver.from_instance(inst, flags=flags)
    A.twa_iterate(21)         # a plain first iteration, then the group
    assert A.twa_get_stats()["graph_iterations"] == 20
    A.twa_iterate(2)          # from a settled state: one iteration in the group
    A.twa_iterate_timed(3)    # plain iterations in between
    A.twa_iterate(34)
    _plain(B, 60)
    _same(A, B)
    A.close(), B.close()


@pytest.mark.parametrize("flags", [F_ADMM, F_NONE, F_MAXVEL, F_MINVEL, F_NONE | F_DENSE])
@pytest.mark.parametrize("case", ["box65_rows_of_64", "swap26_odd_eta"])
def test_group_equals_plain_modes(case, flags):
    import numpy as np
    from paper_1311_4527_amd.twa import Solver
    inst = CASES[case]()
    if flags & (F_MAXVEL | F_MINVEL):
        step = np.linalg.norm(inst.xT - inst.x0, axis=1) / inst.eta
        inst.C = np.repeat((step * (1.3 if flags & F_MAXVEL else 0.8))[:, None], inst.eta, axis=1)
    A, B = Solver.from_instance(inst, flags=flags), Solver.from_instance(inst, flags=flags)
    A.twa_iterate(40)
    A.twa_iterate(20)
    _plain(B, 60)
    _same(A, B)
    A.close(), B.close()


def test_group_queue_drained_within_an_iteration():
    """Standard ADMM queues every factor: with 150 walls a share holds 1,125
    wall factors, more than its queue, which is emptied in between."""
    from paper_1311_4527_amd.twa import Solver
    inst = I.random_box(40, 0.005, 6, n_walls=150, wall_len=(0.01, 0.03), sigma=1e-3, seed=3, alpha=0.1, C=0.01)
    A, B = Solver.from_instance(inst, flags=F_ADMM), Solver.from_instance(inst, flags=F_ADMM)
    A.twa_iterate(8)
    assert A.twa_get_stats()["graph_iterations"] == 7
    _plain(B, 8)
    _same(A, B)
    A.close(), B.close()


def test_group_vo_epoch():
    from paper_1311_4527_amd.twa import Solver
    inst = I.circle_swap(60, 0.02, 1, seed=5, alpha=0.1, C=0.05)
    A, B = Solver.from_instance(inst, flags=F_VO), Solver.from_instance(inst, flags=F_VO)
    A.twa_iterate(90)
    _plain(B, 90)
    _same(A, B)
    A.close(), B.close()


def test_group_from_a_state_that_moved_the_ends():
    """A loaded state with u on the fixed edges and moved end points: the fixed
    nodes come back exactly, as in the plain launches."""
    import numpy as np
    import torch
    from paper_1311_4527_amd.twa import Solver
    inst = CASES["swap26_odd_eta"]()
    z, u, lr = I.random_state(inst, 3)
    z[:, 0] += 0.01
    u[: 2 * inst.p] = 0.02
    S = []
    for k in range(2):
        s = Solver.from_instance(inst)
        s.twa_set_state(*(torch.from_numpy(np.asarray(a, dtype=t)) for a, t in
                          ((z, np.float32), (u, np.float32), (lr, np.uint8))), 0)
        S.append(s)
    S[0].twa_iterate(12)
    _plain(S[1], 12)
    _same(*S)
    for s in S:
        s.close()


def test_group_two_solvers_on_two_streams():
    """Two groups in flight at once keep to themselves."""
    import torch
    from paper_1311_4527_amd.twa import Solver
    insts = [CASES["swap100"](), CASES["box128_64_shares"]()]
    runs = [Solver.from_instance(i, stream=torch.cuda.Stream()) for i in insts]
    for _ in range(5):
        for s in runs:
            s.twa_iterate(40)
    for s, i in zip(runs, insts):
        s.stream.synchronize()
        R = Solver.from_instance(i)
        R.twa_iterate(200)
        _same(s, R)
        R.close(), s.close()


def test_group_with_a_warm_up_schedule():
    from paper_1311_4527_amd.twa import Solver
    inst = CASES["swap18_eta4"]()
    A, B = Solver.from_instance(inst), Solver.from_instance(inst)
    for s in (A, B):
        s.twa_set_schedule(0.25, 7)
    A.twa_iterate(50)
    _plain(B, 50)
    _same(A, B)
    A.close(), B.close()
