"""The activity-bit stream takes one, two or four rows of the pair triangle per
wave, by size; the dense stream has chunks of its own.  Both forms agree bit for
bit at sizes of each kind, ragged in rows, columns and intervals; and a
standard-ADMM instance of many walls and few agents, whose group sums wall
contributions across a wave, equals plain launches."""
import pytest

from paper_1311_4527_amd import instances as I
from tests.test_gpu_group import _plain, _same, F_ADMM, F_DENSE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,eta,walls", [(3, 2, 2), (130, 3, 1), (525, 14, 3), (650, 13, 0), (900, 17, 2)])
def test_stream_rows_equal_dense(p, eta, walls):
    import torch
    from paper_1311_4527_amd.twa import Solver
    inst = I.random_box(p, 0.004, eta, n_walls=walls, sigma=1e-3, seed=8, alpha=0.1, C=1.0 / (p * eta))
    A, B = Solver.from_instance(inst), Solver.from_instance(inst, flags=F_DENSE)
    _plain(A, 24)
    _plain(B, 24)
    assert torch.equal(A.twa_get_trajectories(), B.twa_get_trajectories())
    assert A.twa_get_stats()["active_coll"] == B.twa_get_stats()["active_coll"]
    A.close(), B.close()


def test_group_of_walls_equals_plain():
    from paper_1311_4527_amd.twa import Solver
    inst = I.random_box(5, 0.02, 14, n_walls=32, sigma=1e-3, seed=9, alpha=0.1, C=0.01)
    A, B = Solver.from_instance(inst, flags=F_ADMM), Solver.from_instance(inst, flags=F_ADMM)
    A.twa_iterate(40)
    _plain(B, 40)
    _same(A, B)
    A.close(), B.close()
