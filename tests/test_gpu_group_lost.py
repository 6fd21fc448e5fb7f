"""A wait inside a group of resident workgroups that ran out: every way to the
results says so, and no launch waits that long again.  The flag that a member
sets when it gives up is set from the host here; no wait ever runs out."""
import pytest

from paper_1311_4527_amd import instances as I
from tests.test_gpu_group import _swap

pytestmark = pytest.mark.gpu


def _lose(S, batch=0):
    from paper_1311_4527_amd import twa as T
    assert T.load_library().twa_debug_group_stuck(S.h, batch) == T.TWA_OK


def _raises(call):
    from paper_1311_4527_amd import twa as T
    with pytest.raises(T.TWAError) as e:
        call()
    assert e.value.status == T.TWA_E_DEVICE


CALLS = {
    "quality": lambda S: S.twa_get_quality(),
    "stats": lambda S: S.twa_get_stats(),
    "finite": lambda S: S.twa_check_finite(),
    "until": lambda S: S.twa_iterate_until(100, 10, -1e9),  # (any plan would meet the bar)
}


@pytest.mark.parametrize("call", sorted(CALLS))
def test_results_of_a_lost_group(call):
    import torch
    from paper_1311_4527_amd.twa import Solver
    S = Solver.from_instance(_swap(18, 4))
    S.twa_iterate(20)
    assert not torch.isnan(S.twa_get_trajectories()).any()
    _lose(S)
    assert torch.isnan(S.twa_get_trajectories()).all()
    assert torch.isnan(S.twa_get_state()[0]).all()
    S.twa_iterate(2000)                       # queued: ends at once
    assert torch.isnan(S.twa_get_trajectories()).all()
    _raises(lambda: CALLS[call](S))
    _raises(lambda: S.twa_iterate(1))         # latched
    S.close()


def test_backward_of_a_lost_group():
    import torch
    from paper_1311_4527_amd.twa import Solver, TWA_F_TAPE
    S = Solver.from_instance(_swap(18, 4), flags=TWA_F_TAPE)
    S.twa_iterate(40)
    dz = torch.ones_like(S.twa_get_trajectories())
    S.twa_backward(dz)
    _lose(S)
    _raises(lambda: S.twa_backward(dz))
    S.close()


def test_batch_with_a_lost_group():
    import torch
    from paper_1311_4527_amd.twa import Batch
    insts = [_swap(18, 4), I.circle_swap(26, 0.05, 5, seed=3)]
    B = Batch(insts)
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(10)
    _lose(B.twa_batch_solver(0), batch=1)
    assert torch.isnan(B.twa_batch_get_trajectories(0)).all()
    assert not torch.isnan(B.twa_batch_get_trajectories(1)).any()
    B.twa_batch_iterate(10)
    _raises(lambda: B.twa_batch_solver(0).twa_get_quality())
    _raises(lambda: B.twa_batch_iterate(1))
    B.close()
