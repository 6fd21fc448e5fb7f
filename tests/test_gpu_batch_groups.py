"""Batches at block 0: steady iterations run in a group of resident workgroups
per instance, all groups in one launch.  The state, activity and counts after
any mix of such calls, a captured iteration and the members' own launches equal,
bit for bit, those of plain launches alone."""
import numpy as np
import pytest

from paper_1311_4527_amd import instances as I
from tests.test_gpu_group import _box, _plain, _same, _swap, F_MAXVEL, F_MINVEL, F_NONE

pytestmark = pytest.mark.gpu

MEMBERS = {
    "edges": lambda: [I.circle_swap(2, 0.05, 5, seed=1), _box(3, 2, 1), _box(9, 3, 9), _swap(26, 5, dim=3), _box(63, 4, 2),
                      _box(64, 3, 0), _box(65, 6, 3), _box(66, 7, 0, dim=3), _box(128, 3, 1), _box(129, 2, 1)],
    "one_agent": lambda: [I.random_box(1, 0.01, 4, n_walls=2, sigma=1e-3, seed=2, alpha=0.1, C=0.1), _box(30, 5, 3)],
    "crowded": lambda: [_swap(100, 6), _swap(60, 8), _swap(40, 3)],   # queues emptied within an iteration
    "large": lambda: [_box(200, 16, 7), _box(20, 4, 4)],              # 64 shares beside one
}


@pytest.mark.parametrize("members", sorted(MEMBERS))
def test_batch_groups_equal_plain(members):
    import torch
    from paper_1311_4527_amd.twa import Batch, Solver
    insts = MEMBERS[members]()
    B = Batch(insts)
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(12)      # a plain first iteration, then the groups
    B.twa_batch_iterate(1)
    caught = [torch.empty((B.twa_batch_solver(0).n_edges, insts[0].dim), dtype=torch.float32, device="cuda"),
              torch.empty((B.twa_batch_solver(0).n_factors,), dtype=torch.uint8, device="cuda")]
    B.twa_batch_solver(0).twa_capture_next(*caught)
    B.twa_batch_iterate(7)       # captured, then six in the groups
    B.twa_batch_config(256, 2)
    B.twa_batch_iterate(3)       # the persistent kernel takes the state over
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(37)
    for i, inst in enumerate(insts):
        S = Solver.from_instance(inst)
        _plain(S, 60)
        _same(B.twa_batch_solver(i), S)
        S.close()
    B.close()


@pytest.mark.parametrize("flags", [F_NONE, F_MAXVEL, F_MINVEL])
def test_batch_groups_modes(flags):
    from paper_1311_4527_amd.twa import Batch, Solver
    insts = [_box(30, 5, 3), _swap(26, 5, dim=3), _box(9, 1, 2)]
    for inst in insts:
        step = np.linalg.norm(inst.xT - inst.x0, axis=1) / inst.eta
        if flags & (F_MAXVEL | F_MINVEL):
            inst.C = np.repeat((step * (1.3 if flags & F_MAXVEL else 0.8))[:, None], inst.eta, axis=1)
    B = Batch(insts, flags=flags)
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(40)
    for i, inst in enumerate(insts):
        S = Solver.from_instance(inst, flags=flags)
        _plain(S, 40)
        _same(B.twa_batch_solver(i), S)
        S.close()
    B.close()


def test_batch_groups_more_members_than_resident():
    """400 members take the card's workgroups in turn; members that come late
    run with whoever is there."""
    from paper_1311_4527_amd.twa import Batch, Solver
    insts = I.conf_batch(400, base_seed=40, p_range=(30, 60))
    B = Batch(insts)
    B.twa_batch_config(0, 1)
    B.twa_batch_iterate(20)
    for i in range(0, len(insts), 37):
        S = Solver.from_instance(insts[i])
        _plain(S, 20)
        _same(B.twa_batch_solver(i), S)
        S.close()
    B.close()


def test_two_batches_on_two_streams():
    import torch
    from paper_1311_4527_amd.twa import Batch
    insts = I.conf_batch(40, base_seed=60, p_range=(30, 90))
    R = Batch(insts)
    R.twa_batch_config(256, 40)
    R.twa_batch_iterate(50)
    want = [R.twa_batch_get_trajectories(i) for i in range(len(insts))]
    torch.cuda.synchronize()
    S = [Batch(insts, stream=torch.cuda.Stream()) for _ in range(2)]
    for b in S:
        b.twa_batch_config(0, 1)
    torch.cuda.synchronize()
    for _ in range(5):
        for b in S:
            b.twa_batch_iterate(10)
    torch.cuda.synchronize()
    for b in S:
        for i, w in enumerate(want):
            assert torch.equal(b.twa_batch_get_trajectories(i), w)
        b.close()
    R.close()
