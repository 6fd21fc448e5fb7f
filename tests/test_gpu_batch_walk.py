"""The persistent batch walks the pairs of instances of 64 agents and more by row
chunks, or by several rows of a chunk column, by size and form: the same bits as
the plain launches at sizes of each kind and ragged ones, captures included."""
import pytest

from tests.test_gpu_group import _box, _plain, _same, _swap, F_ADMM, F_DENSE

pytestmark = pytest.mark.gpu

MEMBERS = {
    "chunks": lambda: [_box(64, 3, 0), _box(65, 6, 3), _swap(66, 5, dim=3), _swap(70, 4, dim=3), _box(80, 9, 1), _swap(88, 4)],
    "rows": lambda: [_box(127, 5, 2), _box(128, 4, 0), _swap(130, 5, dim=3), _box(200, 7, 1), _swap(194, 2)],
    "between": lambda: [_box(p, 5, 0) for p in (95, 96)] + [_box(97, 3, 0), _box(112, 3, 1), _swap(72, 3, dim=3)],
}


@pytest.mark.parametrize("flags", [0, F_DENSE, F_ADMM])
@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("members", sorted(MEMBERS))
def test_persistent_batch_equals_plain(members, block, flags):
    import torch
    from paper_1311_4527_amd.twa import Batch, Solver
    insts = MEMBERS[members]()
    B = Batch(insts, flags=flags)
    B.twa_batch_config(block, 3)
    B.twa_batch_iterate(9)
    # iteration 10 of a member, captured
    R = Solver.from_instance(insts[1], flags=flags)
    for _ in range(3):
        R.twa_iterate_timed(3)
    caught = []
    for s in (B.twa_batch_solver(1), R):
        caught.append((torch.empty((s.n_edges, s.dim), dtype=torch.float32, device="cuda"),
                       torch.empty((s.n_factors,), dtype=torch.uint8, device="cuda")))
        s.twa_capture_next(*caught[-1])
    B.twa_batch_iterate(1)
    R.twa_iterate(1)
    torch.cuda.synchronize()
    assert torch.equal(caught[0][0], caught[1][0]) and torch.equal(caught[0][1], caught[1][1])
    R.close()
    B.twa_batch_iterate(4)
    for i, inst in enumerate(insts):
        S = Solver.from_instance(inst, flags=flags)
        _plain(S, 14)
        _same(B.twa_batch_solver(i), S)
        S.close()
    B.close()
