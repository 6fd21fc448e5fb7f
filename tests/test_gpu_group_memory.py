"""The memory of groups of resident workgroups: taken where a group can run, and
no reason for a call to fail (the plain and phased launches need none)."""
import pytest

from paper_1311_4527_amd import instances as I
from tests.test_gpu_group import _plain, _same, _swap

pytestmark = pytest.mark.gpu


class _Nth:
    """torch's caching allocator behind callbacks; call number `fail` gets no
    memory."""

    def __init__(self, fail=None):
        import torch
        import paper_1311_4527_amd.twa as T
        self.calls = 0

        def alloc(n, dev, stream, ctx):
            self.calls += 1
            if self.calls == fail:
                return None
            return torch.cuda.caching_allocator_alloc(int(n), device=int(dev), stream=int(stream or 0))

        def free(p, n, dev, stream, ctx):
            torch.cuda.caching_allocator_delete(int(p))

        self.a, self.f = T._ALLOC_FN(alloc), T._FREE_FN(free)

    def __enter__(self):
        import paper_1311_4527_amd.twa as T
        assert T.load_library().twa_set_allocator(self.a, self.f, None) == 0
        return self

    def __exit__(self, *exc):
        import paper_1311_4527_amd.twa as T
        T.twa_set_allocator(True)


def test_solver_without_memory_for_its_group():
    """The group's buffer is the last one of a create: without it the solver
    runs the plain launches."""
    from paper_1311_4527_amd.twa import Solver
    inst = _swap(18, 4)
    with _Nth() as n:
        A = Solver.from_instance(inst)
    with _Nth(fail=n.calls) as m:  # noqa: F841 (kept until B is closed)
        B = Solver.from_instance(inst)
    _plain(A, 40)
    B.twa_iterate(40)
    _same(A, B)
    A.close(), B.close()


@pytest.mark.parametrize("without", [False, True])
def test_batch_takes_group_memory_when_block_0_is_asked_for(without):
    from paper_1311_4527_amd.twa import Batch, Solver
    insts = [_swap(18, 4), I.circle_swap(26, 0.05, 5, seed=3)]
    with _Nth() as n:
        B = Batch(insts)
        made = n.calls
        B.twa_batch_iterate(3)
        B.twa_batch_config(512, 2)
        assert n.calls == made
        B.close()
    with _Nth(fail=made + 1 if without else None) as n:
        B = Batch(insts)
        B.twa_batch_config(0, 1)
        assert n.calls == made + 1
        B.twa_batch_iterate(40)
        for i, inst in enumerate(insts):
            S = Solver.from_instance(inst)
            _plain(S, 40)
            _same(B.twa_batch_solver(i), S)
            S.close()
        B.close()
