"""The reverse step's node sums (four lanes per node), its radius sums per
interval, and the capture that records queued factors only, where they can go
wrong: waves with a few records and with many blocks of them, collision and
wall records in one wave, a single interval, the dense form.  Against the FP64
reference adjoint, with its bars (tests/test_gpu_adjoint.py); few iterations,
so that both sides take the same decisions."""
import numpy as np
import pytest

from paper_1311_4527_amd import instances as I
from tests.test_gpu_adjoint import _compare, _ref_grad

pytestmark = pytest.mark.gpu

F_DENSE = 1
CASES = {
    "pair": lambda: I.circle_swap(2, 0.3, 3, seed=3, alpha=0.1, C=0.1),                     # one or two records
    "one_interval": lambda: I.circle_swap(17, 0.1, 1, seed=4, alpha=0.1, C=0.05),
    "crowded": lambda: I.circle_swap(70, 0.02, 5, seed=5, alpha=0.1, C=0.01),               # thousands, a ragged tail
    "walls_between": lambda: I.random_box(40, 0.05, 3, n_walls=7, sigma=1e-2, seed=6, alpha=0.1, C=0.01),
}


@pytest.mark.parametrize("flags", [0, F_DENSE])
@pytest.mark.parametrize("case", sorted(CASES))
def test_sums_match_reference(case, flags):
    import torch
    from paper_1311_4527_amd.twa import Solver, TWA_F_TAPE
    inst = CASES[case]()
    K = 5
    v = np.random.default_rng(21).normal(size=inst.z0.shape)
    S = Solver.from_instance(inst, flags=flags | TWA_F_TAPE)
    S.twa_iterate(K)
    assert S.twa_get_stats()["active_coll"] > 0
    got = [t.cpu().numpy().astype(np.float64) for t in S.twa_backward(torch.from_numpy(v.astype(np.float32)))]
    S.close()
    _compare(got, _ref_grad(inst, K, v)[0])
