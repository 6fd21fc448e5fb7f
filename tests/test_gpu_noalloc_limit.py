"""twa_backward_noalloc where its scratch is nearly full: a run that fits with one
radius sum per agent but not with one per node (408 agents, 16 intervals, 4
iterations: 6 records left with sums per node, 1312 with sums per agent, and a
crowd of a few dozen active factors) is still taken."""
import pytest

from paper_1311_4527_amd import instances as I
from tests.test_zz_no_alloc import _check

pytestmark = pytest.mark.gpu


def test_noalloc_with_radius_sums_per_agent():
    inst = I.random_box(408, 0.0003, 16, sigma=1e-3, seed=5, alpha=0.1, C=1.0 / (408 * 16))
    _check(inst, 4, 0)
