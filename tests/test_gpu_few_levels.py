"""Post-order levels of the few-pattern kernels with one to many items per block (full, and with a
remainder), and the line on the matrices of a run's level, against the per-level kernels that an HBM budget
too large to matter selects, and without a gradient."""
import numpy as np
import pytest

from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_GRAD, assert_grad, rel

pytestmark = pytest.mark.gpu

# the kernels form the same products in the same order; a compiler may contract them differently
TOL = {"fp64": 1e-12, "fp32": 1e-6}


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("states,taxa,patterns,categories", [
    (3, 700, 11, 2),   # widest levels above 2,048 items: two to a block, and a remainder
    (4, 1500, 16, 2),  # four-lane items, blocks of several nodes
    (14, 200, 5, 8), (20, 40, 9, 3), (40, 60, 1, 4),  # an item to a block, in a wavefront of its own
    (12, 90, 16, 1), (20, 64, 8, 1), (20, 64, 4, 1)])  # levels below and above the line of a run
def test_levels(states, taxa, patterns, categories, precision):
    prob = W.random_problem(np.random.default_rng(states * taxa), taxa, states, patterns, n_categories=categories,
                            n_intervals=2, missing_frac=0.1, ambiguous_frac=0.1)
    with from_problem(prob, precision, grad_branch=True, kernel="generic", hbm_budget_bytes=1 << 36) as lik:
        want = lik.evaluate(branch=True, site=True)
    for grad in (True, False):
        with from_problem(prob, precision, grad_branch=grad, kernel="generic") as lik:
            got = lik.evaluate(branch=grad, site=True)
        assert rel(got[0], want[0]) <= TOL[precision]
        assert np.max(np.abs(got[1] - want[1])) <= TOL[precision] * np.max(np.abs(want[1]))
        if grad:
            assert_grad(got[2], want[2], TOL_GRAD[precision], "dlogL/dl")


@pytest.mark.parametrize("room", [True, False])
def test_workspace(room):
    """The child vectors in a caller's memory, and per-level kernels in one without room for them."""
    import torch
    from paper_1309_3075_amd.likelihood import EpochLikelihood
    prob = W.random_problem(np.random.default_rng(8), 30, 7, 2, n_intervals=3, missing_frac=0.1)
    need = EpochLikelihood.workspace_bytes(30, 2, 7, 1, "fp64", grad_branch=True)
    vectors = 59 * 2 * 8 * 8
    ws = torch.zeros(need - (0 if room else -(-vectors // 256) * 256), dtype=torch.uint8, device="cuda")
    with from_problem(prob, "fp64", grad_branch=True, workspace=ws) as lik:
        got = lik.evaluate(branch=True, site=True)
    torch.cuda.synchronize()
    with from_problem(prob, "fp64", grad_branch=True) as lik:
        want = lik.evaluate(branch=True, site=True)
    assert rel(got[0], want[0]) <= TOL["fp64"]
    assert np.max(np.abs(got[1] - want[1])) <= TOL["fp64"] * np.max(np.abs(want[1]))
    assert_grad(got[2], want[2], TOL_GRAD["fp64"], "dlogL/dl")
