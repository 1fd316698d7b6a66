"""4-state kernel options set between the steps of an evaluation: the tree walk turned on after the P stage
ran reads that stage's matrices, not what its own buffers held before."""
import numpy as np
import pytest

from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("earlier", [False, True])  # whether an evaluation of other rates left its matrices there
def test_walk_turned_on_between_steps(precision, earlier):
    prob = W.random_problem(np.random.default_rng(77), 21, 4, 150, n_categories=4, n_intervals=3, reversible=True)
    with from_problem(prob, precision, grad_branch=True, options={"tree_walk": 1}) as lik:
        want = lik.evaluate(branch=True)
    with from_problem(prob, precision, grad_branch=True, options={"tree_walk": 1 if earlier else 0}) as lik:
        if earlier:
            nodes = np.arange(prob.parent.shape[0] - 1)
            lik.set_branch_rates(nodes, 2.0 * prob.branch_rate[nodes])
            lik.evaluate(branch=True)
            lik.set_option("tree_walk", 0)
            lik.set_branch_rates(nodes, prob.branch_rate[nodes])
        lik.update_transition_matrices()
        lik.set_option("tree_walk", 1)
        lik.update_partials()
        assert lik.root_log_likelihood() == want[0]
        assert np.array_equal(lik.gradient()[0], want[2])
