"""The 4-state root reduction with 5 to 8 rate categories, where a block serves 32 patterns and not
64: the likelihood, the site vector and the gradient against the oracle, below and above the number
of blocks at which the blocks walk several pattern groups (256 x 32)."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_GRAD, TOL_LOGL, assert_grad, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n_categories, n_patterns", [(5, 33), (8, 129), (8, 8193), (7, 16417)])
def test_root_blocks(n_categories, n_patterns, precision):
    prob = W.random_problem(np.random.default_rng(n_patterns), 5, 4, n_patterns, n_categories=n_categories,
                            n_intervals=2, reversible=True)
    with from_problem(prob, precision, grad_branch=True) as lik:
        logL, site, db, _ = lik.evaluate(branch=True, site=True)
    assert rel(logL, O.log_likelihood(prob)) <= TOL_LOGL[precision]
    assert rel(float(np.dot(site, prob.weights)), logL) <= 1e-12
    assert_grad(db, O.gradient(prob)[0], TOL_GRAD[precision], "dlogL/dl")
