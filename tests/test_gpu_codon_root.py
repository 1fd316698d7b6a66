"""The matrix-core path's root reduction around the pattern count (4,096) where a sixteen-lane group
goes from one pattern to four, and under an HBM budget whose last pattern chunk lies on the other side
of it than the others."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_GRAD, TOL_LOGL, assert_grad, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_categories, n_patterns", [(1, 1), (8, 17), (1, 4096), (3, 4097), (5, 4111)])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_blocks(n_categories, n_patterns, precision):
    prob = W.random_problem(np.random.default_rng(n_patterns), 4, 20, n_patterns, n_categories=n_categories,
                            n_intervals=2, reversible=True)
    with from_problem(prob, precision, grad_branch=True) as lik:
        logL, site, db, _ = lik.evaluate(branch=True, site=True)
    assert rel(logL, O.log_likelihood(prob)) <= TOL_LOGL[precision]
    assert rel(float(np.dot(site, prob.weights)), logL) <= 1e-12
    assert_grad(db, O.gradient(prob)[0], TOL_GRAD[precision], "dlogL/dl")


@pytest.mark.parametrize("last", [64, 4096])
def test_last_chunk(last):
    first = 4160
    prob = W.random_problem(np.random.default_rng(last), 4, 20, first + last, n_categories=1, n_intervals=2,
                            reversible=True)
    with from_problem(prob, "fp64") as lik:
        whole = lik.evaluate(site=True)
    budget = None
    for b in range(1 << 20, 1 << 24, 1 << 16):  # the smallest budget that holds `first` patterns at once
        try:
            with from_problem(prob, "fp64", hbm_budget_bytes=b) as lik:
                got = lik.evaluate(site=True)
        except Exception:
            continue
        budget = b
        assert rel(got[0], whole[0]) <= 1e-12 and np.allclose(got[1], whole[1], rtol=1e-12, atol=0), b
    assert budget
    assert rel(whole[0], O.log_likelihood(prob)) <= TOL_LOGL["fp64"]
