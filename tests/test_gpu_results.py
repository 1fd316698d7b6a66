"""The root reduction in one launch (the last block adds up the others' shares) and the results
through the pinned buffer or, above 65,536 values, a direct copy: pattern counts around the block
sizes of each kernel family, against the oracle and against the weighted sum of the site values."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_GRAD, TOL_LOGL, assert_grad, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("states,categories,patterns,taxa", [
    (4, 4, 1, 5), (4, 3, 63, 5), (4, 4, 65, 5), (4, 1, 257, 5), (4, 2, 65537, 4),   # 4-state root
    (20, 1, 1, 5), (20, 2, 64, 5), (20, 3, 65, 5), (61, 1, 63, 4), (61, 2, 129, 4),  # matrix-core root
    (7, 1, 1, 6), (7, 2, 256, 5), (40, 1, 257, 4)])                                   # generic root
def test_root_and_delivery(states, categories, patterns, taxa, precision):
    prob = W.random_problem(np.random.default_rng(1000 * states + patterns), taxa, states, patterns,
                            n_categories=categories, n_intervals=2)
    with from_problem(prob, precision, grad_branch=True, grad_Q=True) as lik:
        first = lik.evaluate(branch=True, Q=True, site=True)
        for _ in range(3):  # the arrival counter is back at zero after each launch
            again = lik.evaluate(branch=True, Q=True, site=True)
            assert again[0] == first[0]
            for a, b in zip(again[1:], first[1:]):
                assert np.array_equal(a, b)
        separate = lik.log_likelihood(site=True)
        assert separate[0] == first[0] and np.array_equal(separate[1], first[1])
    logL, site, db, dq = first
    # FP64 sums of the same site values in another order
    assert abs(logL - float(np.dot(prob.weights, site))) <= 1e-13 * np.abs(prob.weights * site).sum()
    assert rel(logL, O.log_likelihood(prob)) <= TOL_LOGL[precision]
    ref_b, ref_q = O.gradient(prob)
    assert_grad(db, ref_b, TOL_GRAD[precision], "dlogL/dl")
    assert_grad(dq, ref_q, TOL_GRAD[precision], "dlogL/dQ")
