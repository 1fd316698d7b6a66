"""4-state post-order of a list of nodes in one launch (short paths and small trees) against the
launch per level: the same bits, whichever of the two a call takes, and the oracle."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_LOGL, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("taxa,patterns,categories", [
    (2, 1, 1), (3, 17, 4), (9, 63, 3), (24, 16, 8), (60, 65, 2), (150, 33, 4)])
def test_list_matches_oracle(taxa, patterns, categories, precision):
    prob = W.random_problem(np.random.default_rng(100 * taxa + patterns), taxa, 4, patterns,
                            n_categories=categories, n_intervals=2, missing_frac=0.1, ambiguous_frac=0.1)
    with from_problem(prob, precision, options={"tree_walk": 0}) as lik:
        logL, site, _, _ = lik.evaluate(site=True)
    want = O.log_likelihood(prob)
    assert rel(logL, want) <= TOL_LOGL[precision]
    assert np.isfinite(site).all()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_paths_give_the_bits_of_a_full_evaluation(precision):
    """300 taxa: a full evaluation runs per level, a changed branch's path as a list."""
    rng = np.random.default_rng(5)
    prob = W.random_problem(rng, 300, 4, 1001, n_categories=4, n_intervals=3, missing_frac=0.05)
    prob.branch_rate = prob.branch_rate.copy()
    lik = from_problem(prob, precision, options={"tree_walk": 0})
    lik.evaluate()
    for changed in ([3], [3, 77], [400, 401, 402], list(range(0, 500, 25)), list(range(0, 598, 2))):
        for v in changed:
            prob.branch_rate[v] *= float(rng.uniform(0.6, 1.6))
        lik.set_branch_rates(changed, prob.branch_rate[changed])  # more than 64: by upload
        got = lik.evaluate(site=True)
        with from_problem(prob, precision, options={"tree_walk": 0}) as fresh:
            want = fresh.evaluate(site=True)
        assert got[0] == want[0] and np.array_equal(got[1], want[1]), changed
    # a node listed twice keeps its last rate, the root's entry is ignored
    prob.branch_rate[10] = 1.7
    lik.set_branch_rates([10, lik.n_nodes - 1, 10], [0.3, 5.0, 1.7])
    got = lik.evaluate()[0]
    with from_problem(prob, precision, options={"tree_walk": 0}) as fresh:
        assert got == fresh.evaluate()[0]
    lik.close()
