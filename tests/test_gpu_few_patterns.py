"""Few-pattern kernels of the generic path (runs of narrow tree levels in one block, kept child
vectors) against the oracle: every lane count, pattern counts up to the last the kernels take, tree
shapes from balanced to a chain, restricted passes, and a pattern more than they take."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_GRAD, TOL_LOGL, assert_grad, rel

pytestmark = pytest.mark.gpu


def _chain(prob):
    """The same tips on a caterpillar: node N + k joins node N + k - 1 and tip k + 1."""
    N = prob.n_tips
    parent = np.full(2 * N - 1, -1, dtype=np.int32)
    height = np.zeros(2 * N - 1)
    parent[0] = N
    for k in range(N - 1):
        parent[k + 1] = N + k
        if k:
            parent[N + k - 1] = N + k
        height[N + k] = (k + 1.0) / (N - 1)
    prob.parent, prob.height = parent, height
    return prob


def _check(prob, precision, kernel="auto"):
    with from_problem(prob, precision, grad_branch=True, grad_Q=True, kernel=kernel) as lik:
        assert lik.kernel_path() == "generic"
        logL, _, db, dq = lik.evaluate(branch=True, Q=True)
        again = lik.evaluate(branch=True, Q=True)
        assert again[0] == logL and np.array_equal(again[2], db) and np.array_equal(again[3], dq)
    with from_problem(prob, precision, grad_branch=True, kernel=kernel) as lik:  # dlogL/dP not stored
        branch_only = lik.evaluate(branch=True)
    assert branch_only[0] == logL and np.array_equal(branch_only[2], db)
    ref_b, ref_q = O.gradient(prob)
    assert rel(logL, O.log_likelihood(prob)) <= TOL_LOGL[precision]
    assert_grad(db, ref_b, TOL_GRAD[precision], "dlogL/dl")
    assert_grad(dq, ref_q, TOL_GRAD[precision], "dlogL/dQ")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("states,taxa,patterns,categories,kernel", [
    (3, 2, 1, 1, "auto"), (4, 30, 3, 1, "generic"), (7, 90, 1, 1, "auto"), (8, 17, 16, 1, "auto"),
    (8, 17, 17, 1, "auto"), (9, 40, 2, 1, "auto"), (16, 25, 5, 3, "auto"), (20, 33, 4, 1, "generic"),
    (32, 12, 1, 1, "generic"), (33, 60, 1, 1, "auto"), (40, 30, 2, 2, "auto"), (48, 14, 3, 1, "auto"),
    (50, 20, 1, 1, "generic"), (64, 9, 2, 1, "generic")])
def test_few_patterns(states, taxa, patterns, categories, kernel, precision):
    prob = W.random_problem(np.random.default_rng(states * 100 + taxa), taxa, states, patterns,
                            n_categories=categories, n_intervals=3, missing_frac=0.1, ambiguous_frac=0.1,
                            branch_rate_spread=0.3)
    _check(prob, precision, kernel)


@pytest.mark.parametrize("states,taxa,patterns", [(7, 150, 1), (5, 70, 16), (40, 120, 2)])
def test_chain_of_levels(states, taxa, patterns):
    """More levels than one run's LDS holds."""
    prob = _chain(W.random_problem(np.random.default_rng(taxa), taxa, states, patterns, n_intervals=3))
    _check(prob, "fp64")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("states,patterns,categories", [(7, 1, 1), (40, 2, 1), (14, 3, 2)])
def test_restricted_passes_give_the_bits_of_a_full_one(states, patterns, categories, precision):
    rng = np.random.default_rng(states)
    prob = W.random_problem(rng, 120, states, patterns, n_categories=categories, n_intervals=2)
    prob.branch_rate = prob.branch_rate.copy()
    lik = from_problem(prob, precision, grad_branch=True)
    lik.evaluate()
    for changed in ([0], [5, 130], list(range(0, 238, 9))):
        prob.branch_rate[changed] *= np.exp(0.4 * rng.normal(size=len(changed)))
        lik.set_branch_rates(changed, prob.branch_rate[changed])
        logL, _, db, _ = lik.evaluate(branch=True)
        with from_problem(prob, precision, grad_branch=True) as fresh:
            want = fresh.evaluate(branch=True)
        assert logL == want[0] and np.array_equal(db, want[2]), changed
    lik.close()
