"""Where long epoch chains are cut when the caller sets no line: chains of 7 to 17 segments around the
FP64 line (8 for a small tree) and the FP32 one (16), with dP/dl, dlogL/dQ and the suffix products that
start the parts, against the oracle; FP64 instances against uncut chains too."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_GRAD, TOL_LOGL, assert_grad, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("K, n_intervals", [(14, 8), (16, 9), (31, 12), (48, 16), (50, 17)])
def test_default_line(K, n_intervals, precision):
    prob = W.random_problem(np.random.default_rng(90 + n_intervals), 4, K, 3, n_categories=2,
                            n_intervals=n_intervals, reversible=False)
    with from_problem(prob, precision, grad_branch=True, grad_Q=True) as lik:
        logL, _, db, dq = lik.evaluate(branch=True, Q=True)
        lik.set_option("chain_split", 0)
        whole = lik.evaluate(branch=True, Q=True)
    assert rel(logL, O.log_likelihood(prob)) <= TOL_LOGL[precision]
    ref_b, ref_q = O.gradient(prob)
    assert_grad(db, ref_b, TOL_GRAD[precision], "dlogL/dl")
    assert_grad(dq, ref_q, TOL_GRAD[precision], "dlogL/dQ")
    if precision == "fp64":
        assert rel(logL, whole[0]) <= TOL_LOGL[precision]
        assert_grad(db, whole[2], TOL_GRAD[precision], "dlogL/dl, uncut")
        assert_grad(dq, whole[3], TOL_GRAD[precision], "dlogL/dQ, uncut")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n_tips", [1020, 1030])  # 4,078 and 4,118 stripes: either side of the P stage's two forms
def test_derivative_apart(n_tips, precision):
    prob = W.random_problem(np.random.default_rng(n_tips), n_tips, 17, 2, n_categories=1, n_intervals=3,
                            reversible=False)
    with from_problem(prob, precision, grad_branch=True) as lik:
        logL, _, db, _ = lik.evaluate(branch=True)
    assert rel(logL, O.log_likelihood(prob)) <= TOL_LOGL[precision]
    assert_grad(db, O.gradient(prob)[0], TOL_GRAD[precision], "dlogL/dl")
