"""The condition number of a reversible matrix's eigenvectors, taken from pi, against the SVD's."""
import numpy as np
import pytest

from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.eigen import eigensystem


@pytest.mark.parametrize("K", [2, 4, 20, 61, 64])
def test_reversible_cond(K):
    prob = W.random_problem(np.random.default_rng(K), 4, K, 5, n_categories=1, n_intervals=3, reversible=True)
    for Q, pi in zip(prob.Q, prob.pi_process):
        pi = np.asarray(pi) * np.logspace(0, -6, K)  # a wide pi; the symmetric part is all that is used
        e = eigensystem(Q, pi / pi.sum())
        want = np.linalg.cond(e.V)
        # both extreme singular values carry an error of K eps times the largest
        assert abs(e.cond - want) <= 4 * K * np.finfo(float).eps * want * want
