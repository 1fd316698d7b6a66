"""The matrix-core root reduction under an HBM budget whose last pattern chunk lies on the other side of
4,096 patterns (one pattern per sixteen-lane group, or four) than the others: its blocks may be more than
a full chunk's, or fewer."""
import numpy as np
import pytest

from oracle import epoch_oracle as O
from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem
from tolerances import TOL_LOGL, rel

pytestmark = pytest.mark.gpu

CHUNK = 4160  # patterns of a full chunk: four to a group, 65 blocks


@pytest.mark.parametrize("last", [1, 64, 1041, 4095, 4096, 4097])  # 1 to 256 blocks of one pattern each, and 65
def test_last_chunk(last):
    prob = W.random_problem(np.random.default_rng(last), 4, 20, CHUNK + last, n_categories=1, n_intervals=2,
                            reversible=True, missing_frac=0.05)
    # bytes of a pattern without a gradient: the partials (32 padded states) and the scale exponents of 3 nodes
    with from_problem(prob, "fp32", hbm_budget_bytes=CHUNK * 3 * (32 * 4 + 4)) as lik:
        assert lik.kernel_path() == "matrix_core64"
        first = lik.evaluate(site=True)
        again = lik.evaluate(site=True)  # the counter of arrived blocks is back at zero
    with from_problem(prob, "fp32") as lik:
        whole = lik.evaluate(site=True)
    assert again[0] == first[0] and np.array_equal(again[1], first[1])
    # the same FP32 partials; the FP64 sums of sites differ in their order only
    assert np.array_equal(first[1], whole[1])
    assert rel(first[0], whole[0]) <= 1e-12
    assert rel(first[0], O.log_likelihood(prob)) <= TOL_LOGL["fp32"]
