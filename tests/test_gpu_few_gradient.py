"""dlogL/dP of the few-pattern kernels over several tiles of patterns (33 to 48 states hold four in a
tile) is added up in FP64 across tiles, as the general kernels' partial sums are: one FP32 instance
against the same patterns spread over an alignment of more than 16, whose extra patterns have weight
zero and which therefore takes the general kernels. Within a tile both add the same FP32 terms in the
same order, so the gradients agree to FP64 rounding of the sums."""
import dataclasses

import numpy as np
import pytest

from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import from_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K, n_patterns", [(40, 4), (40, 5), (48, 12), (33, 16), (14, 16)])
def test_tiles_add_up_in_fp64(K, n_patterns):
    prob = W.random_problem(np.random.default_rng(K + n_patterns), 12, K, n_patterns, n_categories=1, n_intervals=3,
                            reversible=False)
    pad = np.repeat(prob.tips[:, :1], 32 - n_patterns, axis=1)
    wide = dataclasses.replace(prob, tips=np.ascontiguousarray(np.concatenate([prob.tips, pad], axis=1)),
                               weights=np.concatenate([prob.weights, np.zeros(32 - n_patterns)]))
    out = []
    for q in (prob, wide):
        with from_problem(q, "fp32", grad_branch=True) as lik:
            out.append(lik.evaluate(branch=True))
    assert abs(out[0][0] - out[1][0]) <= 1e-12 * abs(out[1][0])
    scale = np.abs(out[1][2]).max()
    assert np.abs(out[0][2] - out[1][2]).max() <= 64 * K * np.finfo(float).eps * scale
