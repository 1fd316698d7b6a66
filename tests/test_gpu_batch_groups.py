"""Batches whose FP32 tree-walk members share launches: sizes around the 16- to 64-pattern tiles,
every category count, members outside the groups, and gradients from the batch's host buffer."""
import numpy as np
import pytest

from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.likelihood import EpochBatchEvaluator, from_problem

pytestmark = pytest.mark.gpu


def _prob(seed, taxa, patterns, categories, states=4):
    return W.random_problem(np.random.default_rng(seed), taxa, states, patterns, n_categories=categories,
                            n_intervals=2, missing_frac=0.1, branch_rate_spread=0.2)


MEMBERS = [  # taxa, patterns, categories, precision, options, states
    (2, 1, 4, "fp32", {}, 4), (3, 15, 4, "fp32", {}, 4), (30, 17, 3, "fp32", {}, 4), (12, 1000, 4, "fp32", {}, 4),
    (5, 64, 1, "fp32", {}, 4), (40, 65, 1, "fp32", {}, 4), (9, 33, 2, "fp32", {}, 4), (8, 9, 8, "fp32", {}, 4),
    (17, 7, 8, "fp32", {}, 4), (20, 100, 4, "fp32", {"walk_tiles": 2}, 4), (6, 31, 4, "fp32", {"walk_tiles": 2}, 4),
    (20, 100, 4, "fp32", {"walk_blocks": 1}, 4), (11, 50, 4, "fp64", {}, 4), (11, 50, 4, "fp32", {"tree_walk": 0}, 4),
    (7, 20, 1, "fp32", {}, 7)]


def test_groups_give_single_evaluations():
    probs = [_prob(i, t, p, c, k) for i, (t, p, c, _, _, k) in enumerate(MEMBERS)]
    members = [from_problem(pr, prec, grad_branch=True, options=opt)
               for pr, (_, _, _, prec, opt, _) in zip(probs, MEMBERS)]
    batch = EpochBatchEvaluator(members)
    rng = np.random.default_rng(0)
    for step in range(4):
        if step:  # new branch rates of every member, some by launch and some by upload
            for pr, m in zip(probs, members):
                nodes = np.arange(m.n_nodes if step == 2 else min(5, m.n_nodes))
                pr.branch_rate = pr.branch_rate.copy()
                pr.branch_rate[nodes] *= np.exp(0.3 * rng.normal(size=len(nodes)))
                m.set_branch_rates(nodes, pr.branch_rate[nodes])
        logL = batch.evaluate(grad_branch=True)
        grads = [batch.gradients(i)[0] for i in range(len(members))]
        only = batch.evaluate(grad_branch=False)
        assert np.array_equal(only, logL)
        for i, (pr, (_, _, _, prec, opt, _)) in enumerate(zip(probs, MEMBERS)):
            with from_problem(pr, prec, grad_branch=True, options=opt) as single:
                want, _, db, _ = single.evaluate(branch=True)
            assert logL[i] == want, (step, i)
            assert np.array_equal(grads[i], db), (step, i)
    # a member evaluated on its own since: its new gradient, not the batch's
    batch.evaluate(grad_branch=True)
    before = batch.gradients(3)[0]
    members[3].set_branch_rates([0], [probs[3].branch_rate[0] * 2.0])
    db = members[3].evaluate(branch=True)[2]
    assert not np.array_equal(db, before)
    assert np.array_equal(batch.gradients(3)[0], db)
    batch.close()
    for m in members:
        m.close()
