"""Workloads that the time of this framework is measured on.

Each case is one call, or one short run of calls, as a sampler, an optimiser or a likelihood server makes
them through the package's public entry points: the whole evaluation (``EpochLikelihood.evaluate``) with or
without gradients, one-branch proposals of a Markov chain, the node-height and boundary gradient, one
``torch.autograd`` step over model parameters, and batches (``EpochBatchEvaluator``).  The listed cases are
the repository's own workloads (``workloads.py``, ``bench.py``), the two the method's paper times (522 taxa
with 7 locations under 13 epochs; 109 taxa, 516 codon columns, two epochs), and ragged ones between them.

Inputs come from the seed alone: a coalescent tree, rate matrices, and tip states simulated down the tree
under the change-point process, with per-branch rates and missing data where a case says so.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1309_3075_amd import workloads as W
from paper_1309_3075_amd.autograd import EpochLogLikelihood, EpochModel, gy94_q
from paper_1309_3075_amd.likelihood import EpochBatchEvaluator, from_problem

_BASE = {"kind": "evaluate", "model": "gtr", "states": 4, "taxa": 64, "patterns": 1000, "categories": 1, "epochs": 1,
         "processes": 1, "precision": "fp64", "want": "branch", "site": False, "missing": 0.0, "rate_spread": 0.0,
         "dated": False, "members": 1, "spread": 1.0, "proposals": 0}


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a short alignment's log-likelihood in double precision, what a sampler asks for after
        # a move that changes every branch; launches and latency
        _case("nuc_small_logl", model="hky", taxa=16, patterns=1000, categories=4, epochs=2, processes=2, want="logL",
              site=True),
        # the paper's phylogeography run: one trait column, 522 dated taxa, 7 locations, 13 epochs; a Hamiltonian
        # or optimisation step over branch rates, node heights and transition times
        _case("trait7_time", model="trait", states=7, taxa=522, patterns=1, epochs=13, processes=13, want="time",
              dated=True, rate_spread=0.3),
        # a larger trait study: 40 locations, 12 asymmetric processes cycling over 48 intervals, rate gradients
        _case("trait40_rates", model="trait", states=40, taxa=2000, patterns=1, epochs=48, processes=12,
              precision="fp32", want="branch+Q"),
        # the flagship: whole-genome nucleotide alignment, every branch-length gradient
        _case("nuc_large_grad", taxa=512, patterns=100000, categories=4, epochs=3, processes=3, precision="fp32"),
        # a mid-sized alignment in double precision (the binding's default), odd sizes, gaps, relaxed clock
        _case("nuc_mid_fp64", taxa=203, patterns=20011, categories=4, epochs=3, processes=3, missing=0.02,
              rate_spread=0.3),
        # a Markov chain's one-branch proposals, each answered with a log-likelihood and rejected
        _case("nuc_proposals", kind="proposals", taxa=512, patterns=20011, categories=4, epochs=3, processes=3,
              precision="fp32", want="logL", proposals=16),
        # many small genes at once in a likelihood server
        _case("nuc_batch64", kind="batch", model="hky", taxa=32, patterns=948, categories=4, epochs=2, processes=2,
              precision="fp32", members=64, spread=3.1623),
        # amino-acid-sized model with rate categories and gaps
        _case("aa20_gamma4", model="reversible", states=20, taxa=80, patterns=2003, categories=4, epochs=4, processes=4,
              precision="fp32", missing=0.02, site=True),
        # codon model, branch-length and rate-matrix gradients
        _case("codon_grad", model="codon", states=61, taxa=128, patterns=10000, epochs=4, processes=4,
              precision="fp32", want="branch+Q"),
        # codon model in double precision, ragged
        _case("codon_fp64", model="codon", states=61, taxa=67, patterns=3001, epochs=4, processes=4, rate_spread=0.3),
        # the paper's within-host codon data set (109 taxa, 516 columns, two epochs): one optimiser step over kappa,
        # omega of each epoch and the branch lengths through torch.autograd
        _case("codon_model_step", kind="step", model="codon", states=61, taxa=109, patterns=516, epochs=2, processes=2,
              want="branch+Q"),
        # many codon alignments of uneven size at once in a likelihood server (the largest)
        _case("codon_batch16", kind="batch", model="codon", states=61, taxa=128, patterns=4472, epochs=4, processes=4,
              precision="fp32", members=16, spread=4.4721),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["nuc", "nuc", "codon", "codon", "aa", "trait", "trait", "proposals", "step", "batch_nuc",
                       "batch_codon"])
    epochs = rng.randint(1, 5)
    c = {"epochs": epochs, "processes": epochs, "precision": rng.choice(["fp32", "fp64"]),
         "missing": rng.choice([0.0, 0.02]), "rate_spread": rng.choice([0.0, 0.3]), "site": rng.random() < 0.25}
    if what == "nuc":
        c.update(model=rng.choice(["hky", "gtr"]), taxa=_log_int(rng, 8, 512), patterns=_log_int(rng, 200, 100000),
                 categories=rng.choice([1, 2, 4, 4, 8]), want=rng.choice(["logL", "branch", "branch", "branch+Q"]))
        if c["categories"] == 8:
            c["patterns"] = min(c["patterns"], 40001)
    elif what == "codon":
        c.update(model="codon", states=61, taxa=_log_int(rng, 12, 200), patterns=_log_int(rng, 200, 8000),
                 want=rng.choice(["logL", "branch", "branch+Q"]))
        if rng.random() < 0.25:
            c.update(categories=4, patterns=min(c["patterns"], 2500))
    elif what == "aa":
        c.update(model="reversible", states=20, taxa=_log_int(rng, 12, 200), patterns=_log_int(rng, 200, 8000),
                 categories=rng.choice([1, 4]), want=rng.choice(["logL", "branch", "branch+Q"]))
    elif what == "trait":
        k = rng.choice([3, 5, 7, 9, 14, 15, 20, 31, 40, 47, 56])
        m = _log_int(rng, 1, 48)
        c.update(model="trait", states=k, taxa=_log_int(rng, 50, 2000), patterns=rng.choice([1, 1, 1, 2, 5]), epochs=m,
                 processes=min(m, 12), want=rng.choice(["logL", "branch", "branch+Q", "time"]), missing=0.0,
                 dated=rng.random() < 0.5)
    elif what == "proposals":
        if rng.random() < 0.5:
            c.update(kind="proposals", taxa=_log_int(rng, 64, 512), patterns=_log_int(rng, 1000, 40000), categories=4,
                     want="logL", proposals=16, site=False)
        else:
            c.update(kind="proposals", model="codon", states=61, taxa=_log_int(rng, 32, 128),
                     patterns=_log_int(rng, 500, 6000), want="logL", proposals=16, site=False)
    elif what == "step":
        c.update(kind="step", model="codon", states=61, taxa=_log_int(rng, 16, 128), patterns=_log_int(rng, 200, 4000),
                 want="branch+Q", missing=0.0, rate_spread=0.0, site=False)
    elif what == "batch_nuc":
        c.update(kind="batch", model="hky", taxa=_log_int(rng, 16, 64), patterns=_log_int(rng, 300, 3000),
                 categories=4, members=_log_int(rng, 8, 64), spread=rng.choice([1.5, 3.0]), site=False)
    else:
        c.update(kind="batch", model="codon", states=61, taxa=_log_int(rng, 32, 100), patterns=_log_int(rng, 300, 3000),
                 members=_log_int(rng, 4, 16), spread=rng.choice([1.5, 3.0]), precision="fp32", site=False)
    return _case(**c)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

_DEV = "cuda"


def _member_sizes(case, i):
    """Taxa and patterns of member i: spread geometrically about the case's sizes, the patterns in another order."""
    m, s = case["members"], case["spread"]
    if m == 1:
        return case["taxa"], case["patterns"]
    f = lambda k: s ** (2.0 * k / (m - 1) - 1.0)  # noqa: E731
    return max(4, round(case["taxa"] * f(i) ** 0.6)), max(8, round(case["patterns"] * f((i * 7 + 3) % m)))


def _rate_matrices(case, rng):
    k, s, model = case["states"], case["processes"], case["model"]
    if model == "hky":
        pi = rng.dirichlet(np.full(4, 5.0))
        return [W.hky(2.0 * 2.0 ** (j % 3), pi) for j in range(s)], [pi] * s, pi, {}
    if model == "gtr":
        pis = [rng.dirichlet(np.full(4, 4.0)) for _ in range(s)]
        return [W.gtr(rng.dirichlet(np.full(6, 3.0)), p) for p in pis], pis, pis[-1], {}
    if model == "codon":
        pic = W.f3x4_frequencies(rng.dirichlet(np.full(4, 10.0), size=3))
        kappa, omega = 3.0, [(0.2, 1.0, 2.5, 0.5)[j % 4] * math.exp(0.1 * rng.normal()) for j in range(s)]
        mats = [gy94_q(torch.tensor(kappa, dtype=torch.float64), torch.tensor(w, dtype=torch.float64),
                       torch.tensor(pic)).numpy() for w in omega]
        return mats, [pic] * s, pic, {"kappa": kappa, "omega": omega, "pi": pic}
    if model == "reversible":
        mats, pis = [], []
        for _ in range(s):
            pi = rng.dirichlet(np.full(k, 5.0))
            r = rng.exponential(size=(k, k))
            q = (r + r.T) * pi[None, :]
            np.fill_diagonal(q, 0.0)
            np.fill_diagonal(q, -q.sum(1))
            mats.append(q / -(pi * np.diag(q)).sum())
            pis.append(pi)
        return mats, pis, pis[-1], {}
    # asymmetric location-exchange rates, sparse where there are many locations
    mats = [W.sparse_asymmetric(k, 0.2 if k >= 30 else 1.0, rng) for _ in range(s)]
    return mats, [None] * s, np.full(k, 1.0 / k), {}


def _segments(parent, height, bounds):
    """Stretches of every branch, parent side first: (child node, position in its branch, interval, and where the
    stretch's top and bottom heights stand in the list of node heights followed by boundaries)."""
    n = parent.shape[0]
    b = np.concatenate([[-np.inf], bounds, [np.inf]])
    rows = []
    for v in range(n):
        u = parent[v]
        if u < 0:
            continue
        k = int(np.searchsorted(bounds, height[u], side="left"))
        top, pos = u, 0
        while True:
            if b[k] > height[v]:
                rows.append((v, pos, k, top, n + k - 1))
                top, k, pos = n + k - 1, k - 1, pos + 1
            else:
                rows.append((v, pos, k, top, v))
                break
    return np.array(rows, dtype=np.int64)


def _transition(parent, heights, rates, bounds, phi, mats, cat_rates, segs, scale=None):
    """P[branch][category] by plain torch in 64 bits (heights, bounds, rates, mats: tensors)."""
    dev, k = mats.device, mats.shape[-1]
    s = torch.as_tensor(segs, device=dev)
    at = torch.cat([heights, bounds])
    tau = (at[s[:, 3]] - at[s[:, 4]]) * rates[s[:, 0]]
    if scale is not None:
        tau = tau * scale[s[:, 0]]
    arg = mats[phi[s[:, 2]]][:, None] * (tau[:, None] * cat_rates[None, :])[:, :, None, None]
    f = torch.linalg.matrix_exp(arg)
    n, c = parent.shape[0], cat_rates.shape[0]
    p = torch.eye(k, dtype=torch.float64, device=dev).expand(n, c, k, k)
    for j in range(int(segs[:, 1].max()) + 1):
        m = s[:, 1] == j
        v = s[m, 0]
        p = p.index_copy(0, v, torch.matmul(p[v], f[m]))
    return p


def _problem(case, seed, member=0):
    taxa, patterns = _member_sizes(case, member)
    rng = np.random.default_rng([int(seed), int(member), case["states"], taxa, patterns])
    mats, pis, pi_root, extra = _rate_matrices(case, rng)
    m, k = case["epochs"], case["states"]
    bounds = np.arange(1, m) / m
    phi = (np.arange(m) % case["processes"]).astype(np.int32)
    cat_rates, cat_weights = W.discrete_gamma(0.5, case["categories"])
    tip_h = rng.uniform(0.0, 0.5, size=taxa) if case["dated"] else None
    parent, height = W.coalescent_tree(taxa, rng, 1.0, tip_h)
    rate = np.exp(case["rate_spread"] * rng.normal(size=parent.shape[0]))
    # tip states: each site walks down the tree under the branch's transition matrix and its own category
    gen = torch.Generator(device=_DEV).manual_seed(int(rng.integers(1 << 62)))
    t = lambda x: torch.tensor(np.asarray(x), device=_DEV)  # noqa: E731
    cum = _transition(parent, t(height), t(rate), t(bounds), t(phi).long(), t(np.stack(mats)), t(cat_rates),
                      _segments(parent, height, bounds)).clamp_min(0).cumsum(-1)
    n = parent.shape[0]
    cat = torch.randint(0, len(cat_rates), (patterns,), generator=gen, device=_DEV)
    start = torch.rand(patterns, generator=gen, device=_DEV, dtype=torch.float64)
    cum_root = t(pi_root).cumsum(0)
    state = torch.empty((n, patterns), dtype=torch.long, device=_DEV)
    state[n - 1] = (cum_root[None, :] < start[:, None] * cum_root[-1]).sum(1).clamp_max(k - 1)
    for v in range(n - 2, -1, -1):
        row = cum[v][cat, state[int(parent[v])]]
        u = torch.rand(patterns, generator=gen, device=_DEV, dtype=torch.float64)
        state[v] = (row < (u * row[:, -1])[:, None]).sum(1).clamp_max(k - 1)
    tips = state[:taxa]
    if case["missing"] > 0:
        tips = torch.where(torch.rand(tips.shape, generator=gen, device=_DEV) < case["missing"], k, tips)
    weights = rng.integers(1, 6, size=patterns).astype(np.float64) if patterns > 8 else np.ones(patterns)
    prob = W.Problem(name="case", parent=parent, height=height, branch_rate=rate, boundaries=bounds,
                     interval_process=phi, Q=mats, pi_process=pis, pi_root=pi_root, cat_rates=cat_rates,
                     cat_weights=cat_weights, tips=tips.to(torch.int32).cpu().numpy(), weights=weights, seed=int(seed))
    return prob, extra, rng


def _proposal_list(case, prob, rng):
    nodes = rng.choice(prob.parent.shape[0] - 1, size=case["proposals"], replace=False)
    return [(int(v), float(prob.branch_rate[v]), float(prob.branch_rate[v] * math.exp(0.4 * rng.normal())))
            for v in nodes]


def prepare(case, seed):
    want = case["want"]
    flags = {"grad_branch": want != "logL", "grad_Q": want == "branch+Q", "grad_time": want == "time"}
    if case["kind"] == "batch":
        # a server keeps its instances and the batch, which captures its launches on the first evaluation
        members = [from_problem(_problem(case, seed, i)[0], case["precision"], **flags) for i in range(case["members"])]
        batch = EpochBatchEvaluator(members)
        batch.evaluate(grad_branch=flags["grad_branch"], grad_Q=flags["grad_Q"])
        return {"case": case, "members": members, "batch": batch}
    prob, extra, rng = _problem(case, seed)
    if case["kind"] == "step":
        model = EpochModel(prob, precision=case["precision"], reversible_pi=[extra["pi"]] * prob.n_processes)
        return {"case": case, "model": model, "pi": torch.tensor(extra["pi"]),
                "kappa": torch.tensor(extra["kappa"], dtype=torch.float64, requires_grad=True),
                "omega": torch.tensor(extra["omega"], dtype=torch.float64, requires_grad=True),
                "lengths": model.branch_lengths().requires_grad_(True)}
    lik = from_problem(prob, case["precision"], **flags)
    state = {"case": case, "lik": lik}
    if case["kind"] == "proposals":
        state["proposals"] = _proposal_list(case, prob, rng)
        lik.evaluate()  # the chain's current state
    return state


def run(state):
    case = state["case"]
    want = case["want"]
    if case["kind"] == "batch":
        batch = state["batch"]
        logl = batch.evaluate(grad_branch=want != "logL", grad_Q=want == "branch+Q")
        grads = [batch.gradients(i, branch=True, Q=want == "branch+Q") for i in range(case["members"])] \
            if want != "logL" else []
        return {"logL": logl, "d_branch": np.concatenate([g[0] for g in grads]) if grads else None}
    if case["kind"] == "step":
        Qs = [gy94_q(state["kappa"], w, state["pi"]) for w in state["omega"]]
        logl = EpochLogLikelihood.apply(state["model"], state["lengths"], *Qs)
        g = torch.autograd.grad(logl, [state["kappa"], state["omega"], state["lengths"]])
        return {"logL": logl.detach(), "d_kappa": g[0], "d_omega": g[1], "d_branch": g[2]}
    lik = state["lik"]
    if case["kind"] == "proposals":
        out = np.empty(len(state["proposals"]))
        for i, (v, old, new) in enumerate(state["proposals"]):
            lik.set_branch_rates([v], [new])
            out[i] = lik.evaluate()[0]
            lik.set_branch_rates([v], [old])
        return {"logL": out}
    logl, site, db, dq = lik.evaluate(branch=want != "logL", Q=want == "branch+Q", site=case["site"])
    out = {"logL": logl, "site": site, "d_branch": db, "d_Q": dq}
    if want == "time":
        out["d_height"], out["d_boundary"] = lik.time_gradient()
    return out


# ---------------------------------------------------------------------------
# What one pass cannot do without
# ---------------------------------------------------------------------------


def _one_work(case, taxa, patterns):
    """Tip states (a byte each) and weights read, results written; the pruning, adjoint and epoch-product
    arithmetic.  A tip's vector is a column of its branch's matrix and costs no product."""
    k, c, m, p, n = case["states"], case["categories"], case["epochs"], patterns, 2 * taxa - 1
    segs = n - 1 + sum(taxa / (1.0 + taxa * j / m) for j in range(1, m))
    want = case["want"]
    per = 2.0 * k * k * p * c * (taxa - 2) + 2.0 * n * k * p * c
    flops = per * (1.0 if want == "logL" else 3.0) + segs * c * 4.0 * k ** 3 + (segs - n + 1) * c * 2.0 * k ** 3
    if want == "branch+Q":
        flops += segs * c * 6.0 * k ** 3
    if want == "time":
        flops += segs * c * 4.0 * k ** 3
    out = 8.0 * (1 + (n if want != "logL" else 0) + (case["processes"] * k * k if want == "branch+Q" else 0)
                 + (n + m - 1 if want == "time" else 0) + (p if case["site"] else 0))
    inp = float(taxa) * p + 8.0 * p + 8.0 * case["processes"] * (2 * k * k + k) + 16.0 * segs
    return inp + out, flops


def work(case):
    if case["kind"] == "proposals":
        # the changed branch and its ancestors' partials: two children each, about twice the mean depth
        k, p, c = case["states"], case["patterns"], case["categories"]
        depth = 2.0 * math.log2(case["taxa"])
        b = case["proposals"] * depth * p * (2.0 * c * k * (4 if case["precision"] == "fp32" else 8) + 2.0)
        return {"bytes": b, "flops": case["proposals"] * depth * p * c * 4.0 * k * k}
    parts = [_one_work(case, *_member_sizes(case, i)) for i in range(case["members"])]
    return {"bytes": sum(x[0] for x in parts), "flops": sum(x[1] for x in parts)}


# ---------------------------------------------------------------------------
# The same results by plain torch in 64 bits
# ---------------------------------------------------------------------------


def _log_sites(prob, p, lo, hi, dev):
    """log L of patterns lo..hi from transition matrices p [node][category], pruning with the scale kept apart."""
    k = prob.n_states
    n = prob.parent.shape[0]
    tips = torch.tensor(prob.tips[:, lo:hi].astype(np.int64), device=dev)
    eye = torch.cat([torch.eye(k, dtype=torch.float64, device=dev), torch.ones(1, k, dtype=torch.float64, device=dev)])
    kids = [[] for _ in range(n)]
    for v in range(n - 1):
        kids[prob.parent[v]].append(v)
    vec, log_scale = {}, torch.zeros(hi - lo, dtype=torch.float64, device=dev)
    for u in range(prob.n_tips, n):
        x = None
        for v in kids[u]:
            # [category][pattern][state]
            lv = torch.matmul(eye, p[v].transpose(-1, -2))[:, tips[v]] if v < prob.n_tips else \
                torch.matmul(vec.pop(v), p[v].transpose(-1, -2))
            x = lv if x is None else x * lv
        top = x.detach().amax(dim=(0, 2))
        vec[u] = x / top[None, :, None]
        log_scale = log_scale + torch.log(top)
    root = (vec[n - 1] * torch.tensor(prob.pi_root, device=dev)).sum(-1)
    return torch.log((root * torch.tensor(prob.cat_weights, device=dev)[:, None]).sum(0)) + log_scale


def _exact_one(prob, want, mats=None, scale_grad=False):
    """logL, per-pattern log L and the gradients asked for; mats: the rate matrices as a tensor with its own graph."""
    dev = _DEV
    t = lambda x: torch.tensor(np.asarray(x), device=dev)  # noqa: E731
    grad = want != "logL"
    heights, bounds, rates = t(prob.height), t(prob.boundaries).double(), t(prob.branch_rate)
    q = t(np.stack(prob.Q)) if mats is None else mats
    scale = torch.ones_like(rates)
    if grad:
        scale.requires_grad_(True)
        if want == "branch+Q" and mats is None:
            q.requires_grad_(True)
        if want == "time":
            heights.requires_grad_(True)
            bounds.requires_grad_(True)
    p = _transition(prob.parent, heights, rates, bounds, t(prob.interval_process).long(), q, t(prob.cat_rates),
                    _segments(prob.parent, prob.height, prob.boundaries), scale)
    leaf = p.detach().requires_grad_(grad)
    w = t(prob.weights)
    per = prob.n_tips * len(prob.cat_rates) * prob.n_states * 8 * 12
    step = max(1, int(8e9 // per))
    sites, total = [], 0.0
    for lo in range(0, prob.n_patterns, step):
        hi = min(prob.n_patterns, lo + step)
        s = _log_sites(prob, leaf, lo, hi, dev)
        part = (w[lo:hi] * s).sum()
        if grad:
            part.backward()
        sites.append(s.detach())
        total += float(part.detach())
    out = {"logL": total, "site": torch.cat(sites).cpu().numpy()}
    if grad:
        asked = [scale] + ([q] if want == "branch+Q" else []) + ([heights, bounds] if want == "time" else [])
        g = torch.autograd.grad(p, asked, leaf.grad, allow_unused=True)
        tau = np.zeros(prob.parent.shape[0])
        inner = prob.parent >= 0
        tau[inner] = (prob.height[prob.parent[inner]] - prob.height[inner]) * prob.branch_rate[inner]
        db = np.zeros_like(tau)
        db[tau > 0] = g[0].cpu().numpy()[tau > 0] / tau[tau > 0]
        out["d_branch"] = db
        if want == "branch+Q":
            out["d_Q"] = g[1]
        if want == "time":
            out["d_height"] = g[1].cpu().numpy()
            out["d_boundary"] = g[2].cpu().numpy() if g[2] is not None else np.zeros(len(prob.boundaries))
    return out


def _codon_masks():
    """Sense-codon pairs one nucleotide apart, and which are transitions / change the amino acid (universal code)."""
    code = "FFLLSSSSYY**CC*WLLLLPPPPHHQQRRRRIIIMTTTTNNKKSSRRVVVVAAAADDEEGGGG"
    at = {"A": 2, "C": 1, "G": 3, "T": 0}
    codons = [(a, b, c) for a in "ACGT" for b in "ACGT" for c in "ACGT"]
    aa = {x: code[16 * at[x[0]] + 4 * at[x[1]] + at[x[2]]] for x in codons}
    codons = [x for x in codons if aa[x] != "*"]
    k = len(codons)
    single, ts, ns = (np.zeros((k, k)) for _ in range(3))
    for i, x in enumerate(codons):
        for j, y in enumerate(codons):
            d = [(a, b) for a, b in zip(x, y) if a != b]
            if len(d) == 1:
                single[i, j] = 1.0
                ts[i, j] = set(d[0]) in ({"A", "G"}, {"C", "T"})
                ns[i, j] = aa[x] != aa[y]
    return [torch.tensor(m, device=_DEV) for m in (single, ts, ns)]


def exact(case, seed):
    want = case["want"]
    if case["kind"] == "batch":
        if _one_work(case, case["taxa"], case["patterns"])[1] * case["members"] > 2e12:
            return None
        got = [_exact_one(_problem(case, seed, i)[0], want) for i in range(case["members"])]
        return {"logL": np.array([g["logL"] for g in got]),
                "d_branch": np.concatenate([g["d_branch"] for g in got]) if want != "logL" else None}
    prob, extra, rng = _problem(case, seed)
    if case["kind"] == "step":
        t = lambda x: torch.tensor(np.asarray(x), device=_DEV, dtype=torch.float64).requires_grad_(True)  # noqa: E731
        kappa, omega, pi = t(extra["kappa"]), t(extra["omega"]), torch.tensor(extra["pi"], device=_DEV)
        single, ts, ns = _codon_masks()
        mats = []
        for wv in omega:
            r = single * (1.0 + ts * (kappa - 1.0)) * (1.0 + ns * (wv - 1.0)) * pi[None, :]
            r = r - torch.diag(r.sum(1))
            mats.append(r / -(pi * torch.diagonal(r)).sum())
        mats = torch.stack(mats)
        leaf = mats.detach().requires_grad_(True)
        got = _exact_one(prob, "branch+Q", leaf)
        g = torch.autograd.grad(mats, [kappa, omega], got["d_Q"])
        return {"logL": np.float64(got["logL"]), "d_kappa": g[0], "d_omega": g[1], "d_branch": got["d_branch"]}
    if case["kind"] == "proposals":
        out = []
        for v, old, new in _proposal_list(case, prob, rng):
            prob.branch_rate[v] = new
            out.append(_exact_one(prob, "logL")["logL"])
            prob.branch_rate[v] = old
        return {"logL": np.array(out)}
    got = _exact_one(prob, want)
    out = {"logL": got["logL"], "site": got["site"] if case["site"] else None, "d_branch": got.get("d_branch"),
           "d_Q": got["d_Q"].cpu().numpy() if want == "branch+Q" else None}
    if want == "time":
        out["d_height"], out["d_boundary"] = got["d_height"], got["d_boundary"]
    return out
