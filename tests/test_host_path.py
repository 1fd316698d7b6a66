"""The library's host path on a recording stand-in for the HIP runtime (no GPU, no kernel runs): failures a
GPU run cannot bring about, and the order and number of the calls around the launches."""
import pytest

import fake_hip

CREATE = """
rng = np.random.default_rng(5)
prob = W.random_problem(rng, {taxa}, {states}, {patterns}, n_categories={categories}, n_intervals={intervals}, reversible=True)
lik = from_problem(prob, {precision!r}, **{flags!r})
"""


def created(states=4, taxa=40, patterns=50, categories=1, intervals=2, precision="fp32", **flags):
    return CREATE.format(states=states, taxa=taxa, patterns=patterns, categories=categories, intervals=intervals,
                         precision=precision, flags=flags)


@pytest.mark.parametrize("flags", [{"grad_branch": True}, {"grad_branch": True, "grad_Q": True}])
def test_results_buffer_survives_a_failed_pinned_allocation(tmp_path, flags):
    """A refused staging buffer (more rates at once than it held) leaves the results' place on the host as it
    was: the next evaluation's launch does not write through a null pointer."""
    fake_hip.run(tmp_path, created(**flags) + """
fake.fake_fail_host_mallocs(1)
nodes = np.arange(prob.parent.shape[0] - 1)
try:
    lik.set_branch_rates(nodes, np.ones(len(nodes)))
except _abi.EpochError as e:
    assert e.code == _abi.EPOCH_ERR_OOM
fake.fake_fail_host_mallocs(0)
fake.fake_clear()
lik.evaluate(branch=True, site=True)
dst = [int(l.split()[-1], 16) for l in log() if "publish_kernel" in l]
assert dst and all(d > 4096 for d in dst), dst
""")


def test_refused_branch_rates_change_nothing(tmp_path):
    """Rates of a call that returned an error are not handed over by a later one."""
    fake_hip.run(tmp_path, created(grad_branch=True) + """
n = prob.parent.shape[0]
fake.fake_fail_copies(1)
try:
    lik.set_branch_rates(np.arange(70), np.full(70, 3.0))
    assert False
except _abi.EpochError as e:
    assert e.code == _abi.EPOCH_ERR_HIP
fake.fake_clear()
lik.set_branch_rates(np.arange(1, n - 1), np.full(n - 2, 2.0))
sent = [l.split() for l in log() if l.startswith("copy") and int(l.split()[2]) == 8 * n]
assert len(sent) == 1 and float(sent[0][-1]) == prob.branch_rate[0], sent
""")


@pytest.mark.parametrize("grad", [False, True])
def test_child_vectors_kept_for_a_gradient_only(tmp_path, grad):
    """Seven states, three columns, 40 taxa: the child vectors of every branch with a gradient, of the tips without."""
    rows = 79 if grad else 40
    fake_hip.run(tmp_path, created(states=7, patterns=3, precision="fp64", grad_branch=grad) + f"""
sizes = [int(l.split()[1]) for l in log() if l.startswith("malloc")]
one = 3 * 8 * 8
assert {rows} * one in sizes and {79 + 40 - rows} * one not in sizes, sizes
""")


def launched(tmp_path, evaluate="", **kw):
    """Names of the kernels one evaluation launches, shortened to what stands before the template's arguments."""
    out = fake_hip.run(tmp_path, created(**kw) + f"""
fake.fake_clear()
lik.evaluate({evaluate})
print("\\n".join(l.split()[2] for l in log() if l.startswith("launch")))
""")
    return out.split()


@pytest.mark.parametrize("states, patterns, flags, kernel, absent", [
    # no gradient to keep child vectors for, and no run of several categories
    (16, 1, {"categories": 4}, "post_level_generic", "few_"),
    (16, 1, {"categories": 4, "grad_branch": True}, "few_post_level", "post_level_generic"),
    # a lane per 256-byte row: sixteen columns of one node are more than a run's level takes
    (20, 16, {"kernel": "generic", "grad_branch": True}, "few_post_level", "few_post_run"),
    (7, 1, {"grad_branch": True}, "few_post_run", "post_level"),
    (7, 1, {}, "few_post_run", "post_level"),
])
def test_kernels_for_few_patterns(tmp_path, states, patterns, flags, kernel, absent):
    names = launched(tmp_path, states=states, patterns=patterns, precision="fp64", taxa=64, **flags)
    assert any(kernel in n for n in names) and not any(absent in n for n in names), names


@pytest.mark.parametrize("taxa, patterns, categories, precision, listed", [
    (16, 1000, 4, "fp64", True), (100, 20011, 4, "fp64", True),
    (150, 50000, 1, "fp64", False), (150, 20000, 4, "fp32", False)])
def test_short_list_or_levels(tmp_path, taxa, patterns, categories, precision, listed):
    """Either form where it was measured the faster one."""
    names = launched(tmp_path, taxa=taxa, patterns=patterns, categories=categories, precision=precision)
    assert any("nuc_post_list" in n for n in names) == listed, names
    assert any("nuc_post_level" in n for n in names) != listed, names


def test_batch_waits_for_its_members_before_it_tunes(tmp_path):
    """What a setter left on a member's stream is waited for before the batch's first replay, a timed one."""
    fake_hip.run(tmp_path, created(states=61, taxa=6, patterns=20) + """
other = from_problem(prob, "fp32")
batch = EpochBatchEvaluator([lik, other])
lik.set_branch_rates([0], [2.0])
fake.fake_clear()
batch.evaluate(grad_branch=False)
lines = log()
first = next(i for i, l in enumerate(lines) if l.startswith("graph"))
assert "sync (nil)" in lines[:first], lines[:first]
assert sum(l.startswith("graph") for l in lines) > 6  # it tuned
""")


@pytest.mark.parametrize("kw", [{}, {"precision": "fp64"}, {"states": 7, "patterns": 2}, {"states": 61, "patterns": 90}])
def test_proposals_allocate_no_pinned_memory(tmp_path, kw):
    """Lists of any length, and more rates at once than travel in a launch's arguments."""
    fake_hip.run(tmp_path, created(**kw) + """
lik.set_option("tree_walk", 0)
lik.evaluate()
n = prob.parent.shape[0]
fake.fake_clear()
for k in (1, 4, 16, 64, n - 1):
    lik.set_branch_rates(np.arange(k), np.full(k, 1.5))
    lik.evaluate()
assert lik.work_counts()[0] > 0
assert not [l for l in log() if l.startswith("host")], log()
""")


@pytest.mark.parametrize("states, categories, grad", [(7, 1, True), (7, 1, False), (14, 3, True), (14, 3, False)])
def test_workspace_holds_the_child_vectors(tmp_path, states, categories, grad):
    """With a workspace nothing pattern-sized is allocated beside it; one without room for the child vectors
    is taken, by the per-level kernels; one below that is refused."""
    fake_hip.run(tmp_path, created(states=states, patterns=3, categories=categories, precision="fp64") + f"""
class Workspace:
    def __init__(self, n):
        self.n, self.raw = n, ctypes.create_string_buffer(n + 256)
    def data_ptr(self): return (ctypes.addressof(self.raw) + 255) // 256 * 256
    def numel(self): return self.n
    def element_size(self): return 1

C, P, K, N = {categories}, 3, {states}, 40
row, rows = C * P * (8 if K == 7 else 16) * 8, (2 * N - 1 if {grad} else N)
few = rows * row if {grad} or C == 1 else 0
full = EpochLikelihood.workspace_bytes(N, P, K, C, "fp64", grad_branch={grad})
least = full - -(-few // 256) * 256
for n in (full, least, least - 1):
    fake.fake_clear()
    try:
        lik = from_problem(prob, "fp64", grad_branch={grad}, workspace=Workspace(n))
    except _abi.EpochError as e:
        assert e.code == _abi.EPOCH_ERR_ARG and n < least
        continue
    assert n >= least
    lik.evaluate(branch={grad})
    lines = log()
    assert not few or "malloc %d" % few not in lines
    assert any("few_post" in l for l in lines) == bool(few and n == full), (n, few)
    assert any("post_level_generic" in l for l in lines) == (not few or n == least), (n, few)
    lik.close()
""")


@pytest.mark.parametrize("last, blocks", [(1, 65), (1041, 66), (4096, 256), (4097, 65)])
def test_root_blocks_of_pattern_chunks(tmp_path, last, blocks):
    """Chunks of 4,160 patterns and a last one: the root launches hold the blocks of the chunk with the most."""
    out = fake_hip.run(tmp_path, created(states=20, taxa=4, patterns=4160 + last, hbm_budget_bytes=4160 * 3 * 132) + """
assert lik.kernel_path() == "matrix_core64"
fake.fake_clear()
lik.evaluate()
print("\\n".join(l for l in log() if "codon_root" in l))
""")
    assert [int(l.split()[3]) for l in out.splitlines()] == [blocks] * 2, out


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_chain_split_back_to_its_default(tmp_path, precision):
    """The line on long epoch chains that an instance chose by itself can be had back (-1)."""
    fake_hip.run(tmp_path, created(states=20, patterns=2, intervals=40, precision=precision) + """
def launches():
    fake.fake_clear()
    lik.evaluate()
    return [l.split()[2:] for l in log() if l.startswith("launch")]

default = launches()
lik.set_option("chain_split", 0)
assert launches() != default  # some chain was cut
lik.set_option("chain_split", -1)
assert launches() == default
for bad in (-2, (1 << 30) + 1):
    try:
        lik.set_option("chain_split", bad)
        assert False
    except _abi.EpochError as e:
        assert e.code == _abi.EPOCH_ERR_ARG
""")


@pytest.mark.parametrize("states, taxa, intervals, precision, apart", [
    (61, 40, 3, "fp64", True),     # 316 units
    (40, 683, 1, "fp64", False),   # 4,095 units of one segment: 33 us together, 39 apart
    (20, 1024, 1, "fp32", False),  # 4,094 units
    (61, 800, 1, "fp64", True),    # 6,396 units: one wavefront per SIMD in the joint form
    (61, 800, 1, "fp32", False),
    (20, 1024, 14, "fp32", True)])
def test_derivative_on_wavefronts_of_its_own(tmp_path, states, taxa, intervals, precision, apart):
    """The P stage's two forms, by the units of a launch, their tiles and the longest chain."""
    out = fake_hip.run(tmp_path, created(states=states, taxa=taxa, patterns=1, intervals=intervals, precision=precision,
                                         grad_branch=True) + """
lik.set_option("eigen_precision", 1)
lik.set_option("chain_split", 0)
fake.fake_clear()
lik.evaluate(branch=True)
print("\\n".join(l for l in log() if "pstage_mfma" in l))
""")
    assert ("Lb1ELb1ELi" in out) == apart and ("Lb1ELb0ELi" in out) != apart, out


def test_no_memory_for_the_child_vectors(tmp_path):
    """Refused, they leave an instance of the per-level kernels, and nothing else is allocated after them."""
    fake_hip.run(tmp_path, created(states=7, patterns=3, precision="fp64", grad_branch=True) + """
lik.close()
few = 79 * 3 * 8 * 8
fake.fake_fail_malloc_of(ctypes.c_size_t(few))
fake.fake_clear()
lik = EpochLikelihood(40, 3, 7, 1, 1, 1, "fp64", grad_branch=True)
assert [l for l in log() if l.startswith("malloc")][-1] == "malloc %d" % few
lik.close()
lik = from_problem(prob, "fp64", grad_branch=True)
fake.fake_clear()
lik.evaluate(branch=True)
names = [l.split()[2] for l in log() if l.startswith("launch")]
assert any("post_level_generic" in n for n in names) and not any("few_" in n for n in names), names
""")
