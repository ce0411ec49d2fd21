"""Parity of the HIP library with the fp64 oracle (needs an MI355X).

Every test goes through the C ABI (ctypes binding -> libmpv.so).  Each case
prints its name and shape before touching the GPU.
"""

import numpy as np
import pytest
import torch

import paper_2602_16994_amd as mpv
import workloads
from oracle import mpv_oracle as orc
from tests.parity_util import SUM_REL_ERR, check_properties, compare_with_oracle, result_to_host

pytestmark = pytest.mark.gpu

SI, TV = mpv.MPV_METHOD_SPECINFER, mpv.MPV_METHOD_TRAVERSAL
NSS, NAIVE, SPECTR = mpv.MPV_METHOD_NSS, mpv.MPV_METHOD_NAIVE, mpv.MPV_METHOD_SPECTR
METHOD_NAME = {SI: "specinfer", TV: "traversal", NSS: "nss", NAIVE: "naive", SPECTR: "spectr"}
ALL_METHODS = [SI, TV, NSS, NAIVE, SPECTR]


def announce(*a):
    print("[case]", *a, flush=True)


def run_library(inputs, T, method, debug=True):
    res = mpv.mpv_verify(inputs["parent"], inputs["tokens"], inputs["target"], inputs["draft"], T,
                         inputs["uniforms"], method, debug=debug, draw_uniforms=inputs.get("draw_uniforms"))
    torch.cuda.synchronize()
    return result_to_host(res)


def run_case(cfg, method, trees=None, debug=True):
    announce(cfg.name, METHOD_NAME[method], f"B={cfg.B} N={cfg.N} V={cfg.V} {cfg.dtype} T={cfg.T}")
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, method, debug)
    if debug:
        # the production path (no debug outputs: irrelevant node tasks are skipped) must decide alike
        lean = run_library(inputs, cfg.T, method, debug=False)
        for key in ("accept_len", "path_nodes", "path_tokens", "bonus_token"):
            assert np.array_equal(got[key], lean[key]), f"{key} differs between debug and production runs"
        assert lean["counters"][4] == 0 and got["counters"][4] == 0, "dependency wait timed out"
        assert lean["counters"][5] <= got["counters"][5]
    host = workloads.to_host(inputs)
    check_properties(host["parent"], cfg.V, got, host["tokens"])
    rep = compare_with_oracle(method, host, cfg.T, got, trees=trees, check_debug=debug)
    print("[report]", rep, "counters", got["counters"].tolist(), flush=True)
    return rep, got


def assert_everything_compared(cfg, rep):
    """On the five benchmark configurations: every test that can be performed with probability above
    1e-6 is compared at the flat bar (compare_with_oracle does that for every input).  The others
    ("remote": they follow rejections that cannot happen, or the seventh and eighth rejection under
    one node) are compared with the bar float32 terms allow for the residual mass they are computed
    from; only where that mass is below float32 resolution, or at the zero-mass corner, is a number
    left out (parity_util.remote_tolerance, fragile_tests), and those must stay a minority.
    No SpecTr tolerance may hit its cap."""
    left_out = rep["fragile_tests"] + rep["noise_tests"]
    tests = rep["trees"] * (cfg.N - 1)
    assert left_out <= rep["remote_tests"] + rep["fragile_tests"] and left_out < 0.5 * tests, rep
    assert rep.get("capped_slacks", 0) == 0, rep


def run_benchmark_config(cfg, method):
    """One of the five benchmark configurations (possibly with fewer trees)."""
    rep, got = run_case(cfg, method)
    assert_everything_compared(cfg, rep)
    return rep, got


# ---------------------------------------------------------------- the five configurations

@pytest.mark.parametrize("method", ALL_METHODS)
def test_config1_tiny(method):
    run_benchmark_config(workloads.CONFIGS["tiny"], method)


def test_config2_v32k_root_specinfer():
    # full vocabulary and tree, 6 of the 64 trees
    run_benchmark_config(workloads.scaled(workloads.CONFIGS["v32k_root"], B=6), SI)


@pytest.mark.parametrize("method", ALL_METHODS)
def test_config3_v128k_delayed(method):
    run_benchmark_config(workloads.scaled(workloads.CONFIGS["v128k_delayed"], B=4), method)


def test_config4_v152k_root_traversal_small_batch():
    run_benchmark_config(workloads.scaled(workloads.CONFIGS["v152k_root"], B=3), TV)


@pytest.mark.parametrize("method", ALL_METHODS)
def test_config5_v262k_delayed(method):
    run_benchmark_config(workloads.scaled(workloads.CONFIGS["v262k_delayed"], B=2), method)


@pytest.mark.parametrize("method", [NSS, NAIVE, SPECTR])
def test_config2_and_4_token_following_walks(method):
    # the two root-expanded configurations with the solvers whose output token may be another draft token
    run_benchmark_config(workloads.scaled(workloads.CONFIGS["v32k_root"], B=6), method)
    run_benchmark_config(workloads.scaled(workloads.CONFIGS["v152k_root"], B=3), method)


@pytest.mark.parametrize("method", [NSS, NAIVE, SPECTR])
@pytest.mark.parametrize("V,dtype", [(12, "bf16"), (37, "f32")])
def test_drawn_tokens_are_followed_in_small_vocabularies(method, V, dtype):
    """With a dozen tokens the drawn token is a child's token most of the time (and equal-token
    siblings are common): the walk must move to the first such child, draw again there, and so on."""
    cfg = workloads.Config(f"follow_V{V}", B=300, V=V, K=4, L1=0, L2=3, dtype=dtype, T=1.1,
                           methods=[method], draft_sigma=1.0, target_sigma=0.6, seed=4242 + V)
    rep, got = run_case(cfg, method)
    assert rep["mean_accept_len"] > 0.1               # the walks do get somewhere
    assert np.any(got["accept_len"] >= 2)             # and some follow more than one token


class TreeRows:
    """host["target"] / host["draft"] for a batch too large to copy at once: tree b's rows are
    copied to the host (widened to float32, which is exact) when the oracle asks for them."""

    def __init__(self, tensor):
        self.tensor = tensor
        self.last = (None, None)

    def __getitem__(self, b):
        if self.last[0] != b:
            self.last = (b, self.tensor[b].float().cpu().numpy())
        return self.last[1]


def full_size_case(cfg, method, debug_trees):
    """A benchmark configuration at full size, in the launch configuration the benchmark times (no
    debug outputs): every tree's decisions against the oracle; then the per-node probabilities of
    `debug_trees`, run as a batch of their own with the debug outputs on, which must decide alike."""
    announce(cfg.name, METHOD_NAME[method], "full size", f"B={cfg.B} N={cfg.N} V={cfg.V}")
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, method, debug=False)
    assert got["counters"][4] == 0, "dependency wait timed out"
    host = {
        "parent": inputs["parent"],
        "tokens": inputs["tokens"].cpu().numpy(),
        "uniforms": inputs["uniforms"].cpu().numpy(),
        "draw_uniforms": inputs["draw_uniforms"].cpu().numpy(),
        "target": TreeRows(inputs["target"]),
        "draft": TreeRows(inputs["draft"]),
    }
    check_properties(host["parent"], cfg.V, got, host["tokens"])
    rep = compare_with_oracle(method, host, cfg.T, got, check_debug=False)
    assert rep["trees"] == cfg.B
    print("[report]", rep, "counters", got["counters"].tolist(),
          "mean accepted length (all trees)", float(got["accept_len"].mean()), flush=True)
    sub = {k: (v[debug_trees].contiguous() if torch.is_tensor(v) else v) for k, v in inputs.items()}
    got2 = run_library(sub, cfg.T, method, debug=True)
    rep2 = compare_with_oracle(method, workloads.to_host(sub), cfg.T, got2)
    if method in (SI, TV):
        assert_everything_compared(cfg, rep2)
    for key in ("accept_len", "path_nodes", "path_tokens", "bonus_token"):
        assert np.array_equal(got2[key], got[key][debug_trees]), key
    print("[report]", rep2, flush=True)


def test_config4_full_size_every_tree():
    # the batch the benchmark times: all 256 trees against the oracle, per-node probabilities of 16
    full_size_case(workloads.CONFIGS["v152k_root"], TV, list(range(0, 256, 16)))


@pytest.mark.parametrize("name,method", [("v32k_root", SI), ("v128k_delayed", SI), ("v128k_delayed", TV),
                                         ("v262k_delayed", SI), ("v262k_delayed", TV)])
def test_configs_2_3_5_full_size_every_tree(name, method):
    cfg = workloads.CONFIGS[name]
    full_size_case(cfg, method, list(range(0, cfg.B, max(1, cfg.B // 4)))[:4])


# ---------------------------------------------------------------- shapes, tails, edge cases

RAGGED = [
    # (V, dtype, K, L1, L2, B, T)
    (1000, "f32", 3, 0, 2, 5, 1.0),       # V % 4 == 0 but rows of 4000 B
    (1023, "f32", 2, 1, 2, 4, 0.7),       # rows misaligned to 16 B
    (1001, "bf16", 3, 1, 1, 4, 1.2),      # odd V: rows start at 2-byte offsets
    (50257, "bf16", 4, 0, 3, 3, 0.8),     # several tiles and a ragged tail
    (50257, "f32", 2, 2, 2, 2, 0.2),      # cold temperature
    (7, "f32", 2, 0, 2, 9, 1.0),          # vocabulary smaller than a vector tile
    (1, "bf16", 2, 0, 1, 2, 1.0),         # a single token
    (4096, "bf16", 16, 0, 1, 3, 1.0),     # maximum children under one node
    (2048, "f32", 1, 0, 12, 3, 1.0),      # one deep chain (single path)
    (8192, "bf16", 1, 5, 0, 3, 1.0),      # trunk only (K=1, L2=0)
    (3000, "bf16", 4, 3, 4, 2, 1.0),      # N = 20
]


@pytest.mark.parametrize("method", ALL_METHODS)
@pytest.mark.parametrize("V,dtype,K,L1,L2,B,T", RAGGED)
def test_ragged_shapes(method, V, dtype, K, L1, L2, B, T):
    cfg = workloads.Config(f"ragged_V{V}_{dtype}_K{K}_{L1}_{L2}", B=B, V=V, K=K, L1=L1, L2=L2, dtype=dtype,
                           T=T, methods=[method], draft_sigma=2.0, target_sigma=1.0, seed=V + 31 * K + L1)
    run_case(cfg, method)


# How a row is split over a team's workgroups (the launch picks the team size from V, B and the
# chip): the cases below sit on the edges of that choice.
TEAM_SHAPES = [
    # (V, dtype, K, L1, L2, B, T, trees compared)
    (151937, "bf16", 2, 0, 2, 130, 1.0, 12),   # more trees than teams: the fewest members that hold a row (not a power
                                              # of two), one slot per lane beyond the kept ones; odd V: misaligned rows,
                                              # head elements with the first member, tail with the last
    (450001, "bf16", 2, 0, 1, 2, 0.9, 2),      # beyond what 16 members keep on chip: the rest is read again in every sweep
    (1 << 21, "bf16", 2, 0, 1, 1, 1.0, 1),     # the largest vocabulary the boundary admits
    (300001, "f32", 2, 1, 1, 2, 1.0, 2),       # float rows, 16 members, ragged tail
    (24577, "bf16", 3, 0, 2, 200, 1.0, 8),     # a row that just fits one workgroup, many trees
]


@pytest.mark.parametrize("method", [SI, TV, mpv.MPV_METHOD_SPECTR])
@pytest.mark.parametrize("V,dtype,K,L1,L2,B,T,ntrees", TEAM_SHAPES)
def test_team_shapes(method, V, dtype, K, L1, L2, B, T, ntrees):
    cfg = workloads.Config(f"team_V{V}_{dtype}_B{B}", B=B, V=V, K=K, L1=L1, L2=L2, dtype=dtype,
                           T=T, methods=[method], draft_sigma=2.0, target_sigma=1.0, seed=V % 9973 + B)
    step = max(1, B // ntrees)
    run_case(cfg, method, trees=list(range(0, B, step))[:ntrees])


@pytest.mark.parametrize("method", [SI, TV])
@pytest.mark.parametrize("scale", [2000.0, 2e-4])
def test_logit_magnitudes(method, scale):
    """bf16 rows are kept on chip in half precision: logits of thousands and of thousandths (with a
    temperature to match) must come out as exactly as ordinary ones."""
    cfg = workloads.Config(f"scale_{scale}", B=4, V=40000, K=3, L1=1, L2=2, dtype="bf16", T=0.5 * scale,
                           methods=[method], draft_sigma=2.0 * scale, target_sigma=1.0 * scale, seed=77)
    run_case(cfg, method)


@pytest.mark.parametrize("method", ALL_METHODS)
def test_root_only_tree(method):
    # N = 1: nothing to verify, the bonus token is a plain sample from p(.|root)
    cfg = workloads.Config("root_only", B=5, V=5000, K=1, L1=0, L2=0, dtype="bf16", T=1.0,
                           methods=[method], draft_sigma=2.0, target_sigma=1.0, seed=99)
    rep, got = run_case(cfg, method)
    assert np.all(got["accept_len"] == 0)


@pytest.mark.parametrize("method", ALL_METHODS)
def test_irregular_tree(method):
    parent = [-1, 0, 0, 1, 1, 2, 5, 5, 0, 8, 9]
    announce("irregular tree", METHOD_NAME[method])
    cfg = workloads.Config("irregular", B=6, V=2500, K=1, L1=0, L2=0, dtype="f32", T=0.9,
                           methods=[method], draft_sigma=2.0, target_sigma=1.2, seed=5)
    cfg.parent = parent
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, method)
    rep = compare_with_oracle(method, workloads.to_host(inputs), cfg.T, got)
    print("[report]", rep, flush=True)


@pytest.mark.parametrize("method", [SI, TV])
def test_identical_models_accept_first_leaf(method):
    announce("p == q", METHOD_NAME[method])
    cfg = workloads.Config("same", B=4, V=3000, K=3, L1=1, L2=2, dtype="bf16", T=1.0,
                           methods=[method], draft_sigma=2.0, target_sigma=0.0, seed=17)
    inputs = workloads.make_inputs(cfg, "cuda")
    inputs["target"] = inputs["draft"].clone()
    got = run_library(inputs, cfg.T, method)
    assert np.all(got["accept_len"] == 3)
    assert np.all(got["path_nodes"] == np.array([1, 2, 3]))
    compare_with_oracle(method, workloads.to_host(inputs), cfg.T, got)


@pytest.mark.parametrize("method", ALL_METHODS)
def test_duplicate_sibling_tokens_and_masked_vocabulary(method):
    # equal tokens under one parent are separate nodes; -inf logits have zero mass
    announce("duplicates + -inf", METHOD_NAME[method])
    cfg = workloads.Config("dups", B=8, V=640, K=4, L1=0, L2=2, dtype="f32", T=1.0,
                           methods=[method], draft_sigma=1.5, target_sigma=1.5, seed=23)
    inputs = workloads.make_inputs(cfg, "cuda")
    inputs["tokens"][:, 3] = inputs["tokens"][:, 1]          # chains 1 and 2 start with the same token
    inputs["tokens"][:, 5] = inputs["tokens"][:, 1]
    inputs["target"][:, :, 100:200] = float("-inf")           # tokens the target can never emit
    got = run_library(inputs, cfg.T, method)
    host = workloads.to_host(inputs)
    compare_with_oracle(method, host, cfg.T, got)
    assert not np.any((got["bonus_token"] >= 100) & (got["bonus_token"] < 200))
    for b in range(cfg.B):
        for t in got["path_tokens"][b][: got["accept_len"][b]]:
            assert not (100 <= t < 200)


@pytest.mark.parametrize("method", ALL_METHODS)
@pytest.mark.parametrize("T", [0.2, 1.0])
def test_peaked_rows_long_vocabulary(method, T):
    """Rows kept on chip use a per-lane reference fixed at the start of the sweep;
    a few logits far above everything else (40 units, T = 0.2: 288 binary orders)
    overflow that form and must take the online repeat."""
    announce("peaked rows", METHOD_NAME[method], T)
    cfg = workloads.Config("peaked", B=3, V=131072, K=3, L1=1, L2=1, dtype="bf16", T=T,
                           methods=[method], draft_sigma=1.0, target_sigma=0.7, seed=77)
    inputs = workloads.make_inputs(cfg, "cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    for name, boost in (("draft", 40.0), ("target", 38.0)):
        idx = torch.randint(4096, cfg.V, (cfg.B, cfg.N, 3), generator=gen, device="cuda")
        inputs[name].scatter_add_(2, idx, torch.full(idx.shape, boost, device="cuda", dtype=inputs[name].dtype))
    # draft tokens must still come from the (now peaked) draft rows
    for n in range(1, cfg.N):
        q = torch.softmax(inputs["draft"][:, cfg.parent[n]].float() / T, dim=-1)
        inputs["tokens"][:, n] = torch.multinomial(q, 1, generator=gen).squeeze(1).to(torch.int32)
    got = run_library(inputs, T, method)
    rep = compare_with_oracle(method, workloads.to_host(inputs), T, got)
    print("[report]", rep, flush=True)


@pytest.mark.parametrize("method", ALL_METHODS)
def test_many_small_tasks_through_the_queue(method):
    """Far more node tasks than workgroups, short rows, a bushy tree: the task queue hands out
    thousands of tasks, Traversal appends children level after level.  Decisions of every tree
    are compared with the oracle; per-node probabilities on a sample."""
    announce("queue stress", METHOD_NAME[method])
    cfg = workloads.Config("queue_stress", B=1500, V=96, K=1, L1=0, L2=0, dtype="f32", T=1.0,
                           methods=[method], draft_sigma=1.0, target_sigma=0.7, seed=404)
    cfg.parent = [-1, 0, 0, 0, 1, 1, 2, 4, 4, 5, 6, 6, 7, 9, 9, 10, 12, 13]
    inputs = workloads.make_inputs(cfg, "cuda")
    host = workloads.to_host(inputs)
    lean = run_library(inputs, cfg.T, method, debug=False)
    assert lean["counters"][4] == 0
    rep = compare_with_oracle(method, host, cfg.T, lean, check_debug=False)
    print("[report]", rep, "counters", lean["counters"].tolist(), flush=True)
    full = run_library(inputs, cfg.T, method, debug=True)
    compare_with_oracle(method, host, cfg.T, full, trees=range(0, cfg.B, 50))
    for key in ("accept_len", "path_nodes", "path_tokens", "bonus_token"):
        assert np.array_equal(full[key], lean[key])


@pytest.mark.parametrize("method", [SI, TV])
def test_more_trees_than_workgroups_delayed_tree(method):
    """More trees than workgroups, a trunk before the branching node: Traversal then handles the
    first branch before the rest of the branching node (which gets a second task only if
    nothing in that branch is accepted), SpecInfer runs only the nodes on the accepted path.
    Decisions of every tree against the oracle, and against the run that computes every node."""
    announce("many trees, delayed tree", METHOD_NAME[method])
    cfg = workloads.Config("many_delayed", B=700, V=1536, K=3, L1=2, L2=2, dtype="bf16", T=0.9,
                           methods=[method], draft_sigma=1.5, target_sigma=1.0, seed=808)
    inputs = workloads.make_inputs(cfg, "cuda")
    host = workloads.to_host(inputs)
    lean = run_library(inputs, cfg.T, method, debug=False)
    assert lean["counters"][4] == 0
    rep = compare_with_oracle(method, host, cfg.T, lean, check_debug=False)
    print("[report]", rep, "counters", lean["counters"].tolist(), flush=True)
    full = run_library(inputs, cfg.T, method, debug=True)
    compare_with_oracle(method, host, cfg.T, full, trees=range(0, cfg.B, 35))
    for key in ("accept_len", "path_nodes", "path_tokens", "bonus_token"):
        assert np.array_equal(full[key], lean[key])
    n_internal = 3 + 3                                   # root, trunk, branching node, first node of each branch
    assert full["counters"][5] == cfg.B * n_internal     # every node task ran
    assert lean["counters"][5] < full["counters"][5]     # not so when only decisions are wanted


@pytest.mark.parametrize("B,V,dtype", [(511, 64, "f32"), (512, 64, "f32"), (513, 64, "f32"),       # 512 teams of one
                                       (47, 40000, "bf16"), (97, 40000, "bf16"), (257, 40000, "bf16")])   # teams of several
@pytest.mark.parametrize("method,L2", [(SI, 2), (SI, 1), (TV, 2), (TV, 1), (NSS, 2)])
def test_first_tasks_are_counted_off_once(method, L2, B, V, dtype):
    """As many trees as teams, one less, one more, and more: a team's first task comes with its last
    member, the further ones are asked for ahead of time, from a node task or while a token is sampled.
    Every tree must get its outcome, and a tree's node tasks run once: a top-down walk's are those of the inner nodes it
    comes to, NSS has none, and Traversal's are the root's where that is the only inner node (L2 = 1; with more it
    depends on which branches are followed at the same time)."""
    announce("first tasks", METHOD_NAME[method], B, V, L2)
    cfg = workloads.Config("first_tasks", B=B, V=V, K=2, L1=0, L2=L2, dtype=dtype, T=1.0,
                           methods=[method], draft_sigma=1.5, target_sigma=1.0, seed=77)
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, method, debug=False)
    assert got["counters"][4] == 0 and got["counters"][7] <= B
    tasks = int(got["counters"][5])
    if method == SI:
        assert tasks == int(np.minimum(got["accept_len"] + 1, L2).sum())
    elif method == NSS:
        assert tasks == 0
    elif L2 == 1:
        assert tasks == B
    else:
        assert B <= tasks <= 3 * B
    compare_with_oracle(method, workloads.to_host(inputs), cfg.T, got, trees=range(0, B, max(1, B // 40)), check_debug=False)
    assert np.all((got["bonus_token"] >= 0) & (got["bonus_token"] < V)) and np.all((got["accept_len"] >= 0) & (got["accept_len"] <= L2))


@pytest.mark.parametrize("B,V,K,L1,L2", [(2, 1500, 4, 2, 3), (24, 1500, 8, 0, 5), (96, 1500, 4, 2, 3), (96, 16000, 8, 0, 5),
                                         (200, 1500, 3, 1, 4), (300, 700, 8, 0, 3)])
def test_branches_are_handed_to_idle_teams(B, V, K, L1, L2):
    """Traversal with more teams than trees: the branches of a tree are followed at the same time, by teams that
    wait for the dispatcher, take its place when it finds a task for itself, and are handed a task and the lock by
    turns.  Every tree is decided (nothing may be left in a mailbox), and as the oracle decides."""
    announce("idle teams", B, V, K, L1, L2)
    cfg = workloads.Config("idle_teams", B=B, V=V, K=K, L1=L1, L2=L2, dtype="bf16", T=0.8,
                           methods=[TV], draft_sigma=2.0, target_sigma=1.0, seed=78)
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, TV, debug=False)
    assert got["counters"][4] == 0
    compare_with_oracle(TV, workloads.to_host(inputs), cfg.T, got, trees=range(0, B, max(1, B // 24)), check_debug=False)
    for _ in range(20):
        again = run_library(inputs, cfg.T, TV, debug=False)
        assert again["counters"][4] == 0
        for key in ("accept_len", "path_nodes", "path_tokens", "bonus_token"):
            assert np.array_equal(got[key], again[key])


@pytest.mark.parametrize("B", [199, 200, 201, 207, 208])
def test_the_branching_node_is_split_whatever_the_number_of_trees_modulo_8(B):
    """No team to spare (teams of several members, as many as trees): a tree's branching node handles its first child first.
    Teams that are added only to make a multiple of 8 do not count as spare."""
    announce("split", B)
    cfg = workloads.Config("split", B=B, V=40000, K=2, L1=0, L2=2, dtype="bf16", T=1.0,
                           methods=[TV], draft_sigma=1.5, target_sigma=1.0, seed=80)
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, TV, debug=False)
    assert got["counters"][4] == 0 and got["counters"][7] > 0          # rejected first subtrees: the node's second task
    compare_with_oracle(TV, workloads.to_host(inputs), cfg.T, got, trees=range(0, B, B // 20), check_debug=False)


@pytest.mark.parametrize("V,dtype,B", [(5, "bf16", 3), (63, "f32", 3), (515, "bf16", 3), (1025, "f32", 700), (33001, "bf16", 3),
                                       (300001, "f32", 2), (524293, "bf16", 2)])
@pytest.mark.parametrize("method", ALL_METHODS)
def test_the_draw_reads_rows_of_any_offset(method, V, dtype, B):
    """The drawn token where rows start at any element of a 16-byte vector, are shorter than one, end inside one, fill a
    part of a tile, and where a wave has more tiles than it keeps in registers."""
    announce("draw", METHOD_NAME[method], B, V, dtype)
    cfg = workloads.Config("draw", B=B, V=V, K=2, L1=0, L2=2, dtype=dtype, T=1.0,
                           methods=[method], draft_sigma=1.5, target_sigma=1.0, seed=79)
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, method, debug=False)
    assert got["counters"][4] == 0
    compare_with_oracle(method, workloads.to_host(inputs), cfg.T, got, trees=range(0, B, max(1, B // 30)), check_debug=False)


@pytest.mark.parametrize("V,dtype,B", [
    (8192, "bf16", 400), (8200, "bf16", 400),                             # one member: 4 slots (SpecTr: 6), the most of the short kernel;
    (12287, "bf16", 400), (12288, "bf16", 400), (12296, "bf16", 400),     # one vector more
    (24576, "bf16", 400), (24577, "bf16", 400), (25601, "bf16", 400),     # one member: 12 slots full, one more, half of it
    (12287, "f32", 400),
    (425984, "bf16", 2), (425992, "bf16", 2),                             # 16 members: the 13th slot full; one vector too many
])
@pytest.mark.parametrize("method", ALL_METHODS[:1] + ALL_METHODS[2:])
def test_the_draw_at_the_edges_of_what_is_kept(method, V, dtype, B):
    """Top-down rules draw from the part that a workgroup keeps: at its last slot, at the one that is read again, and
    beyond them, where the rows are read once more by the other way (which the debug run takes everywhere)."""
    cfg = workloads.Config("kept edges", B=B, V=V, K=2, L1=0, L2=1, dtype=dtype, T=0.9, methods=[method], draft_sigma=1.0, target_sigma=0.7, seed=97 + V)
    rep, _ = run_case(cfg, method, trees=range(min(B, 12)))
    assert rep["trees"] == min(B, 12)


@pytest.mark.parametrize("V,dtype", [(8192, "bf16"), (8200, "bf16"), (8195, "bf16"), (12287, "bf16"), (12288, "bf16"), (12296, "bf16"), (4095, "f32"), (6145, "f32")])
@pytest.mark.parametrize("method", ALL_METHODS[:1] + ALL_METHODS[2:])
def test_a_child_s_rows_asked_for_ahead_at_the_edges_of_what_the_registers_hold(method, V, dtype):
    """Parts of 4 slots (SpecTr: 6), the most of the kernel that asks for the first child's pair while its parent is tested, and
    one vector to either side: walks on through an inner first child (taken up from where it lies), through the second
    (what was asked for is overwritten) or neither.  Rows of a child start at other offsets than their parent's."""
    announce("ahead edges", METHOD_NAME[method], V, dtype)
    B = 400
    cfg = workloads.Config("ahead edges", B=B, V=V, K=2, L1=0, L2=2, dtype=dtype, T=0.9, methods=[method], draft_sigma=2.5, target_sigma=1.0, seed=101 + V)
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_library(inputs, cfg.T, method, debug=False)
    assert got["counters"][4] == 0
    compare_with_oracle(method, workloads.to_host(inputs), cfg.T, got, trees=range(0, B, 4), check_debug=False)
    if method != NSS:                                 # (which tests nothing and asks for rows as it comes to them)
        through = lambda child, length: np.any((got["path_nodes"][:, 0] == child) & (got["accept_len"] == length))
        assert through(1, 1) and through(1, 2) and np.any(got["accept_len"] == 0)
        assert method == NAIVE or (through(3, 1) and through(3, 2))          # (Naive comes to the second child by its draws alone)


@pytest.mark.parametrize("V,dtype", [(1000, "f32"), (5003, "bf16"), (20000, "bf16"), (131072, "f32")])
def test_a_draft_row_without_any_token_leaves_the_target_row_to_draw_from(V, dtype):
    """The draft row is masked throughout and so is the child's token in the target row: the child is rejected, no mass
    can be taken from p, and the token is drawn from p."""
    announce("masked draft row", V, dtype)
    B = 8
    gen = torch.Generator(device="cuda").manual_seed(V)
    target = torch.randn(B, 2, V, generator=gen, device="cuda").mul_(2.0)
    target[:, 0, 7] = float("-inf")
    draft = torch.full((B, 2, V), float("-inf"), device="cuda")
    inputs = dict(parent=[-1, 0], tokens=torch.full((B, 2), 7, dtype=torch.int32, device="cuda"), uniforms=torch.rand(B, 2, generator=gen, device="cuda"),
                  target=target.to(torch.float32 if dtype == "f32" else torch.bfloat16), draft=draft.to(torch.float32 if dtype == "f32" else torch.bfloat16))
    got = run_library(inputs, 1.0, SI, debug=False)
    assert got["counters"][4] == 0 and np.all(got["accept_len"] == 0)
    for b in range(B):
        token, gap = orc.sample_index(orc.softmax_T(inputs["target"][b, 0].float().cpu().numpy(), 1.0), float(inputs["uniforms"][b, 0]))
        assert gap < 1e-6 or got["bonus_token"][b] == token


@pytest.mark.parametrize("V,dtype", [(1003, "f32"), (1003, "bf16"), (20011, "bf16")])
@pytest.mark.parametrize("method", [NAIVE, SPECTR])
def test_a_draw_without_any_mass_is_the_same_with_and_without_debug_outputs(method, V, dtype):
    """Equal rows and a child's token that is masked in both: the child is rejected and (p - q)_+ has no mass.  Rows start at
    any element of a 16-byte vector."""
    announce("no mass", METHOD_NAME[method], V, dtype)
    B = 12
    gen = torch.Generator(device="cuda").manual_seed(V)
    rows = torch.randn(B, 2, V, generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    rows[:, 0, 9] = float("-inf")
    inputs = dict(parent=[-1, 0], tokens=torch.full((B, 2), 9, dtype=torch.int32, device="cuda"), target=rows, draft=rows.clone(),
                  uniforms=torch.rand(B, 2, generator=gen, device="cuda"), draw_uniforms=torch.rand(B, 2, generator=gen, device="cuda"))
    with_outputs, lean = run_library(inputs, 1.0, method), run_library(inputs, 1.0, method, debug=False)
    assert lean["counters"][4] == 0 and np.all(lean["accept_len"] == 0)
    assert np.array_equal(lean["bonus_token"], with_outputs["bonus_token"])


@pytest.mark.parametrize("method,V,B", [(SI, 4096, 64), (SI, 65536, 24), (NAIVE, 65536, 100), (SI, 131072, 100)])
def test_a_draw_weighs_p_against_q_no_worse_than_its_terms_are(method, V, B):
    """Partitions between 2^63 and 2^64, where a float that is lowered by one loses its last bit: p and q, alike to 1e-4 in the
    first half of the row and to 2e-3 in the second, then differ by 2.6e-6 too much or too little, and a draw from
    (p - q)_+ in the first half lands 2.6 % off.  Allowed: the rounding of rho (2^-24) and what the sums are off by
    (SUM_REL_ERR), over 1e-4."""
    announce("p against q", METHOD_NAME[method], V, B)
    near = 1e-4
    rng = np.random.default_rng(V + B)
    base = rng.standard_normal((B, V))
    base += ((63.0 + rng.uniform(0.05, 0.95, B)) * np.log(2.0) - np.log(np.sum(np.exp(base), axis=1)))[:, None]
    apart = rng.choice([-1.0, 1.0], (B, V)) * np.where(np.arange(V) < V // 2, near, 2e-3)
    apart[:, V - 1] = -8.0                            # the child's token: rejected
    draft, target = base.astype(np.float32), (base + apart).astype(np.float32)
    uniforms = np.full((B, 2), 0.99, dtype=np.float32)
    cdfs = []
    for b in range(B):
        r = np.maximum(orc.softmax_T(target[b], 1.0) - orc.softmax_T(draft[b], 1.0), 0.0)
        cdfs.append(np.cumsum(r) / np.sum(r))
        uniforms[b, 0] = 0.5 * cdfs[b][V // 2 - 1]
    rows = lambda x: torch.from_numpy(np.stack([x, x], axis=1)).cuda()
    inputs = dict(parent=[-1, 0], tokens=torch.full((B, 2), V - 1, dtype=torch.int32, device="cuda"), target=rows(target), draft=rows(draft),
                  uniforms=torch.from_numpy(uniforms).cuda(), draw_uniforms=torch.from_numpy(uniforms).cuda())
    got = run_library(inputs, 1.0, method, debug=False)
    assert got["counters"][4] == 0 and np.all(got["accept_len"] == 0)
    off = []
    for b in range(B):
        t, u = int(got["bonus_token"][b]), float(uniforms[b, 0])
        off.append(max(0.0, (cdfs[b][t - 1] if t else 0.0) - u, u - cdfs[b][t]) / u)
    print("[report] off by at most", max(off), flush=True)
    assert max(off) <= (2.0 ** -24 + SUM_REL_ERR) / near


def test_a_draw_at_a_leaf_weighs_its_waves_exactly_against_each_other():
    """Two tokens in the shares of two waves, ten apart: where the draw goes from one to the other is found to a float of u.
    Each token's mass is off by one v_exp_f32 (2^-24 or a little less), the rest is exact: 1e-7 in the mean square over the
    rows (with a float 2^(difference of the waves' references) between them, 2.5e-7)."""
    announce("leaf, two waves")
    V, rows, steps = 1024, 96, np.arange(-16, 17)
    # a temperature whose log2(e)/T is a float
    T = min((np.float32(0.9 + i * 1e-5) for i in range(20000)), key=lambda t: abs(float(np.float32(np.log2(np.e) / float(t))) * float(t) / np.log2(np.e) - 1.0))
    rng = np.random.default_rng(5)
    a, gap = rng.uniform(-4.0, 4.0, rows).astype(np.float32), rng.uniform(9.0, 11.0, rows).astype(np.float32)
    z = np.full((rows, V), -np.inf, dtype=np.float32)
    z[:, 300], z[:, 900] = a, a + gap                 # (64 vectors of 4 elements per wave: the second wave's and the fourth's)
    step = np.array([orc.softmax_T(z[r, [300, 900]], float(T))[0] for r in range(rows)])
    at = step.astype(np.float32).view(np.int32)
    u = (at[:, None] + steps[None, :]).astype(np.int32).view(np.float32)
    B = u.size
    target = torch.from_numpy(np.repeat(z, len(steps), axis=0)).cuda().view(B, 1, V)
    inputs = dict(parent=[-1], tokens=torch.zeros(B, 1, dtype=torch.int32, device="cuda"), target=target, draft=target,
                  uniforms=torch.from_numpy(np.ascontiguousarray(u).reshape(B, 1)).cuda())
    got = run_library(inputs, float(T), SI, debug=False)
    assert got["counters"][4] == 0
    first = (got["bonus_token"].reshape(rows, len(steps)) == 300).sum(axis=1)          # u below the step: the first token
    assert np.all((first > 0) & (first < len(steps)))
    found = np.array([0.5 * (float(u[r, first[r] - 1]) + float(u[r, first[r]])) for r in range(rows)])
    off = np.sqrt(np.mean((found / step - 1.0) ** 2))
    print("[report] off by", off, "at most", np.max(np.abs(found / step - 1.0)), flush=True)
    assert off <= 1e-7


@pytest.mark.parametrize("V,dtype,B,members", [(20000, "bf16", 300, 2), (12500, "f32", 100, 4), (60000, "bf16", 90, 8), (50001, "bf16", 37, 7), (262144, "bf16", 2, 16)])
@pytest.mark.parametrize("method", ALL_METHODS)
def test_teams_whose_members_are_on_different_chiplets(method, V, dtype, B, members, monkeypatch):
    """Consecutive workgroups run on different chiplets: a team of them counts its members there and exchanges words at device
    scope, which no launch of the library chooses.  (members: of the top-down rules' teams.  K = 3, trunk 1, chains of 2: draws, branches and drawn tokens that are followed;
    the drafted tokens of a tree come from a few, so that they are.)"""
    announce("teams apart", METHOD_NAME[method], B, V, dtype, members)
    lib = mpv.binding.load_library()
    apart = lib.mpv_test_verify_teams_apart
    apart.restype, apart.argtypes = lib.mpv_verify.restype, lib.mpv_verify.argtypes
    cfg = workloads.Config("apart", B=B, V=V, K=3, L1=1, L2=2, dtype=dtype, T=0.8,
                           methods=[method], draft_sigma=3.0, target_sigma=1.0, seed=83 + V)
    inputs = workloads.make_inputs(cfg, "cuda")
    together = [run_library(inputs, cfg.T, method, debug=debug) for debug in (True, False)]
    monkeypatch.setattr(lib, "mpv_verify", apart)
    for expect, debug in zip(together, (True, False)):
        got = run_library(inputs, cfg.T, method, debug=debug)
        assert got["counters"][4] == 0
        for key in ("accept_len", "path_nodes", "path_tokens", "bonus_token") + (("accept_prob", "final_residual") if debug else ()):
            assert np.array_equal(got[key], expect[key]), key                        # (the same parts, the same order of additions)
    compare_with_oracle(method, workloads.to_host(inputs), cfg.T, got, trees=range(0, B, max(1, B // 10)), check_debug=False)


def test_out_of_range_tokens_are_counted_not_followed():
    announce("bad tokens")
    cfg = workloads.Config("badtok", B=3, V=500, K=2, L1=0, L2=2, dtype="f32", T=1.0,
                           methods=[SI], draft_sigma=1.0, target_sigma=1.0, seed=3)
    inputs = workloads.make_inputs(cfg, "cuda")
    inputs["tokens"][:, 1] = cfg.V + 5
    inputs["tokens"][:, 3] = -2
    for method in (SI, TV):
        got = run_library(inputs, cfg.T, method, debug=False)
        assert got["counters"][3] == 2 * cfg.B
        assert np.all(got["accept_len"] == 0)


def test_empty_batch_is_a_no_op():
    announce("B = 0")
    z = torch.empty(0, 3, 16, device="cuda")
    res = mpv.mpv_verify([-1, 0, 0], torch.empty(0, 3, dtype=torch.int32, device="cuda"), z, z, 1.0,
                         torch.empty(0, 3, device="cuda"), SI, max_depth=1)
    torch.cuda.synchronize()
    assert res.accept_len.numel() == 0


def test_results_are_bitwise_reproducible():
    announce("determinism")
    cfg = workloads.scaled(workloads.CONFIGS["v128k_delayed"], B=8, V=40000)
    inputs = workloads.make_inputs(cfg, "cuda")
    a = run_library(inputs, cfg.T, TV)
    b = run_library(inputs, cfg.T, TV)
    for k in a:
        if a[k] is not None:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


def test_every_uniform_decides_as_the_oracle_does():
    """Many decisions on few logits: one tree's rows are shared by 512 batch
    entries that differ only in their uniforms, so every branch of both rules is
    exercised against the oracle (whose per-node probabilities are computed once)."""
    announce("uniform sweep")
    cfg = workloads.Config("usweep", B=1, V=1500, K=3, L1=1, L2=2, dtype="bf16", T=1.0,
                           methods=[SI, TV], draft_sigma=2.0, target_sigma=1.5, seed=41)
    one = workloads.make_inputs(cfg, "cuda")
    B = 512
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    inputs = {
        "parent": one["parent"],
        "tokens": one["tokens"].expand(B, -1).contiguous(),
        "target": one["target"].expand(B, -1, -1).contiguous(),
        "draft": one["draft"].expand(B, -1, -1).contiguous(),
        "uniforms": torch.rand(B, cfg.N, generator=gen, device="cuda"),
    }
    host = workloads.to_host(inputs)
    for method in (SI, TV):
        got = run_library(inputs, cfg.T, method, debug=False)
        rep = compare_with_oracle(method, host, cfg.T, got, check_debug=False)
        stops = {tuple(r[:l]) for r, l in zip(got["path_nodes"].tolist(), got["accept_len"].tolist())}
        print("[report]", METHOD_NAME[method], rep, "distinct accepted paths", len(stops), flush=True)
        assert len(stops) >= 3


# ---------------------------------------------------------------- the other entry points

@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [1, 5, 1024, 4099, 151936])
def test_row_stats(dtype, V):
    announce("row_stats", dtype, V)
    rows = 7
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    z = (torch.randn(rows, V, generator=gen, device="cuda") * 4).to(dtype)
    for T in (0.2, 1.0, 1.2):
        out = mpv.mpv_row_stats(z, T).cpu().numpy().astype(np.float64)
        zz = z.float().cpu().numpy().astype(np.float64)
        m = zz.max(axis=1)
        lz = np.log(np.exp((zz - m[:, None]) / T).sum(axis=1))
        assert np.array_equal(out[:, 0], m)
        np.testing.assert_allclose(out[:, 1], lz, atol=1e-5)


def test_fill_uniforms_matches_the_documented_generator():
    announce("fill_uniforms")
    for seed, count in [(0, 1), (12345, 1000), (2 ** 63 + 11, 257)]:
        got = mpv.mpv_fill_uniforms(seed, count).cpu().numpy()
        want = orc.uniforms_from_seed(seed, count)
        assert got.dtype == np.float32 and np.array_equal(got, want)


@pytest.mark.parametrize("mask", [-3e9, -1e10, -1e30, float(np.finfo(np.float32).min), -np.inf])
@pytest.mark.parametrize("method", ALL_METHODS)
def test_masked_tokens_of_any_low_logit(method, mask):
    """float32 rows with tokens masked by a large negative logit: whole waves of them at the front (a wave's first vector),
    the padding at the end, single ones in between, and rows whose first element before the aligned vectors is one."""
    announce("masked", METHOD_NAME[method], mask)
    cfg = workloads.Config("masked", B=12, V=2102, K=2, L1=1, L2=2, dtype="f32", T=0.8,
                           methods=[method], draft_sigma=1.5, target_sigma=1.0, seed=81)
    inputs = workloads.make_inputs(cfg, "cuda")
    off = torch.rand(cfg.V, generator=torch.Generator().manual_seed(5)) < 0.3
    off[:700] = True
    off[-90:] = True
    off[1500] = False
    for rows, n in ((inputs["target"], 3), (inputs["draft"], 5)):
        few = off.clone()
        few[700::n] = True                                    # (the two rows do not mask the same tokens)
        few[1500] = False
        rows[:, :, few] = mask
        rows[3:5, :, 1:] = torch.where(rows[3:5, :, 1:] == mask, torch.randn_like(rows[3:5, :, 1:]), rows[3:5, :, 1:])
    gen = torch.Generator(device="cuda").manual_seed(6)
    for n in range(1, cfg.N):
        q = torch.softmax(inputs["draft"][:, cfg.parent[n]] / cfg.T, dim=-1)
        inputs["tokens"][:, n] = torch.multinomial(q, 1, generator=gen).squeeze(1).to(torch.int32)
    host = workloads.to_host(inputs)
    for debug in (True, False):
        got = run_library(inputs, cfg.T, method, debug)
        assert got["counters"][4] == 0
        compare_with_oracle(method, host, cfg.T, got, check_debug=debug)
    rows = inputs["draft"].view(-1, cfg.V)
    out = mpv.mpv_row_stats(rows, cfg.T).cpu().numpy().astype(np.float64)
    z = rows.double().cpu()
    assert np.array_equal(out[:, 0], z.max(dim=1).values.numpy())
    np.testing.assert_allclose(out[:, 1], torch.logsumexp((z - z.max(dim=1, keepdim=True).values) / cfg.T, dim=1).numpy(), atol=1e-5)
