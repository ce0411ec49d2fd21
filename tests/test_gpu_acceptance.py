"""Parity of mpv_acceptance_rates (App. C) with the fp64 oracle (needs an MI355X).

Through the C ABI (ctypes binding -> libmpv.so).  Bar: every internal node's acceptance rate
within PROB_ATOL absolute (SpecTr: plus the conditioning slack of its division factor, see
tests/parity_util.py); leaves exactly 0.
"""

import numpy as np
import pytest
import torch

import paper_2602_16994_amd as mpv
import workloads
from oracle import acceptance_oracle as acc
from oracle import mpv_oracle as orc
from tests.parity_util import PROB_ATOL, spectr_slack

pytestmark = pytest.mark.gpu

SI, TV = mpv.MPV_METHOD_SPECINFER, mpv.MPV_METHOD_TRAVERSAL
NSS, NAIVE, SPECTR = mpv.MPV_METHOD_NSS, mpv.MPV_METHOD_NAIVE, mpv.MPV_METHOD_SPECTR
SOLVERS = [SI, NSS, NAIVE, SPECTR]
NAME = {SI: "specinfer", NSS: "nss", NAIVE: "naive", SPECTR: "spectr"}


def announce(*a):
    print("[case]", *a, flush=True)


def run_and_compare(parent, target, draft, T, method, trees=None):
    alpha, counters = mpv.mpv_acceptance_rates(parent, target, draft, T, method)
    torch.cuda.synchronize()
    got = alpha.cpu().numpy()
    cnt = counters.cpu().numpy()
    B, N = got.shape
    children = orc.children_lists(parent)
    n_internal = sum(1 for ch in children if ch)
    assert cnt[4] == 0 and cnt[5] == B * n_internal
    zt, zd = target.float().cpu().numpy(), draft.float().cpu().numpy()
    host = {"parent": list(parent), "target": zt, "draft": zd}
    worst = 0.0
    for b in (range(B) if trees is None else trees):
        want = acc.acceptance_rates(method, parent, zt[b], zd[b], T)
        for n in range(N):
            if not children[n]:
                assert got[b, n] == 0.0
                continue
            tol = PROB_ATOL
            if method == SPECTR and len(children[n]) > 1:
                tol += len(children[n]) * spectr_slack(host, b, n, T, len(children[n]))
            err = abs(float(got[b, n]) - want[n])
            worst = max(worst, err / tol)
            assert err <= tol, f"tree {b} node {n} (k={len(children[n])}): {got[b, n]} vs {want[n]} (bar {tol:.1e})"
    assert np.all((got >= 0.0) & (got <= 1.0))
    print("[report] worst error / bar = %.3f, mean rate at the root %.4f" % (worst, float(got[:, 0].mean())), flush=True)
    return got


@pytest.mark.parametrize("method", SOLVERS)
@pytest.mark.parametrize("name,B", [("tiny", 1), ("v32k_root", 6), ("v128k_delayed", 4), ("v152k_root", 3), ("v262k_delayed", 2)])
def test_configurations(method, name, B):
    cfg = workloads.scaled(workloads.CONFIGS[name], B=B)
    announce("acceptance rates", name, NAME[method], f"B={cfg.B} N={cfg.N} V={cfg.V} {cfg.dtype} T={cfg.T}")
    inputs = workloads.make_inputs(cfg, "cuda")
    run_and_compare(cfg.parent, inputs["target"], inputs["draft"], cfg.T, method)


@pytest.mark.parametrize("method", SOLVERS)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_every_child_count_and_ragged_vocabulary(method, dtype):
    # nodes with 1, 2, 3, 5, 8 and 16 children; more trees than workgroups; odd V
    parent = [-1, 0, 0, 1, 1, 1, 2, 2, 2, 2, 2] + [3] * 8 + [4] * 16 + [5]
    announce("acceptance rates, irregular tree", NAME[method], dtype)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(21)
    B, N, V = 300, len(parent), 1003
    zd = (torch.randn(B, N, V, generator=gen, device="cuda") * 2.0).to(dtype)
    zt = (zd.float() + torch.randn(B, N, V, generator=gen, device="cuda")).to(dtype)
    run_and_compare(parent, zt, zd, 0.9, method, trees=range(0, B, 25))


def test_identical_models_tiny_vocabulary_and_root_only_tree():
    announce("acceptance rates, degenerate cases")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    parent = mpv.root_tree(3, 2)
    z = torch.randn(8, len(parent), 40, generator=gen, device="cuda")
    for method in (SI, NAIVE, SPECTR):
        alpha, _ = mpv.mpv_acceptance_rates(parent, z, z.clone(), 1.0, method)
        torch.cuda.synchronize()
        got = alpha.cpu().numpy()
        internal = [n for n, ch in enumerate(orc.children_lists(parent)) if ch]
        np.testing.assert_allclose(got[:, internal], 1.0, atol=1e-5)
    run_and_compare(parent, z, z.clone(), 1.0, NSS)
    # V = 2
    z2 = torch.randn(16, len(parent), 2, generator=gen, device="cuda")
    d2 = torch.randn(16, len(parent), 2, generator=gen, device="cuda")
    for method in SOLVERS:
        run_and_compare(parent, z2, d2, 0.7, method)
    # a root without children: nothing to compute
    alpha, _ = mpv.mpv_acceptance_rates([-1], torch.randn(4, 1, 64, device="cuda"), torch.randn(4, 1, 64, device="cuda"), 1.0, SI)
    torch.cuda.synchronize()
    assert torch.all(alpha == 0)


def test_errors():
    parent = [-1, 0]
    z = torch.zeros(2, 2, 16, device="cuda")
    with pytest.raises(mpv.MpvError):
        mpv.mpv_acceptance_rates(parent, z, z, 1.0, TV)          # not an OTLP solver
    with pytest.raises(mpv.MpvError):
        mpv.mpv_acceptance_rates(parent, z, z, 0.0, SI)
    alpha, _ = mpv.mpv_acceptance_rates(parent, torch.zeros(0, 2, 16, device="cuda"), torch.zeros(0, 2, 16, device="cuda"), 1.0, SI)
    assert alpha.numel() == 0


def test_benchmark_batch_sampled():
    cfg = workloads.CONFIGS["v152k_root"]
    announce("acceptance rates on the benchmark batch", f"B={cfg.B}")
    inputs = workloads.make_inputs(cfg, "cuda")
    got = run_and_compare(cfg.parent, inputs["target"], inputs["draft"], cfg.T, SI, trees=[0, 128, 255])
    # the paper's observation (Sec. 5): with i.i.d. rows there is no trend with depth here, but the
    # root (k = 8) must accept more often than the chain nodes (k = 1)
    assert got[:, 0].mean() > got[:, 1].mean()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_small_terms_are_not_lost_beside_a_large_one(dtype):
    """Equal target and draft rows: Naive's rate is sum min(p, q) = 1.  One token has almost all of the mass; a lane meets it in
    its first vector of a later sweep, and each of its other tokens is less than half a unit in the last place of the large term
    (2^-25): added one by one next to it they leave no trace (about 50 of them: 1.3e-6).  Added to each other first, a vector at
    a time, each of at most 7 vectors next to the large term is rounded by 2^-25 at most: 2.1e-7; the exponentials and the
    factors of p add 1e-7."""
    V, B = 151936, 64 if dtype == torch.bfloat16 else 24
    parent = mpv.delayed_tree(8, 0, 5)
    N = len(parent)
    print("[case] acceptance, one large term", dtype, f"B={B} N={N} V={V}", flush=True)
    row = torch.zeros(V, device="cuda")
    row[6 * 256 * (8 if dtype == torch.bfloat16 else 4)] = 17.5           # (the sweeps begin with the seventh slot of a lane)
    assert 2.0 ** -26 < 1.0 / (float(torch.tensor(17.5).exp()) + V) < 2.0 ** -25
    rows = row.to(dtype).expand(B, N, V).contiguous()
    alpha, counters = mpv.mpv_acceptance_rates(parent, rows, rows, 1.0, mpv.MPV_METHOD_NAIVE)
    torch.cuda.synchronize()
    inner = sorted(set(parent[1:]))
    err = float((alpha[:, inner].double() - 1.0).abs().max())
    print("[report] largest error:", err, flush=True)
    assert int(counters[4]) == 0 and err <= 3.1e-7
