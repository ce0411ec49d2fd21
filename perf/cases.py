"""Performance cases of the verification library: what a user of it has it do, through its public Python entry points.

A case is a dict of plain values:
  kind     "verify"    one mpv_verify call on a batch of draft trees (the step of a serving loop)
           "merged"    mpv_merge_duplicates + mpv_verify on trees of distinct contexts (one shape per tree)
           "estimate"  mpv_block_efficiency (offline scoring of a tree shape)
           "rates"     mpv_acceptance_rates (offline comparison of the solvers)
           "nucleus"   mpv_nucleus_mask on the target and draft rows, then mpv_verify on the masked rows
  B, V     trees in the batch, vocabulary size
  K, L1, L2  tree: a trunk of L1 nodes, then K chains of L2 nodes (L1 = 0: root expansion)
  dtype    "f32" | "bf16" logits
  T        temperature;  method: MPV_METHOD_*;  top_p (nucleus only)
  rows     how the logits are distributed (see _rows)
  scratch  "own" (workspace reused between calls) | "library" (mpv_verify_static)

Vocabulary sizes, tree shapes, data types, temperatures and distributions are those of workloads.py, the benchmark and
the tests; draw() spreads over the ranges that these span.
"""

import math

import numpy as np
import torch

import paper_2602_16994_amd as mpv

SPECINFER, TRAVERSAL, NSS, NAIVE, SPECTR = 0, 1, 2, 3, 4


def _case(kind, B, V, K, L1, L2, dtype, T, method, rows, top_p=1.0, scratch="own", name=None):
    c = dict(kind=kind, B=B, V=V, K=K, L1=L1, L2=L2, dtype=dtype, T=T, method=method, rows=rows, top_p=top_p, scratch=scratch)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small tree: nothing but launches and dependent steps (a toy model, a unit test, the last request of a batch)
        _case("verify", 1, 1024, 2, 0, 3, "f32", 1.0, SPECINFER, "smooth", name="tiny_specinfer"),
        # one interactive request of a large model: latency of a single tree, scratch inside the library
        _case("verify", 1, 128256, 4, 2, 3, "bf16", 0.6, TRAVERSAL, "peaked", scratch="library", name="one_request_traversal"),
        # a serving batch of a 32 000-token model with float32 logits
        _case("verify", 64, 32000, 4, 0, 4, "f32", 1.0, SPECINFER, "peaked", name="v32k_root_specinfer"),
        # a serving batch on delayed trees, bottom-up rule
        _case("verify", 64, 128256, 4, 2, 3, "bf16", 0.6, TRAVERSAL, "peaked", name="v128k_delayed_traversal"),
        # the largest vocabulary, top-down rule, low acceptance
        _case("verify", 32, 262144, 8, 3, 3, "bf16", 0.8, SPECINFER, "wide", name="v262k_delayed_specinfer"),
        # the benchmark batch: more trees than the chip takes at once
        _case("verify", 256, 151936, 8, 0, 5, "bf16", 1.0, TRAVERSAL, "boosted", name="v152k_root_traversal"),
        # odd sizes throughout (rows that start at any address), a rule that draws a token at every node
        _case("verify", 37, 50001, 5, 1, 3, "bf16", 0.7, SPECTR, "boosted", name="ragged_spectr"),
        # trees of distinct contexts as drafted: overlapping paths share nodes, nearly every tree has a shape of its own
        _case("merged", 64, 128256, 4, 2, 3, "bf16", 0.6, SPECINFER, "peaked", name="v128k_merged_specinfer"),
        _case("merged", 256, 151936, 8, 0, 5, "bf16", 1.0, TRAVERSAL, "boosted", name="v152k_merged_traversal"),
        # offline: expected block efficiency of every tree, acceptance rate of the solver at every node
        _case("estimate", 64, 151936, 8, 0, 5, "bf16", 1.0, TRAVERSAL, "boosted", name="v152k_estimate_traversal"),
        _case("rates", 64, 151936, 8, 0, 5, "bf16", 1.0, SPECINFER, "boosted", name="v152k_rates_specinfer"),
        # a serving batch under nucleus sampling: every row masked, then verified
        _case("nucleus", 64, 128256, 4, 2, 3, "bf16", 1.0, TRAVERSAL, "boosted", top_p=0.9, name="v128k_nucleus_traversal"),
    ]


# logits of the largest listed case (bytes) and the share of it that the offline kinds, which read every row, may have
_MOST_BYTES = 2 * 256 * 41 * 151936 * 2
_SHARE = {"verify": 1.0, "merged": 1.0, "estimate": 0.3, "rates": 0.3, "nucleus": 0.3}


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["verify", "merged", "estimate", "rates", "nucleus"], [6, 2, 1, 1, 2])[0]
    # (float32 rows over a large vocabulary have upper sets that differ by less mass than 32-bit sums resolve: which of two
    # neighbouring thresholds comes out then depends on the order of additions, and masked rows cannot be compared one by one)
    dtype = "bf16" if kind == "nucleus" else rng.choices(["bf16", "f32"], [3, 1])[0]
    K, L1, L2 = rng.randint(2, 8), rng.choice([0, 0, 1, 2, 3]), rng.randint(2, 5)
    while 1 + L1 + K * L2 > 60:
        K -= 1
    N = 1 + L1 + K * L2
    V = _log_uniform(rng, 1000, 262144)
    if rng.random() < 0.5:
        V = max(1024, V // 64 * 64)                # padded vocabularies are as common as odd ones
    most = int(_SHARE[kind] * _MOST_BYTES / (2 * N * V * (4 if dtype == "f32" else 2)))
    B = _log_uniform(rng, 1, max(1, min(64 if kind == "nucleus" else 256, most)))
    methods = {"rates": [SPECINFER, NSS, NAIVE, SPECTR]}.get(kind, [SPECINFER, TRAVERSAL, TRAVERSAL, NSS, NAIVE, SPECTR])
    return _case(kind, B, V, K, L1, L2, dtype, rng.choice([0.6, 0.8, 1.0]), rng.choice(methods),
                 rng.choice(["smooth", "peaked", "boosted", "wide"]), top_p=rng.choice([0.9, 0.99]) if kind == "nucleus" else 1.0,
                 scratch=rng.choice(["own", "library"]) if kind == "verify" and B * N < 50000 else "own")


def _rows(style, rows, V, gen, dev):
    """rows x V draft and target logits in float32: the four distributions of the benchmark's configurations."""
    z = torch.randn(rows, V, generator=gen, device=dev)
    if style == "smooth":                          # close models
        zd, scale, sigma = z * 2.0, 1.0, 0.5
    elif style == "peaked":                        # a heavy head
        u = torch.rand(rows, V, generator=gen, device=dev).clamp_(1e-20, 1.0)
        head = z > _upper_quantile(50.0 / V)
        zd, scale, sigma = z - 3.0 * torch.log((-torch.log(u)).clamp_(min=1e-20)), 1.0, 0.9
        zd += 4.0 * head
    elif style == "boosted":                       # a smooth row with a few raised tokens
        zd, scale, sigma = z * 2.5 + 5.0 * (z > _upper_quantile(20.0 / V)), 1.0, 1.2
    else:                                          # "wide": a sharp draft, a flatter target
        zd, scale, sigma = z * 3.0, 0.8, 1.5
    return zd, scale * zd + sigma * torch.randn(rows, V, generator=gen, device=dev)


def _upper_quantile(p):
    return math.sqrt(2.0) * float(torch.erfinv(torch.tensor(1.0 - 2.0 * min(p, 0.4), dtype=torch.float64)))


def _nucleus_probs(q, top_p):
    """The rows of q truncated to the smallest upper set that holds top_p, not renormalised."""
    s = q.sort(dim=-1, descending=True).values
    last = (s.cumsum(dim=-1) < top_p).sum(dim=-1, keepdim=True).clamp_(max=q.shape[-1] - 1)
    return q * (q >= s.gather(-1, last))


def prepare(case, seed):
    B, V, dev = case["B"], case["V"], torch.device("cuda")
    parent = mpv.delayed_tree(case["K"], case["L1"], case["L2"])
    N = len(parent)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    target = torch.empty(B, N, V, dtype=dtype, device=dev)
    draft = torch.empty(B, N, V, dtype=dtype, device=dev)
    chunk = max(1, (1 << 27) // (N * V))
    for b0 in range(0, B, chunk):
        b1 = min(B, b0 + chunk)
        zd, zt = _rows(case["rows"], (b1 - b0) * N, V, gen, dev)
        draft[b0:b1] = zd.view(b1 - b0, N, V).to(dtype)
        target[b0:b1] = zt.view(b1 - b0, N, V).to(dtype)
        del zd, zt
    merged = case["kind"] == "merged"
    tokens = torch.zeros(B, N, dtype=torch.int32, device=dev)
    same = {}                                      # merged: (tree, node of the parent's context, token) -> first slot drafted for it
    node = np.zeros((B, N), dtype=np.int64)
    for n in range(1, N):                          # drafting: every slot's token is drawn from its parent's draft row
        q = torch.softmax(draft[:, parent[n]].float() / case["T"], dim=-1)
        if case["kind"] == "nucleus":
            q = _nucleus_probs(q, case["top_p"])
        tokens[:, n] = torch.multinomial(q, 1, generator=gen).squeeze(1).to(torch.int32)
        if merged:                                 # models are functions of the context: equal contexts have equal rows
            drawn = tokens[:, n].cpu().tolist()
            node[:, n] = [same.setdefault((b, int(node[b, parent[n]]), drawn[b]), n) for b in range(B)]
            again = np.flatnonzero(node[:, n] != n)
            if again.size:
                ib, im = torch.from_numpy(again).to(dev), torch.from_numpy(node[again, n]).to(dev)
                draft[ib, n] = draft[ib, im]
                target[ib, n] = target[ib, im]
    state = dict(case=case, parent=parent, tokens=tokens, target=target, draft=draft, out=None)
    state["uniforms"] = torch.rand(B, N, generator=gen, device=dev)
    state["draw_uniforms"] = torch.rand(B, N, generator=gen, device=dev)
    if merged:
        state["tokens_host"] = tokens.cpu().numpy()
    if case["kind"] == "nucleus":
        state["masked"] = (torch.empty_like(target), torch.empty_like(draft))
    return state


def _verify(s, target, draft, **more):
    c = s["case"]
    draws = s["draw_uniforms"] if c["method"] >= NSS else None
    s["out"] = r = mpv.mpv_verify(s["parent"], s["tokens"], target, draft, c["T"], s["uniforms"], c["method"], out=s["out"],
                                  draw_uniforms=draws, static_scratch=c["scratch"] == "library", **more)
    return [r.accept_len, r.path_nodes, r.path_tokens, r.bonus_token]


def run(s):
    c = s["case"]
    if c["kind"] == "verify":
        return _verify(s, s["target"], s["draft"])
    if c["kind"] == "merged":
        merged_parent, context_node = mpv.mpv_merge_duplicates(s["parent"], s["tokens_host"])
        more = {"context_node": torch.from_numpy(context_node).to("cuda")} if c["method"] == SPECTR else {}
        return _verify(s, s["target"], s["draft"], merged_parent=merged_parent, **more)
    if c["kind"] == "estimate":
        s["out"] = r = mpv.mpv_block_efficiency(s["parent"], s["tokens"], s["target"], s["draft"], c["T"], c["method"], out=s["out"])
        return [r.expected, r.reach_prob]
    if c["kind"] == "rates":
        return [mpv.mpv_acceptance_rates(s["parent"], s["target"], s["draft"], c["T"], c["method"])[0]]
    zt, tau_t, kept_t = mpv.mpv_nucleus_mask(s["target"], c["T"], c["top_p"], out=s["masked"][0])
    zd, tau_d, kept_d = mpv.mpv_nucleus_mask(s["draft"], c["T"], c["top_p"], out=s["masked"][1])
    return [zt, tau_t, kept_t, zd, tau_d, kept_d] + _verify(s, zt, zd)


def work(case):
    """Bytes: rows are read once, at the nodes that the operation cannot do without.  A verification needs the row pairs
    along the path that it accepts (Traversal: of one path down to a leaf) and the row that the bonus token is drawn from;
    how far a path is accepted is what these distributions give.  Operations: a dozen per element of a pair."""
    parent = mpv.delayed_tree(case["K"], case["L1"], case["L2"])
    depth, inner = case["L1"] + case["L2"], len(set(parent[1:]))
    row = case["V"] * (4 if case["dtype"] == "f32" else 2)
    if case["kind"] in ("estimate", "rates"):
        return {"bytes": case["B"] * inner * 2.0 * row, "flops": case["B"] * inner * 12.0 * case["V"]}
    accepted = {"smooth": 0.8, "peaked": 0.7, "boosted": 0.4, "wide": 0.15}[case["rows"]]
    pairs = depth if case["method"] == TRAVERSAL else 0.0 if case["method"] == NSS else min(depth, 1.0 + accepted * depth)
    single = 0.5 if case["method"] != NSS else 1.0 + (0.3 if case["rows"] in ("boosted", "wide") else 0.6) * depth
    need = {"bytes": case["B"] * (2.0 * pairs + single) * row, "flops": case["B"] * 12.0 * (pairs + single) * case["V"]}
    if case["kind"] == "nucleus":
        rows = 2.0 * case["B"] * len(parent)
        need = {"bytes": need["bytes"] + 2.0 * rows * row, "flops": need["flops"] + 6.0 * rows * case["V"]}
    return need


def tolerance(case):
    # Probabilities: against float64, the 2-norm over all nodes is off by at most 7e-7 and one value by at most 2.5e-6
    # (SpecInfer's rates on "boosted" rows; the other rules and rows by less), four times that is allowed.
    # Whole numbers: a decision within rounding of its uniform may fall the other way (row sums in 32 bits are good to
    # about 1e-7).  The nucleus thresholds are values of the row.
    if case["kind"] in ("estimate", "rates"):
        return {"rel": 3e-6, "max": 1e-5}
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.01}
