"""Parity of mpv_nucleus_mask with the fp64 oracle, and of verification on masked rows (needs an MI355X).

Through the C ABI (ctypes binding -> libmpv.so).  Bars: the kept set, the threshold and the
number of kept tokens must be identical to the oracle's, except where the library's threshold is
the right one for a top_p within MASS_BAND of the one given (its float32 sums may stop a value
earlier or later when the mass of an upper set {z >= t} comes that close to top_p); such rows
are counted and must be few.
"""

import numpy as np
import pytest
import torch

import paper_2602_16994_amd as mpv
import workloads
from oracle import block_efficiency_oracle as beo
from oracle import mpv_oracle as orc
from oracle import nucleus_oracle as nuc
from tests.parity_util import compare_with_oracle, node_tolerances, result_to_host

pytestmark = pytest.mark.gpu

MASS_BAND = 1e-6
ALL_METHODS = [mpv.MPV_METHOD_SPECINFER, mpv.MPV_METHOD_TRAVERSAL, mpv.MPV_METHOD_NSS, mpv.MPV_METHOD_NAIVE,
               mpv.MPV_METHOD_SPECTR]


def announce(*a):
    print("[case]", *a, flush=True)


def check_rows(z, T, top_p, masked, thr, kept):
    """z: the rows given to the library (torch, on the device); the rest: its outputs."""
    zh = z.float().cpu().numpy().reshape(-1, z.shape[-1])
    mh = masked.float().cpu().numpy().reshape(zh.shape)
    th = thr.cpu().numpy().reshape(-1)
    kh = kept.cpu().numpy().reshape(-1)
    near = 0
    for r in range(len(zh)):
        tau, n_kept, margin = nuc.nucleus_threshold(zh[r], T, top_p)
        # whatever the threshold, the output is the input restricted to {z >= threshold}
        keep = zh[r] >= th[r]
        assert np.array_equal(mh[r][keep], zh[r][keep]) and np.all(np.isneginf(mh[r][~keep])), f"row {r}: not a masked copy"
        assert kh[r] == int(keep.sum()), f"row {r}: kept count {kh[r]} vs {int(keep.sum())}"
        if th[r] == tau:
            assert kh[r] == n_kept
            continue
        # another threshold: then it must be the right one for a top_p within the band of the one given,
        # i.e. its set reaches top_p - band and would not reach top_p + band without its smallest value
        p = orc.softmax_T(zh[r], T)
        with_it, without_it = float(p[keep].sum()), float(p[zh[r] > th[r]].sum())
        assert with_it >= top_p - MASS_BAND and without_it < top_p + MASS_BAND, (
            f"row {r}: threshold {th[r]} (mass {with_it:.9f}, {without_it:.9f} without its smallest value) vs "
            f"oracle {tau}, top_p {top_p}, oracle margin {margin:.3e}")
        near += 1
    return near


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [1, 7, 1003, 32000, 151936])
def test_random_rows(dtype, V):
    announce("nucleus random rows", dtype, "V", V)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    rows = 24 if V > 10000 else 64
    z = (torch.randn(rows, V, generator=gen, device="cuda") * 2.5).to(dtype)
    near = 0
    for T, top_p in ((1.0, 0.9), (1.0, 0.99), (0.6, 0.5), (1.2, 0.999)):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, T, top_p)
        torch.cuda.synchronize()
        near += check_rows(z, T, top_p, masked, thr, kept)
    print("[report] rows within the band:", near, "of", 4 * rows, flush=True)
    # flat rows over a large vocabulary: successive upper sets differ by 1e-7 of mass, less than
    # float32 sums resolve, so the band is hit often there (and only there)
    assert near <= (2 if V < 100000 else rows)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_equal_logits_are_kept_or_dropped_together(dtype):
    announce("nucleus ties", dtype)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    z = torch.randint(-4, 5, (48, 4099), generator=gen, device="cuda").to(dtype)      # nine distinct values
    for top_p in (0.3, 0.7, 0.95):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, 1.0, top_p)
        torch.cuda.synchronize()
        assert check_rows(z, 1.0, top_p, masked, thr, kept) <= 1
        assert torch.all(kept >= (z == z.max(dim=1, keepdim=True).values).sum(dim=1))


def test_top_p_one_in_place_and_rows_with_dropped_tokens():
    announce("nucleus edge cases")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    z = (torch.randn(5, 3, 777, generator=gen, device="cuda") * 2).to(torch.bfloat16)     # leading dimensions; odd V
    masked, thr, kept = mpv.mpv_nucleus_mask(z, 1.0, 1.0)
    torch.cuda.synchronize()
    assert torch.equal(masked, z) and torch.all(kept == 777) and tuple(thr.shape) == (5, 3)
    out1, thr1, kept1 = mpv.mpv_nucleus_mask(z, 0.8, 0.9)
    z2 = z.clone()
    out2, thr2, kept2 = mpv.mpv_nucleus_mask(z2, 0.8, 0.9, inplace=True)
    torch.cuda.synchronize()
    assert out2.data_ptr() == z2.data_ptr()
    assert torch.equal(out1.view(torch.int16), out2.view(torch.int16)) and torch.equal(thr1, thr2) and torch.equal(kept1, kept2)
    # rows that already hold -inf entries
    again, thr3, kept3 = mpv.mpv_nucleus_mask(out1, 0.8, 0.5)
    torch.cuda.synchronize()
    assert check_rows(out1, 0.8, 0.5, again, thr3, kept3) <= 1
    assert torch.all(kept3 <= kept1)
    # the result is the same on every call
    out4, _, _ = mpv.mpv_nucleus_mask(z, 0.8, 0.9)
    torch.cuda.synchronize()
    assert torch.equal(out1.view(torch.int16), out4.view(torch.int16))


def test_errors():
    z = torch.zeros(2, 16, device="cuda")
    for bad in (0.0, -0.5, 1.5, float("nan")):
        with pytest.raises(mpv.MpvError):
            mpv.mpv_nucleus_mask(z, 1.0, bad)
    with pytest.raises(mpv.MpvError):
        mpv.mpv_nucleus_mask(z, 0.0, 0.9)
    empty, _, _ = mpv.mpv_nucleus_mask(torch.zeros(0, 16, device="cuda"), 1.0, 0.9)
    assert empty.numel() == 0


def nucleus_inputs(cfg, top_p):
    """cfg's inputs with both logit tensors masked by the library and the draft tokens drawn again
    from the masked draft rows (x ~ q must hold for the truncated q)."""
    inputs = workloads.make_inputs(cfg, "cuda")
    mpv.mpv_nucleus_mask(inputs["target"], cfg.T, top_p, inplace=True)
    mpv.mpv_nucleus_mask(inputs["draft"], cfg.T, top_p, inplace=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(cfg.seed + 9)
    for n in range(1, cfg.N):
        q = torch.softmax(inputs["draft"][:, cfg.parent[n]].float() / cfg.T, dim=-1)
        inputs["tokens"][:, n] = torch.multinomial(q, 1, generator=gen).squeeze(1).to(torch.int32)
    torch.cuda.synchronize()
    return inputs


@pytest.mark.parametrize("method", ALL_METHODS)
@pytest.mark.parametrize("name,B,top_p", [("v32k_root", 6, 0.9), ("v128k_delayed", 4, 0.99), ("v152k_root", 3, 0.9)])
def test_verification_of_masked_rows(method, name, B, top_p):
    cfg = workloads.scaled(workloads.CONFIGS[name], B=B)
    announce("nucleus + verification", name, "method", method, "top_p", top_p)
    inputs = nucleus_inputs(cfg, top_p)
    assert torch.isneginf(inputs["target"]).any() and torch.isneginf(inputs["draft"]).any()
    res = mpv.mpv_verify(inputs["parent"], inputs["tokens"], inputs["target"], inputs["draft"], cfg.T,
                         inputs["uniforms"], method, debug=True, draw_uniforms=inputs["draw_uniforms"])
    torch.cuda.synchronize()
    got = result_to_host(res)
    host = workloads.to_host(inputs)
    rep = compare_with_oracle(method, host, cfg.T, got)
    print("[report]", rep, flush=True)
    # the bonus token is never a dropped one
    zt = host["target"]
    for b in range(cfg.B):
        stop = got["path_nodes"][b][got["accept_len"][b] - 1] if got["accept_len"][b] > 0 else 0
        if method in (mpv.MPV_METHOD_SPECINFER, mpv.MPV_METHOD_TRAVERSAL):
            assert np.isfinite(zt[b, stop, got["bonus_token"][b]])
    # expected block efficiency on the same masked rows
    be = mpv.mpv_block_efficiency(inputs["parent"], inputs["tokens"], inputs["target"], inputs["draft"], cfg.T, method)
    torch.cuda.synchronize()
    reach = be.reach_prob.cpu().numpy()
    for b in range(cfg.B):
        _, want = beo.expected_block_efficiency(method, host["parent"], host["tokens"][b], host["target"][b],
                                                host["draft"][b], cfg.T)
        tol = node_tolerances(method, host, b, cfg.T)          # 1e-5, plus SpecTr's (capped) conditioning slack
        assert np.all(np.abs(reach[b] - want) <= tol), (b, float(np.max(np.abs(reach[b] - want) - tol)))


def test_benchmark_batch_rows_sampled():
    # every row of the benchmark batch's target tensor in one launch; a sample of rows through the oracle
    cfg = workloads.CONFIGS["v152k_root"]
    announce("nucleus on the benchmark batch", f"rows={cfg.B * cfg.N} V={cfg.V}")
    inputs = workloads.make_inputs(cfg, "cuda")
    z = inputs["target"]
    masked, thr, kept = mpv.mpv_nucleus_mask(z, cfg.T, 0.9)
    torch.cuda.synchronize()
    flat = z.view(-1, cfg.V)
    rows = [0, 1, 4099, 7777, cfg.B * cfg.N - 1]
    near = check_rows(flat[rows], cfg.T, 0.9, masked.view(-1, cfg.V)[rows], thr.view(-1)[rows], kept.view(-1)[rows])
    assert near <= 1
    assert int(kept.min()) >= 1 and int(kept.max()) < cfg.V


# Row lengths around the switch of the workgroup size (2048 vectors) and around whole chunks of a sweep; row shapes that
# lead through each way of finding the threshold: "few" tokens hold the mass (the list suffices), "flat" rows (the list is
# not enough or overflows: bins), "level" rows (thousands of nearly equal logits: one bin holds more than the list).
@pytest.mark.parametrize("shape", ["few", "flat", "level"])
@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 8), (torch.bfloat16, 65), (torch.bfloat16, 8192), (torch.bfloat16, 16383), (torch.bfloat16, 16391),
                                     (torch.bfloat16, 32768), (torch.bfloat16, 40961), (torch.float32, 3), (torch.float32, 8195), (torch.float32, 16384),
                                     (torch.float32, 20481)])
def test_ways_of_finding_the_threshold(shape, dtype, V):
    announce("nucleus ways", shape, dtype, "V", V)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V + len(shape))
    rows = 6
    z = torch.randn(rows, V, generator=gen, device="cuda") * {"few": 4.0, "flat": 0.5, "level": 1e-3}[shape]
    if shape == "few":
        z[:, V // 2] += 12.0
        z[1, : V - 1] = -float("inf")                 # one token, at the end of a row that starts with -inf
        z[2] = -float("inf")                          # nothing to drop
    z = z.to(dtype)
    use = z[[r for r in range(rows) if shape != "few" or r != 2]]
    for T, top_p in ((1.0, 0.9), (0.7, 0.999)):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, T, top_p)
        place = z.clone()
        mpv.mpv_nucleus_mask(place, T, top_p, inplace=True)
        torch.cuda.synchronize()
        same = torch.int16 if dtype == torch.bfloat16 else torch.int32
        assert torch.equal(place.view(same), masked.view(same))
        if shape == "few":
            assert torch.equal(masked[2].view(same), z[2].view(same)) and int(kept[2]) == V
        sel = [r for r in range(rows) if shape != "few" or r != 2]
        near = check_rows(use, T, top_p, masked[sel], thr[sel], kept[sel])
        # float32 rows without a head: neighbouring upper sets differ by about 1/V of mass, which the band of 1e-6 resolves
        # at these lengths except where it happens to straddle one
        assert near <= 1


# Rows whose leading logits are all -inf (a masked vocabulary).  The sweep takes whole chunks of 4 vectors per lane (1024 lanes
# for rows of 2048 vectors or more, 256 for shorter ones); the -inf run covers one or two chunks, or ends a few logits before
# or after the edge of one.  Behind it: the most likely token, alone less than 1 - top_p of the mass; then dozens of likely
# tokens, which reach top_p without it; and eight tokens of equal logit, far enough apart to fall to several waves.
@pytest.mark.parametrize("dtype,V,chunk", [(torch.bfloat16, 151936, 32768), (torch.bfloat16, 100003, 32768), (torch.bfloat16, 16383, 8192),
                                           (torch.bfloat16, 15000, 8192), (torch.float32, 70000, 16384), (torch.float32, 50001, 16384),
                                           (torch.float32, 8191, 4096)])
def test_rows_that_begin_with_minus_infinity(dtype, V, chunk):
    announce("nucleus leading -inf", dtype, "V", V)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    leads = [lead for lead in (chunk, 2 * chunk, chunk - 3, chunk + 5) if lead + 2000 <= V]
    z = torch.full((3 * len(leads), V), -float("inf"), device="cuda")
    for i, lead in enumerate(leads):
        room = V - lead - 200
        step = max(1, room // 48)
        z[3 * i, lead + 57] = 2.25
        z[3 * i, lead + 200: lead + 200 + 40 * step: step] = torch.linspace(1.0, 2.0, 40, device="cuda")
        z[3 * i + 1, lead + 3: lead + 11] = 2.0
        z[3 * i + 1, lead + 200: lead + 200 + 40 * step: step] = 2.0
        z[3 * i + 2, lead:] = torch.randn(V - lead, generator=gen, device="cuda") * 3.0
    z = z.to(dtype)
    for T, top_p in ((1.0, 0.9), (0.8, 0.7)):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, T, top_p)
        torch.cuda.synchronize()
        near = check_rows(z, T, top_p, masked, thr, kept)
        assert near <= (0 if dtype == torch.bfloat16 else 1)        # (float32 rows of noise: see MASS_BAND)


# Logits and temperature with exact masses: the scale of the exponent, log2(e) / T in float32, is 1, and a token of logit -n has
# 2^-n of the largest one's mass.  Every sum below has few enough bits that its order does not matter.
EXACT_T = float(np.float32(1.4426950408889634))


def test_the_threshold_does_not_depend_on_where_the_tokens_are():
    """The same tokens in two orders: with the likely ones in front, the list of likely tokens suffices; behind 65536 tokens of
    equal logit it overflows.  top_p lies where the mass of the two million least likely tokens decides: their 2^-20 of the
    largest one's makes the most likely token alone fall short of it."""
    V = 1 << 21
    assert np.float32(1.4426950408889634 / np.float64(np.float32(EXACT_T))) == np.float32(1.0)
    z = torch.full((2, V), -41.0, device="cuda")
    z[0, 0], z[0, 1], z[0, 2: 2 + 65536] = 0.0, -1.0, -30.0
    z[1, :65536], z[1, V - 2], z[1, V - 9] = -30.0, 0.0, -1.0
    head = 1.5 + 65536 * 2.0 ** -30
    tail = (V - 65538) * 2.0 ** -41
    top_p = float(np.float32(0.5 * (1.0 / head + 1.0 / (head + tail))))
    # 1 / head - 1 / (head + tail) is 4e-7; float32 sums in any order and the rounding of top_p move the line by 6e-8 each
    assert top_p * (head + tail) > 1.0 + 2e-7 and top_p * head < 1.0 - 2e-7
    for dtype in (torch.bfloat16, torch.float32):
        announce("nucleus order of tokens", dtype)
        _, thr, kept = mpv.mpv_nucleus_mask(z.to(dtype), EXACT_T, top_p)
        torch.cuda.synchronize()
        assert thr.tolist() == [-1.0, -1.0] and kept.tolist() == [2, 2]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_repeated_calls_agree(dtype):
    """Rows whose largest logits rise along the row, so that what a wave lists depends on when it hears of the others' maxima."""
    announce("nucleus repeated calls", dtype)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    V = 131072
    z = torch.randn(48, V, generator=gen, device="cuda") * 1.5 + torch.linspace(0.0, 6.0, V, device="cuda")
    z = z.to(dtype)
    for top_p in (0.3, 0.9):
        first = mpv.mpv_nucleus_mask(z, 1.0, top_p)
        for _ in range(8):
            again = mpv.mpv_nucleus_mask(z, 1.0, top_p)
            torch.cuda.synchronize()
            assert torch.equal(again[1], first[1]) and torch.equal(again[2], first[2])
            assert torch.equal(again[0], first[0])


# Rows on which one bin (a 32nd of a binary order) holds more tokens than the list: equal logits, two or a few distinct ones,
# nearly equal ones far from zero, and around zero, where the keys of neighbouring values lie far apart.  Both sizes of the
# workgroup (2048 vectors or more, and less), rows that start at any address.
@pytest.mark.parametrize("shape", ["equal", "two", "steps", "level", "around_zero", "negative"])
@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 9001), (torch.bfloat16, 16392), (torch.bfloat16, 40961), (torch.float32, 6003),
                                     (torch.float32, 8196), (torch.float32, 20481)])
def test_rows_of_few_or_nearly_equal_logits(shape, dtype, V):
    announce("nucleus few or nearly equal logits", shape, dtype, "V", V)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    z = torch.randn(5, V, generator=gen, device="cuda")
    z = {"equal": torch.full_like(z, -1.25), "two": -1.0 * (z > 0.3), "steps": torch.round(z * 1.5) * 2.0, "level": 9.0 + z * 0.004,
         "around_zero": z * 0.002, "negative": -30.0 + z * 0.02}[shape].to(dtype)
    z[3, : V // 3] = -float("inf")
    z[4, ::7] = -float("inf")
    same = torch.int16 if dtype == torch.bfloat16 else torch.int32
    for T, top_p in ((1.0, 0.9), (0.7, 0.3), (1.3, 0.999)):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, T, top_p)
        place = z.clone()
        mpv.mpv_nucleus_mask(place, T, top_p, inplace=True)
        torch.cuda.synchronize()
        assert torch.equal(place.view(same), masked.view(same))
        # float32 rows: upper sets of neighbouring values differ by 1/V or so, 5e-5 and more; the sums are within MASS_BAND, so
        # at most a few in a hundred of such rows have one that close to top_p
        assert check_rows(z, T, top_p, masked, thr, kept) <= (1 if dtype == torch.float32 else 0)


# The largest token comes behind thousands of tokens that filled the list while the cut was too low.  It reaches top_p alone, or with
# a few of the others, or not with any list; its equals, if any, are kept with it.  (7.5 and 15 above a background of standard
# deviation 2: shares of the mass from 0.4 to 0.999.)
@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 16385), (torch.bfloat16, 50001), (torch.float32, 8000), (torch.float32, 50001),
                                     (torch.float32, 131072)])
def test_the_largest_token_comes_late(dtype, V):
    announce("nucleus late largest token", dtype, "V", V)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V + 1)
    z = torch.randn(8, V, generator=gen, device="cuda") * 2.0
    for r in range(8):
        z[r, V - 7 - r] = 8.0 + (7.5, 15.0)[r % 2] - r / 8
    z[4, V - 2] = z[4, V - 11]                           # the largest twice
    z[5, V - 500: V - 20] = 9.0                          # hundreds of equals below it
    z[6, V - 6000: V - 900] = z[6].max()                 # thousands of equals: more than any list
    z = z.to(dtype)
    for T, top_p in ((1.0, 0.9), (1.0, 0.98), (1.1, 0.7)):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, T, top_p)
        again = mpv.mpv_nucleus_mask(z, T, top_p)
        torch.cuda.synchronize()
        assert torch.equal(again[1], thr) and torch.equal(again[2], kept) and torch.equal(again[0], masked)
        assert check_rows(z, T, top_p, masked, thr, kept) <= (1 if dtype == torch.float32 else 0)


def test_one_wave_or_four_find_the_same_threshold():
    """Up to 1024 short rows share the bisection of more than 512 listed tokens among four waves, more rows leave it to one."""
    announce("nucleus, rows of 1000 listed tokens")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(41)
    z = torch.randn(1025, 1000, generator=gen, device="cuda")
    for top_p in (0.9, 0.4):
        many = mpv.mpv_nucleus_mask(z, 1.0, top_p)
        few = mpv.mpv_nucleus_mask(z[:1024], 1.0, top_p)
        torch.cuda.synchronize()
        for a, b in zip(many, few):
            assert torch.equal(a[:1024], b)
        # (upper sets of neighbouring values differ by 1e-3 of the mass)
        assert check_rows(z[:12], 1.0, top_p, few[0][:12], few[1][:12], few[2][:12]) == 0


@pytest.mark.parametrize("dtype,V,lead", [(torch.float32, 50001, 16384), (torch.float32, 6003, 4096), (torch.float32, 2000, 1),
                                          (torch.bfloat16, 100003, 32768), (torch.bfloat16, 4001, 3000)])
@pytest.mark.parametrize("mask", [-1e10, -1e30, float(torch.finfo(torch.bfloat16).min)])
def test_masked_tokens_of_any_low_logit(dtype, V, lead, mask):
    """Tokens masked by a large negative logit instead of -inf: before the first token that counts, after the last, in
    between, and rows of nothing else (nothing is dropped there)."""
    announce("nucleus masked", dtype, V, lead, mask)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V + 1)
    z = torch.randn(7, V, generator=gen, device="cuda") * 3.0
    z[:3, :lead] = mask
    z[1:5, -(V // 10):] = mask
    z[4:6][torch.rand(2, V, generator=gen, device="cuda") < 0.5] = mask
    z[6] = mask
    z = z.to(dtype)
    for T, top_p in ((1.0, 0.9), (0.7, 0.99)):
        masked, thr, kept = mpv.mpv_nucleus_mask(z, T, top_p)
        torch.cuda.synchronize()
        near = check_rows(z[:6], T, top_p, masked[:6], thr[:6], kept[:6])
        assert near <= 1
        assert torch.equal(masked[6], z[6]) and int(kept[6]) == V
