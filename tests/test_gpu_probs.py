"""GPU parity of `spec_verify_probs` (distributions handed over as probabilities, App. A's arrays) with the
oracle's probability form on the same values: the probabilities are made on the device from the seeded
synthetic logits (softmax at the workload's temperature, rounded to the input dtype) and the oracle reads
exactly those rounded values."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import workloads
from tests import parity
from tests.test_gpu_parity import _custom, _say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _probs_inputs(cfg, seed, top_k=0):
    inp = workloads.generate(cfg, seed=seed, device=DEV, top_k_target=top_k, top_k_draft=top_k and 3 * top_k)
    dt = inp["target_logits"].dtype
    P = torch.softmax(inp["target_logits"].float() / cfg.temperature, -1).to(dt)
    Q = torch.softmax(inp["draft_logits"].float() / cfg.temperature, -1).to(dt)
    # the drafter produced X_i, so q(X_i) > 0 even after rounding to the input dtype
    q_tok = torch.gather(Q.float(), 2, inp["draft_tokens"].long().unsqueeze(-1))
    assert bool((q_tok > 0).all())
    return P, Q, inp


def _host(t):
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).cpu().numpy().view(np.uint16), oracle.BF16
    return t.cpu().numpy(), oracle.F32


def _run_gpu(sv, algo, P, Q, inp, **kw):
    B, g1, _ = P.shape
    dbg = torch.full((B, g1, 3), float("nan"), dtype=torch.float32, device=DEV)
    tau, y = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"], debug_out=dbg, **kw)
    torch.cuda.synchronize()
    return {"accept_len": tau.cpu().numpy(), "next_token": y.cpu().numpy(), "dbg": dbg.cpu().numpy()}


def _run_oracle(algo, P, Q, inp):
    hp, dt = _host(P)
    hq, _ = _host(Q)
    return oracle.verify_probs(parity.ALGOS[algo][0], hp, hq, inp["draft_tokens"].cpu().numpy(),
                               inp["uniforms"].cpu().numpy(), dtype=dt)


SHAPES = [
    (1, 4, 1000, "f32"),
    (8, 8, 32000, "f32"),
    (16, 8, 128256, "bf16"),
    (4, 2, 8200, "bf16"),        # a chunk and a ragged tail, aligned
    (5, 3, 8191, "f32"),         # odd V: scalar loads
    (3, 1, 50257, "bf16"),       # gamma = 1, odd V
    (2, 64, 2000, "bf16"),       # the largest gamma
    (300, 3, 700, "f32"),
]


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", SHAPES)
def test_probs_parity(algo, B, gamma, V, dtype):
    import paper_2403_10444_amd as sv
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=1.0, T=0.8)
    P, Q, inp = _probs_inputs(cfg, seed=900 + B + gamma)
    rep = parity.compare(_run_gpu(sv, algo, P, Q, inp), _run_oracle(algo, P, Q, inp),
                         label=f"probs {B}x{gamma}x{V} {dtype} {algo}", greedy=(algo == "greedy"))
    _say(rep)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
def test_probs_with_zero_probabilities(algo):
    """Top-k warped rows: most tokens have probability exactly zero, independently in the two models."""
    import paper_2403_10444_amd as sv
    cfg = _custom(16, 6, 20000, "bf16", sigma_t=3.0, sigma_d=1.0, T=0.9)
    P, Q, inp = _probs_inputs(cfg, seed=321, top_k=40)
    assert float((P == 0).float().mean()) > 0.9
    rep = parity.compare(_run_gpu(sv, algo, P, Q, inp), _run_oracle(algo, P, Q, inp),
                         label=f"probs top-k {algo}", greedy=(algo == "greedy"))
    _say(rep)


@pytest.mark.parametrize("algo", ["block", "token"])
def test_probs_with_draft_lengths_and_padded_rows(algo):
    """Per-sequence draft lengths and padded rows (NaN in everything that must not be read): sequence b must come
    out as the oracle gives it on its leading rows."""
    import paper_2403_10444_amd as sv
    B, gamma, V = 20, 6, 12000
    cfg = _custom(B, gamma, V, "bf16", sigma_t=2.5, sigma_d=1.0, T=1.0)
    P, Q, inp = _probs_inputs(cfg, seed=55)
    lens = np.array([1 + (b * 5) % gamma for b in range(B)], dtype=np.int32)
    Pb = torch.full((B, gamma + 1, V + 24), float("nan"), dtype=P.dtype, device=DEV)
    Qb = torch.full((B, gamma, V + 8), float("nan"), dtype=Q.dtype, device=DEV)
    Pb[..., :V] = P
    Qb[..., :V] = Q
    for b in range(B):
        Pb[b, lens[b] + 1:] = float("nan")
        Qb[b, lens[b]:] = float("nan")
    got = _run_gpu(sv, algo, Pb[..., :V], Qb[..., :V], inp, draft_lens=torch.as_tensor(lens, device=DEV))
    hp, dt = _host(P)
    hq, _ = _host(Q)
    tok, uni = inp["draft_tokens"].cpu().numpy(), inp["uniforms"].cpu().numpy()
    n_safe = 0
    for g in np.unique(lens):
        sel = np.nonzero(lens == g)[0]
        ref = oracle.verify_probs(parity.ALGOS[algo][0], hp[sel, :g + 1], hq[sel, :g], tok[sel, :g], uni[sel, :g + 1], dtype=dt)
        safe = ref["margins"].min(axis=1) >= parity.MARGIN
        n_safe += int(safe.sum())
        assert np.array_equal(got["accept_len"][sel][safe], ref["accept_len"][safe])
        assert np.array_equal(got["next_token"][sel][safe], ref["next_token"][safe])
    assert n_safe >= 0.8 * B


def test_probs_unnormalised_rows_are_used_as_given():
    """The hand-computed case of the oracle's pins (gamma = 1, V = 3, rows that do not sum to one)."""
    import paper_2403_10444_amd as sv
    p = torch.tensor([[[1 / 8, 5 / 8, 1 / 4], [1 / 4, 1 / 4, 1 / 4]]], dtype=torch.float32, device=DEV)
    q = torch.tensor([[[1 / 2, 1 / 4, 1 / 8]]], dtype=torch.float32, device=DEV)
    tok = torch.zeros((1, 1), dtype=torch.int32, device=DEV)
    for algo in ("block", "token"):
        for eta, u, tau, y in ((0.3, 0.8, 0, 2), (0.3, 0.7, 0, 1), (0.2, 0.7, 1, 2), (0.2, 0.1, 1, 0)):
            uni = torch.tensor([[eta, u]], dtype=torch.float32, device=DEV)
            a, b = sv.spec_verify_probs(algo, p, q, tok, uni)
            torch.cuda.synchronize()
            assert (int(a[0]), int(b[0])) == (tau, y), (algo, eta, u)


# (where the weights are formed - by every workgroup, or by a kernel in front - and how the finishing kernel walks: the last
# positions of long drafts, rows at the edges of a wave's quarter of a chunk, thousands of rows of up to half a chunk on both sides of the rule, 5000
# of them; rows of 40 share a workgroup, packed.hpp)
@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(3, 64, 2049, "f32"), (4, 5, 2048, "bf16"), (5, 3, 4097, "bf16"), (3, 2, 8193, "f32"), (4, 1, 16383, "bf16"),
                                             (499, 3, 40, "f32"), (501, 3, 40, "bf16"), (501, 3, 4100, "bf16"),
                                             (1000, 4, 2100, "bf16"), (1001, 4, 2100, "f32"), (1001, 4, 4096, "bf16"), (1001, 4, 4097, "bf16"), (860, 6, 1030, "f32")])
def test_weights_and_walk_at_their_edges(algo, B, gamma, V, dtype):
    import paper_2403_10444_amd as sv
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.0, sigma_d=0.4, T=1.0)
    P, Q, inp = _probs_inputs(cfg, seed=B + V)
    inp["uniforms"][0, :] = 0.0                                       # the whole draft, then the first token with weight
    P[0, gamma, :5] = 0.0
    inp["uniforms"][1, gamma] = 1.0 - 2.0 ** -24                      # the last token with weight, or next to it
    ref = _run_oracle(algo, P, Q, inp)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert safe[2:].all() or safe[2:].mean() > 0.99
    got = _run_gpu(sv, algo, P, Q, inp)
    tau, y = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"])        # (sums that cannot matter left out)
    for key, plain in (("accept_len", tau), ("next_token", y)):
        assert np.array_equal(got[key][safe], ref[key][safe]), key
        assert np.array_equal(got[key], plain.cpu().numpy()), key
    # the two rows of extreme uniforms, next to an edge by their nature
    assert (got["accept_len"][0], got["next_token"][0]) == (gamma, 5)
    assert ref["margins"][1, 0] >= parity.MARGIN and got["accept_len"][1] == ref["accept_len"][1]
    t = int(ref["accept_len"][1])
    weights = P[1, t].double().cpu().numpy()
    if t < gamma:
        weights = np.maximum(ref["dbg"][1, t, 0] * weights - Q[1, t].double().cpu().numpy(), 0.0)
    assert parity.in_cell(weights, 1.0 - 2.0 ** -24, int(got["next_token"][1]))


# (rows of sixteen chunks, summed sixteen lanes to a position, and of seventeen; more positions than the segments of one pass; one launch and two; drafted tokens
# that the target rules out, and in one sequence one that the draft rules out: its ratio is infinite, its weight 1)
@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(2, 17, 131072, "bf16"), (2, 5, 131073, "bf16"), (40, 16, 131072, "bf16"), (70, 20, 9000, "f32"), (3, 33, 2500, "f32")])
def test_sums_and_weights_of_many_positions(algo, B, gamma, V, dtype):
    import paper_2403_10444_amd as sv
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.0, sigma_d=0.4, T=1.0)
    P, Q, inp = _probs_inputs(cfg, seed=B + V)
    tok = inp["draft_tokens"].long()
    P[1, gamma // 2, tok[1, gamma // 2]] = 0.0
    if algo != "greedy":
        Q[0, 2, tok[0, 2]] = 0.0
    ref = _run_oracle(algo, P, Q, inp)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert safe.any()                                                 # (the others: a uniform next to an edge, by the oracle's margin)
    got = _run_gpu(sv, algo, P, Q, inp)
    tau, y = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"])
    for key, plain in (("accept_len", tau), ("next_token", y)):
        assert np.array_equal(got[key][safe], ref[key][safe]), key
        assert np.array_equal(plain.cpu().numpy()[safe], ref[key][safe]), key
    if algo == "block":
        # (the weights: products of float probabilities' ratios through log2 in double, a dozen decimals)
        assert np.allclose(got["dbg"][..., 0], ref["dbg"][..., 0], rtol=2.0 ** -22, atol=1e-30)


@pytest.mark.parametrize("B,dtype", [(80, "f32"), (81, "f32"), (160, "bf16"), (161, "bf16")])
def test_token_verification_on_both_sides_of_what_runs_at_once(B, dtype):
    """Without the report the weights of Alg. 1 come from a kernel in front from that many workgroups on (eight per sequence here)."""
    import paper_2403_10444_amd as sv
    cfg = _custom(B, 3, 9000, dtype, sigma_t=2.0, sigma_d=0.6, T=1.0)
    P, Q, inp = _probs_inputs(cfg, seed=B)
    ref = _run_oracle("token", P, Q, inp)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert safe.mean() > 0.95
    tau, y = sv.spec_verify_probs("token", P, Q, inp["draft_tokens"], inp["uniforms"])
    assert np.array_equal(tau.cpu().numpy()[safe], ref["accept_len"][safe]) and np.array_equal(y.cpu().numpy()[safe], ref["next_token"][safe])


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(60, 1, 60000, "bf16"), (70, 1, 60000, "bf16"),      # 960 and 1120 workgroups: one launch and two (gamma < 4)
                                             (50, 4, 60000, "f32"), (52, 4, 60000, "f32")])        # 2000 and 2080 (gamma >= 4)
def test_probs_one_launch_on_whatever_the_workspace_holds(algo, B, gamma, V, dtype):
    """Calls of one launch count on words of their own call only: the same results on a workspace that was never prepared and
    holds other calls' words, ones or random bytes, call after call, and on a captured call replayed with other inputs."""
    import paper_2403_10444_amd as sv
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=1.0, T=0.8)
    P, Q, inp = _probs_inputs(cfg, seed=B + gamma)
    want = _run_gpu(sv, algo, P, Q, inp)
    parity.compare(want, _run_oracle(algo, P, Q, inp), label=f"probs {B}x{gamma}x{V} {dtype} {algo}", greedy=(algo == "greedy"))
    n = sv.spec_verify_workspace_bytes(B, gamma, V)
    gen = torch.Generator(device=DEV).manual_seed(1)
    ws = torch.randint(0, 256, (n,), dtype=torch.uint8, device=DEV, generator=gen)
    for fill in (None, None, 255, 0, 1):
        if fill is not None:
            ws.fill_(fill)
        got = _run_gpu(sv, algo, P, Q, inp, workspace=ws)
        for key in want:
            assert np.array_equal(got[key], want[key], equal_nan=True), (key, fill)
    # the sums that matter only (no report), by a graph on the same workspace; the inputs change between its replays
    tau, y = (torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"], workspace=ws, accept_len=tau, next_token=y)
    first = inp["uniforms"].clone()
    for turn in range(3):
        inp["uniforms"].copy_(first if turn == 1 else (first + 0.3 * (turn + 1)).remainder(1.0).clamp(max=1 - 2.0 ** -24))
        tau.fill_(-7), y.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        eager = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"])
        torch.cuda.synchronize()
        assert torch.equal(tau, eager[0]) and torch.equal(y, eager[1]), turn


def test_probs_more_sums_than_a_workgroup_keeps():
    """8775 sums a sequence (Alg. 4: and as many rejected masses): two launches, the second one reads them from memory again."""
    import paper_2403_10444_amd as sv
    B, gamma, V = 2, 64, 1100000
    cfg = _custom(B, gamma, V, "bf16", sigma_t=2.5, sigma_d=1.0, T=0.8)
    P, Q, inp = _probs_inputs(cfg, seed=3)
    got = _run_gpu(sv, "greedy", P, Q, inp)
    for b in range(B):
        w = torch.as_tensor(got["dbg"][b, :gamma, 0]).double()
        S = torch.stack([(float(w[i]) * P[b, i].double() - Q[b, i].double()).clamp_(min=0).sum() for i in range(gamma)]).cpu().numpy()
        R = torch.stack([(Q[b, i].double() - float(w[i]) * P[b, i].double()).clamp_(min=0).sum() for i in range(gamma)]).cpu().numpy()
        # (w is reported as a float, and the sums are of floats: 2^-24 each, and some 2^-22 for the float sums of a chunk)
        tol = 5e-7 * np.maximum(got["dbg"][b, :gamma, 0], 1.0)
        assert np.all(np.abs(got["dbg"][b, :gamma, 1] - S) <= tol)
        h = np.where(R > 0, np.minimum(S / np.maximum(R, 1e-300), 1.0), 1.0)
        assert np.all(np.abs(got["dbg"][b, 1:gamma, 2] - h[1:]) <= 1e-5)
        tests = inp["uniforms"][b, :gamma].cpu().numpy() < got["dbg"][b, 1:, 2]
        assert got["accept_len"][b] == (np.nonzero(tests)[0].max() + 1 if tests.any() else 0)
        assert 0 <= got["next_token"][b] < V


@pytest.mark.parametrize("algo", ["block", "greedy"])
def test_probs_words_that_look_like_the_next_calls(algo):
    """What an unprepared workspace holds is never taken for the call's own, also where it carries the numbers of other calls, counted on."""
    import paper_2403_10444_amd as sv
    B, gamma, V = 12, 4, 40000
    P, Q, inp = _probs_inputs(_custom(B, gamma, V, "bf16", sigma_t=2.5, sigma_d=1.0, T=0.8), seed=17)
    want = _run_gpu(sv, algo, P, Q, inp)
    ws = torch.zeros(sv.spec_verify_workspace_bytes(B, gamma, V) // 8, dtype=torch.int64, device=DEV)
    junk = int(np.float32(0.25).view(np.int32))
    for step in (1, 2, 3):
        # (waits that run out leave words of the call behind whatever a call clears)
        sv.spec_verify_debug_config(0, 0)
        try:
            _run_gpu(sv, algo, P, Q, inp, workspace=ws.view(torch.uint8))
        finally:
            sv.spec_verify_debug_config(0, -1)
        upper = (ws >> 32).cpu().numpy()
        numbers, count = np.unique(upper[upper != 0], return_counts=True)
        for _ in range(step - 1):
            _run_gpu(sv, algo, P, Q, inp)
        number = int(numbers[count.argmax()]) + step if len(numbers) else step
        ws.fill_(number << 32 | junk)
        got = _run_gpu(sv, algo, P, Q, inp, workspace=ws.view(torch.uint8))
        for key in want:
            assert np.array_equal(got[key], want[key], equal_nan=True), (key, step)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
def test_probs_recorded_calls_replayed_after_waits_that_run_out(algo):
    """A recorded call carries the same arguments every time: none of a replay's words may count for the next one, whose inputs differ."""
    import paper_2403_10444_amd as sv
    B, gamma, V = 12, 4, 40000
    P, Q, inp = _probs_inputs(_custom(B, gamma, V, "bf16", sigma_t=2.5, sigma_d=1.0, T=0.8), seed=18)
    P2, Q2, inp2 = _probs_inputs(_custom(B, gamma, V, "bf16", sigma_t=2.0, sigma_d=1.5, T=0.8), seed=19)
    ws = torch.zeros(sv.spec_verify_workspace_bytes(B, gamma, V), dtype=torch.uint8, device=DEV)
    p, q, tok, u = P.clone(), Q.clone(), inp["draft_tokens"].clone(), inp["uniforms"].clone()
    tau, y = (torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2))
    sv.spec_verify_probs(algo, p, q, tok, u, workspace=ws, accept_len=tau, next_token=y)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    sv.spec_verify_debug_config(0, 0)
    try:
        with torch.cuda.graph(graph, stream=side):
            sv.spec_verify_probs(algo, p, q, tok, u, workspace=ws, accept_len=tau, next_token=y)
    finally:
        sv.spec_verify_debug_config(0, -1)
    for turn in range(6):
        a, b, c = (P, Q, inp) if turn % 2 else (P2, Q2, inp2)
        p.copy_(a), q.copy_(b), tok.copy_(c["draft_tokens"]), u.copy_(c["uniforms"])
        tau.fill_(-7), y.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        eager = sv.spec_verify_probs(algo, p, q, tok, u)
        torch.cuda.synchronize()
        assert torch.equal(tau, eager[0]) and torch.equal(y, eager[1]), turn


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(12, 4, 40000, "bf16"), (9, 5, 12917, "f32"), (30, 3, 16389, "bf16"), (7, 8, 8192, "f32"), (40, 2, 300, "bf16"),
                                             (3, 64, 20001, "bf16")])
def test_probs_waits_that_run_out(algo, B, gamma, V, dtype):
    """The workgroup that finishes a sequence forms the shares itself that it stops waiting for: the same results, bit for bit."""
    import paper_2403_10444_amd as sv
    P, Q, inp = _probs_inputs(_custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=1.0, T=0.8), seed=B + V)
    lens = torch.tensor([1 + (3 * b) % gamma for b in range(B)], dtype=torch.int32, device=DEV)
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    runs = []
    for limit in (-1, 0, 0, -1):
        sv.spec_verify_debug_config(0, limit)
        try:
            got = _run_gpu(sv, algo, P, Q, inp, workspace=ws)
            tau, y = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"], draft_lens=lens, workspace=ws)
            runs.append((got["accept_len"], got["next_token"], got["dbg"], tau.cpu().numpy(), y.cpu().numpy()))
        finally:
            sv.spec_verify_debug_config(0, -1)
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert np.array_equal(a, b, equal_nan=True)
    assert sv.spec_verify_workspace_check(ws, B, gamma, V) == 0


# few sequences of long drafts over 1537 ... 2048 tokens: both sides of the lines to the kernels that spread a sequence's rows over the device
@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype,packed", [
    (32, 12, 1537, "bf16", False), (33, 12, 2048, "bf16", True), (32, 11, 2047, "bf16", True), (5, 15, 1536, "f32", True), (64, 10, 1537, "f32", False),
    (65, 10, 2048, "f32", True), (64, 9, 2048, "f32", True), (1, 15, 2048, "f32", False)])
def test_few_long_drafts_over_short_rows(B, gamma, V, dtype, packed, algo):
    import paper_2403_10444_amd as sv
    P, Q, inp = _probs_inputs(_custom(B, gamma, V, dtype, sigma_t=2.0, sigma_d=0.7, T=1.0), seed=B + V)
    got, ref = _run_gpu(sv, algo, P, Q, inp), _run_oracle(algo, P, Q, inp)
    assert sv.spec_verify_debug_last_form()[0] == (sv.binding.SV_FORM_SEQUENCES if packed else 0)
    tau, y = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"])
    assert sv.spec_verify_debug_last_form()[0] == (sv.binding.SV_FORM_SEQUENCES if packed else 0)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert safe.mean() >= 0.9 or B == 1
    for key, plain in (("accept_len", tau), ("next_token", y)):
        assert np.array_equal(got[key][safe], ref[key][safe]) and np.array_equal(plain.cpu().numpy()[safe], ref[key][safe]), key


# Alg. 1 without the report: both sides of the lines from which short rows go to the kernels that stop at the first failed test (32 MiB of target rows; 128)
@pytest.mark.parametrize("B,gamma,V,dtype,lanes", [
    (481, 16, 1024, "f32", 32), (482, 16, 1024, "f32", 0), (963, 16, 1024, "bf16", 32), (964, 16, 1024, "bf16", 0), (600, 15, 1024, "f32", 32),
    (455, 8, 2048, "f32", 64), (456, 8, 2048, "f32", 0), (700, 7, 2048, "f32", 64), (1985, 32, 512, "f32", 16), (1986, 32, 512, "f32", 0)])
def test_short_rows_of_which_few_are_needed(B, gamma, V, dtype, lanes):
    import paper_2403_10444_amd as sv
    P, Q, inp = _probs_inputs(_custom(B, gamma, V, dtype, sigma_t=2.0, sigma_d=1.0, T=1.0), seed=B + V)
    tau, y = sv.spec_verify_probs("token", P, Q, inp["draft_tokens"], inp["uniforms"])
    assert sv.spec_verify_debug_last_form()[:2] == ((sv.binding.SV_FORM_SEQUENCES, lanes) if lanes else (0, 0))
    some = np.array(sorted({0, 1, B // 2, B - 1, *range(0, B, 16)}))
    ref = _run_oracle("token", P[some], Q[some], {k: v[some] for k, v in inp.items()})
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert safe.mean() > 0.99
    assert np.array_equal(tau.cpu().numpy()[some][safe], ref["accept_len"][safe]) and np.array_equal(y.cpu().numpy()[some][safe], ref["next_token"][safe])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,gamma", [(30, 3), (60, 64), (700, 3)])               # (packed.hpp: workgroups of several sequences, of one)
def test_probs_rows_shorter_than_a_vector(B, gamma, dtype):
    import paper_2403_10444_amd as sv
    for V in (1, 2, 3, 5, 7, 9):
        P, Q, inp = _probs_inputs(_custom(B, gamma, V, dtype, sigma_t=1.0, sigma_d=0.5, T=1.0), seed=V + B)
        for algo in ("block", "token", "greedy"):
            got, ref = sv.spec_verify_probs(algo, P, Q, inp["draft_tokens"], inp["uniforms"]), _run_oracle(algo, P, Q, inp)
            torch.cuda.synchronize()
            tau, y = (t.cpu().numpy() for t in got)
            safe = ref["margins"].min(axis=1) >= parity.MARGIN
            assert np.array_equal(tau[safe], ref["accept_len"][safe]) and np.array_equal(y[safe], ref["next_token"][safe]), (V, algo)
            assert np.all((y >= 0) & (y < V))
