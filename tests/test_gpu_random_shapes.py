"""Seeded random shapes and options against the oracle: batch, draft length, vocabulary (tiny, odd, chunk
boundaries, wide rows), dtype, algorithm, temperature, kernel path, top-k masking, per-sequence draft
lengths and padded rows (everything that must not be read is NaN), two calls in a row on one workspace.
Sequences are compared with the oracle's result on their own leading rows."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2403_10444_amd as sv
import workloads
from tests import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PATHS = {"default": 0, "staged": 1, "fused": 3, "fused-large": 4}


def _draw_case(rng, it, probs):
    B = int(rng.integers(1, 40))
    gamma = int(rng.integers(1, 13))
    V = int(rng.choice([rng.integers(2, 300), rng.integers(300, 9000), rng.integers(9000, 70000),
                        rng.integers(70000, 300000), 8192, 16384, 131072, 131080, 8 * rng.integers(100, 6000)]))
    dtype = str(rng.choice(["bf16", "f32"]))
    T = float(rng.choice([0.5, 0.8, 1.0, 1.5]))
    cfg = workloads.Config(f"random{it}", B, gamma, V, dtype, float(rng.choice([1.0, 3.0, 6.0])),
                           float(rng.choice([0.3, 1.0, 2.5])), T, bool(rng.integers(0, 2)), 1)
    return dict(cfg=cfg, algo=str(rng.choice(["block", "token", "greedy"])), path=str(rng.choice(list(PATHS))),
                top_k=int(rng.choice([0, 0, 0, 5, 50])) if V > 200 else 0, use_lens=bool(rng.integers(0, 2)),
                pad_t=int(rng.choice([0, 0, 8, 3, 24])), pad_d=int(rng.choice([0, 0, 8, 5, 16])),
                lens_seed=int(rng.integers(1 << 30)))


def _host(t):
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).cpu().numpy().view(np.uint16), oracle.BF16
    return t.cpu().numpy(), oracle.F32


def _check(case, it, probs):
    """(False: not compared, the case is outside the contract.)"""
    cfg, algo = case["cfg"], case["algo"]
    B, gamma, V, T = cfg.B, cfg.gamma, cfg.V, cfg.temperature
    inp = workloads.generate(cfg, seed=1000 + it, device=DEV, top_k_target=case["top_k"], top_k_draft=3 * case["top_k"])
    rows_t, rows_d = inp["target_logits"], inp["draft_logits"]
    if probs:
        rows_t = torch.softmax(rows_t.float() / T, -1).to(rows_t.dtype)
        rows_d = torch.softmax(rows_d.float() / T, -1).to(rows_d.dtype)
        if not bool((torch.gather(rows_d.float(), 2, inp["draft_tokens"].long().unsqueeze(-1)) > 0).all()):
            return False                             # a drafted token's probability rounded to zero: outside the contract
    lens = (np.random.default_rng(case["lens_seed"]).integers(1, gamma + 1, size=B).astype(np.int32)
            if case["use_lens"] else np.full(B, gamma, np.int32))
    tb = torch.full((B, gamma + 1, V + case["pad_t"]), float("nan"), dtype=rows_t.dtype, device=DEV)
    db = torch.full((B, gamma, V + case["pad_d"]), float("nan"), dtype=rows_d.dtype, device=DEV)
    tb[..., :V] = rows_t
    db[..., :V] = rows_d
    for b in range(B):
        tb[b, lens[b] + 1:] = float("nan")
        db[b, lens[b]:] = float("nan")
    dbg = torch.full((B, gamma + 1, 3), float("nan"), dtype=torch.float32, device=DEV)
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    dl = torch.as_tensor(lens, device=DEV) if case["use_lens"] else None
    sv.spec_verify_debug_config(PATHS[case["path"]], -1)
    try:
        for _ in range(2):
            if probs:
                tau, y = sv.spec_verify_probs(algo, tb[..., :V], db[..., :V], inp["draft_tokens"], inp["uniforms"],
                                              draft_lens=dl, debug_out=dbg, workspace=ws)
            else:
                tau, y = sv.spec_verify_ex(algo, tb[..., :V], db[..., :V], inp["draft_tokens"], inp["uniforms"], T,
                                           draft_lens=dl, debug_out=dbg, workspace=ws)
        # the same without the debug block: residual masses that cannot matter are then left out, and the
        # decisions must not change
        if probs:
            tau2, y2 = sv.spec_verify_probs(algo, tb[..., :V], db[..., :V], inp["draft_tokens"], inp["uniforms"],
                                            draft_lens=dl, workspace=ws)
        else:
            tau2, y2 = sv.spec_verify_ex(algo, tb[..., :V], db[..., :V], inp["draft_tokens"], inp["uniforms"], T,
                                         draft_lens=dl, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(tau, tau2) and torch.equal(y, y2), case
    finally:
        sv.spec_verify_debug_config(0, -1)
    assert sv.spec_verify_workspace_check(ws, B, gamma, V) == 0
    tau, y, dbg = tau.cpu().numpy(), y.cpu().numpy(), dbg.cpu().numpy()
    ht, odt = _host(rows_t)
    hd, _ = _host(rows_d)
    tok, uni = inp["draft_tokens"].cpu().numpy(), inp["uniforms"].cpu().numpy()
    for g in np.unique(lens):
        sel = np.nonzero(lens == g)[0]
        args = (parity.ALGOS[algo][0], ht[sel, :g + 1], hd[sel, :g], tok[sel, :g], uni[sel, :g + 1])
        ref = oracle.verify_probs(*args, dtype=odt) if probs else oracle.verify(*args, T, dtype=odt)
        m = ref["margins"]
        tau_bad = tau[sel] != ref["accept_len"]
        y_bad = (y[sel] != ref["next_token"]) & ~tau_bad
        unexcused = (tau_bad & ~(m[:, 0] < parity.MARGIN)) | (y_bad & ~(m[:, 1] < parity.MARGIN))
        assert not unexcused.any(), (case, int(g), sel[unexcused].tolist())
        S, w = ref["dbg"][:, :, 1], ref["dbg"][:, :, 0]
        tol = parity.S_RTOL * S + parity.S_FLOOR * np.maximum(w, 1e-30)
        assert np.all(np.abs(dbg[sel, :g + 1, 1].astype(np.float64) - S) <= tol), (case, int(g))
    return True


@pytest.mark.parametrize("probs", [False, True], ids=["logits", "probs"])
@pytest.mark.parametrize("block", range(4))
def test_random_shapes_and_options(block, probs):
    rng = np.random.default_rng(7000 + 10 * block + (1 if probs else 0))
    for j in range(25):
        it = 100 * block + j
        _check(_draw_case(rng, it, probs), it, probs)


@pytest.mark.parametrize("block", range(2))
def test_weights_from_the_ratios_of_all_positions(block, monkeypatch):
    """The fused kernel with its pruning where every position forms w_i from the earlier positions' ratios itself (calls
    whose positions follow each other faster than a word travels): random shapes, longer drafts among them."""
    monkeypatch.setitem(PATHS, "fused-ratios", 6)
    rng = np.random.default_rng(7900 + block)
    for j in range(20):
        case = _draw_case(rng, 900 + 20 * block + j, False)
        if j % 4 == 0:
            case["cfg"] = workloads.with_overrides(case["cfg"], B=3, gamma=int(rng.choice([16, 33, 64])), V=min(case["cfg"].V, 20000))
        _check(dict(case, path="fused-ratios"), 900 + 20 * block + j, False)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(16, 8, 40000, "bf16"), (40, 16, 9000, "f32"), (300, 4, 20000, "bf16")])
def test_a_wait_for_ratios_that_runs_out_is_reported_not_hung(B, gamma, V, dtype, algo):
    """The same form with a spin limit of zero: every wave that finds a word missing gives up at once, the kernel ends normally,
    a sequence that any of them belongs to reports -1 for both outputs and every other one is complete and right."""
    cfg = workloads.Config(f"out_B{B}_g{gamma}_V{V}", B, gamma, V, dtype, 3.0, 1.0, 1.0, False, 1)
    inp = workloads.generate(cfg, seed=14 + B, device=DEV)
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    ref = parity.run_oracle(algo, inp, 1.0)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    for limit in (0, 3, -1):                                 # (negative: the library's own limit, nothing runs out)
        sv.spec_verify_workspace_init(ws, B, gamma, V)
        sv.spec_verify_debug_config(6, limit)
        try:
            tau, y = parity.ALGOS[algo][1](inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], 1.0, workspace=ws)
            torch.cuda.synchronize()
            status = sv.spec_verify_workspace_check(ws, B, gamma, V)
        finally:
            sv.spec_verify_debug_config(0, -1)
        assert sv.spec_verify_debug_last_chain() == 0
        tau, y = tau.cpu().numpy(), y.cpu().numpy()
        failed = tau < 0
        assert np.array_equal(failed, y < 0)
        assert status in (0, 5) and (status == 5 or not failed.any())
        if limit < 0:
            assert status == 0
        right = safe & ~failed
        assert np.array_equal(tau[right], ref["accept_len"][right]) and np.array_equal(y[right], ref["next_token"][right])


@pytest.mark.parametrize("lens", [False, True])
@pytest.mark.parametrize("gamma,V,dtype", [(8, 9000, "bf16"), (16, 3000, "f32"), (4, 70000, "bf16")])
def test_the_report_changes_neither_the_kernel_nor_the_way_to_w(gamma, V, dtype, lens):
    """Whether the caller asks for every S_i decides about neither (a uniform next to an edge would otherwise fall to one side
    with the report and to the other without): calls from less than one resident set to a dozen."""
    groups, forms = (V + 8191) // 8192, set()
    for sets in (0.7, 1.3, 1.8, 2.2, 2.6, 3.0, 3.5, 4.2, 5.0, 6.0, 7.0, 8.5, 10.0, 12.0):
        B = int(sets * 1280 / (groups * (gamma + 1))) + 1
        rows = torch.zeros((B, gamma + 1, V), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
        tokens = torch.zeros((B, gamma), dtype=torch.int32, device=DEV)
        uniforms = torch.full((B, gamma + 1), 0.5, device=DEV)
        dl = torch.full((B,), gamma, dtype=torch.int32, device=DEV) if lens else None
        ws, seen = sv.alloc_workspace(B, gamma, V, DEV), []
        for dbg in (None, torch.empty((B, gamma + 1, 3), device=DEV)):
            sv.spec_verify_ex("block", rows, rows[:, 1:].contiguous(), tokens, uniforms, 1.0, draft_lens=dl, workspace=ws, debug_out=dbg)
            kernel = sv.spec_verify_debug_last_kernel()
            seen.append((kernel, sv.spec_verify_debug_last_chain() if kernel == sv.binding.SV_KERNEL_FUSED else None))
        assert seen[0] == seen[1], (B, sets)
        forms.add(seen[0])
    assert len(forms) >= (3 if gamma > 4 else 2)             # the kernel for few resident sets, both forms of the fused one (short drafts: the chain)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype,lens", [(40, 16, 20000, "bf16", False), (64, 8, 70001, "bf16", True), (150, 6, 9000, "f32", False),
                                                  (512, 2, 17000, "bf16", False)])
def test_calls_of_a_few_resident_sets_on_the_fused_kernel(algo, B, gamma, V, dtype, lens, monkeypatch):
    """Both ways to w_i as the library picks them (1.6 to 3.6 sets), and the same call on the kernel for few resident sets."""
    monkeypatch.setitem(PATHS, "fused-auto", 2)
    cfg = workloads.Config(f"sets_B{B}_g{gamma}_V{V}", B, gamma, V, dtype, 3.0, 0.7, 0.9, False, 1)
    for path in ("fused-auto", "default"):
        _check(dict(cfg=cfg, algo=algo, path=path, top_k=0, use_lens=lens, pad_t=0, pad_d=0, lens_seed=B), 950 + B, False)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(6, 1, 9000, "bf16"), (7, 5, 20001, "bf16"), (5, 5, 12000, "f32"), (3, 64, 2500, "f32")])
def test_every_token_accepted_without_the_chain(algo, B, gamma, V, dtype):
    """The finisher of a sequence whose last test passes asks no earlier position: its neighbours' do (every other sequence here)."""
    import paper_2403_10444_amd as sv
    cfg = workloads.Config(f"accepted_B{B}_g{gamma}_V{V}", B, gamma, V, dtype, 2.0, 0.6, 0.9, False, 1)
    inp = workloads.generate(cfg, seed=B + V, device="cuda:0")
    inp["uniforms"][::2, :gamma] = 0.0
    sv.spec_verify_debug_config(6, -1)
    try:
        got = parity.run_gpu(algo, inp, cfg.temperature)
        assert sv.spec_verify_debug_last_chain() == 0
    finally:
        sv.spec_verify_debug_config(0, -1)
    assert (got["accept_len"][::2] == gamma).all()
    parity.compare(got, parity.run_oracle(algo, inp, cfg.temperature), label=cfg.name + "/" + algo, greedy=algo == "greedy")


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,sigma,lens", [(30, 8, 50257, 0.5, False), (59, 16, 22739, 0.8, True), (90, 2, 40000, 0.4, False), (150, 1, 40000, 0.4, False)])
def test_more_than_one_set_leaves_out_what_the_next_position_rules_out(algo, B, gamma, V, sigma, lens):
    """The kernel for calls of few resident sets, 1.2 to 2.4 of them, close models: many weights of 1 and passed tests of Alg. 1."""
    cfg = workloads.Config(f"beyond_B{B}_g{gamma}_V{V}", B, gamma, V, "bf16", 3.0, sigma, 0.9, False, 1)
    _check(dict(cfg=cfg, algo=algo, path="default", top_k=0, use_lens=lens, pad_t=0, pad_d=0, lens_seed=B), 970 + B, False)
    assert (sv.spec_verify_debug_last_kernel(), sv.spec_verify_debug_last_together(), sv.spec_verify_debug_last_form()) == (7, 0, (0, 0, 0))
