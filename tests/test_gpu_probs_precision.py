"""Probabilities: what the float32 outputs show of the weights' precision.  A weight is kept in 48 bits so that a residual far smaller than the
probabilities it is left of keeps its relative accuracy: rows in which w p - q is 2^-36 of p, against exact rational arithmetic."""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
import pytest
import torch

import paper_2403_10444_amd as sv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _nearly_cancelling(rng):
    """24-bit integers a < b, c, d with a c - b d = k, k some 2^-36 (at least 2^-37) of a c."""
    while True:
        a, b = sorted(int(v) for v in rng.integers(1 << 23, 1 << 24, 2))
        k = int(rng.integers(1 << 11, 1 << 12))
        if a == b or math.gcd(a, b) != 1:
            continue
        c = k * pow(a, -1, b) % b
        if c < 1 << 23:
            continue
        d = (a * c - k) // b
        if d >= 1 << 23:
            return a, b, c, d


# (several sequences to a workgroup, one, the kernels for wider rows in one launch and in two, and with the weights from a kernel in front)
@pytest.mark.parametrize("large_ratio", [False, True])
@pytest.mark.parametrize("algo", ["block", "greedy"])
@pytest.mark.parametrize("B,gamma,V", [(64, 3, 7), (64, 20, 31), (64, 3, 300), (64, 5, 2000), (64, 3, 2500), (500, 4, 2500), (1001, 4, 2500), (300, 8, 9000)])
def test_a_residual_far_below_its_row(B, gamma, V, algo, large_ratio):
    """w = a / b, and at one token w c - d with a c - b d = k: S is k / b (in units of 2^-24).  `large_ratio`: ratios of 2^60 come before, whose
    weight is 1 (Alg. 2) - what they leave in sums of logarithms must not blur a / b.
    Bound: w is rounded to 2^-49 (two floats), its logarithm and power to 2^-51; fma(w_hi, p, -q) to 2^-24 of a value below 2^-23 of p:
    2^-47 of p in all, 2^-10 of a residual of 2^-37 of p; the sum's own rounding is far below that."""
    if large_ratio and algo == "greedy":
        pytest.skip("Alg. 4 keeps the large weight")
    rng = np.random.default_rng(B + V)
    at = gamma - 1                                                  # the row pair whose residual is looked at
    P = torch.full((B, gamma + 1, V), 2.0 ** -10)
    Q = torch.full((B, gamma, V), 2.0 ** -10)
    tok = torch.from_numpy(rng.integers(0, V, (B, gamma)).astype(np.int32))
    want = np.empty(B)
    for b in range(B):
        a, bb, c, d = _nearly_cancelling(rng)
        if large_ratio:
            for i in range(at - 1):
                P[b, i, tok[b, i]], Q[b, i, tok[b, i]] = 2.0 ** -2, 2.0 ** -62
        P[b, at - 1, tok[b, at - 1]], Q[b, at - 1, tok[b, at - 1]] = a * 2.0 ** -24, bb * 2.0 ** -24
        x = int(rng.integers(0, V))
        P[b, at], Q[b, at] = 0.0, 2.0 ** -10
        P[b, at, x], Q[b, at, x] = c * 2.0 ** -24, d * 2.0 ** -24
        want[b] = float(Fraction(a * c - bb * d, bb) / (1 << 24))
    dbg = torch.zeros((B, gamma + 1, 3), device=DEV)
    sv.spec_verify_probs(algo, P.to(DEV), Q.to(DEV), tok.to(DEV), torch.full((B, gamma + 1), 0.5, device=DEV), debug_out=dbg)
    got = dbg[:, at, 1].double().cpu().numpy()
    assert np.all(np.abs(got - want) <= 2.0 ** -10 * want), float(np.max(np.abs(got - want) / want))


# (32 probabilities of a row per lane, 16, 8)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,gamma,V", [(3, 4, 2048), (800, 3, 1024), (2, 40, 500), (2, 64, 128), (4, 12, 1000), (3, 20, 500), (4, 2, 500)])
def test_sums_of_short_rows(B, gamma, V, dtype):
    """One large probability in front of every lane's share of a row, all others half a unit of its last place: a float chain loses each of them, sums of at most
    eight terms at most seven.  Bound: seven roundings of 2^-24, one of the reported float."""
    vec = 4 if dtype == torch.float32 else 8
    P = torch.full((B, gamma + 1, V), 2.0 ** -24, dtype=dtype)
    lanes = V // 32 if V > 128 else 4
    P[..., :lanes * vec:vec] = 1.0
    Q = torch.zeros((B, gamma, V), dtype=dtype)
    Q[..., 0] = 1.0
    P[..., 0] = 1.0
    want = P[:, :gamma].double().sum(-1) - 1.0                      # (w = 1; token 0 is in both rows)
    args = P.to(DEV), Q.to(DEV), torch.zeros((B, gamma), dtype=torch.int32, device=DEV), torch.full((B, gamma + 1), 0.5, device=DEV)
    for algo in ("block", "token", "greedy"):
        dbg = torch.zeros((B, gamma + 1, 3), device=DEV)
        sv.spec_verify_probs(algo, *args, debug_out=dbg)
        assert sv.spec_verify_debug_last_form()[0] == sv.binding.SV_FORM_SEQUENCES
        got = dbg[:, :gamma, 1].double().cpu()
        assert bool(((got - want).abs() <= 8 * 2.0 ** -24 * want).all()), float(((got - want).abs() / want).max())


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V", [(6, 5, 8), (6, 17, 8), (6, 5, 30), (6, 5, 100), (6, 5, 200), (6, 20, 300), (6, 5, 500), (6, 5, 900), (6, 5, 2000)])
def test_tokens_that_one_row_rules_out(B, gamma, V, algo):
    """Drafted tokens with q = 0 (no draft has them: r is infinite, a weight of 1 in Alg. 2, an infinite one in Alg. 4), with p = 0 behind them, and both: the same whatever
    the row's width is - the rows with as many tokens of probability 0 behind them as the kernels for wider rows want."""
    gen = torch.Generator().manual_seed(V + gamma)
    P, Q = (torch.softmax(2.0 * torch.randn((B, n, V), generator=gen), -1) for n in (gamma + 1, gamma))
    tok = torch.multinomial(Q.view(-1, V), 1, generator=gen).view(B, gamma).to(torch.int32)
    uni = torch.randint(0, 1 << 24, (B, gamma + 1), generator=gen) * 2.0 ** -24
    for b, (no_q, no_p) in enumerate([((0,), ()), ((0,), (1,)), ((1,), (2,)), ((1, 2), (0, 3)), ((), (2,)), ((2,), (2,))]):
        for i in no_q:
            Q[b, i, tok[b, i]] = 0.0
        for i in no_p:
            P[b, i, tok[b, i]] = 0.0
    out = []
    for width in (V, 2500):
        p, q = torch.zeros((B, gamma + 1, width)), torch.zeros((B, gamma, width))
        p[..., :V], q[..., :V] = P, Q
        dbg = torch.zeros((B, gamma + 1, 3), device=DEV)
        tau, y = sv.spec_verify_probs(algo, p.to(DEV), q.to(DEV), tok.to(DEV), uni.to(DEV), debug_out=dbg)
        assert (sv.spec_verify_debug_last_form()[0] == sv.binding.SV_FORM_SEQUENCES) == (width == V)
        out.append((tau.cpu().numpy(), y.cpu().numpy(), dbg.cpu().numpy()))
    (tau, y, dbg), (tau_wide, y_wide, dbg_wide) = out
    assert np.array_equal(tau, tau_wide) and np.array_equal(y, y_wide)
    # (float sums of other chunks: some 2^-21 each; a difference of infinities is one in both)
    assert np.allclose(dbg, dbg_wide, rtol=1e-6, atol=1e-9, equal_nan=True)
    if algo == "greedy":
        assert np.all(np.isinf(dbg[1, 1:, 0]))                     # an infinite ratio in front of one of 0
