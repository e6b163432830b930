"""Comparison of the HIP path with the CPU oracle on the same seeded inputs."""
from __future__ import annotations

import numpy as np
import torch

import oracle
import paper_2403_10444_amd as sv
import workloads

# Accept lengths and tokens must be bit-exact unless a uniform lies this close to a decision
# boundary (|eta_i - h_i| for the tests that fixed tau; distance of u*total to the edge of the
# chosen token's CDF cell, relative to the total).
MARGIN = 1e-6
# Residual masses: 1e-5 relative, plus a floor proportional to w_i for the rows where S_i is a small difference of
# large numbers (S_i << w_i: w_i p_i and q_i nearly agree on the tokens that carry the mass).  There fp32 cannot give
# 1e-5 of S_i: the row's two normalisers and w_i itself come out of fp32 sums of hardware exp2 values and are good to
# about 1e-7 relative each, and an error of that size in w_i or a normaliser moves S_i by that fraction of the whole
# active mass (<= w_i), whatever S_i is.  Measured over the five configurations: |dS| <= 4.5e-7 w_i, 99 % of rows below
# 1.8e-7 w_i.  Every comparison counts the rows that are outside 1e-5 relative (and so pass by the floor only); the
# counts per configuration are written out at the end of a test session (see record()).
S_RTOL = 1e-5
S_FLOOR = 6e-7
# ... and their share is bounded: of a comparison's rows (where there are at least 200) at most this fraction may lie
# outside 1e-5 relative (measured over the five configurations: at most 2.4 % on the fused kernel, 3.0 % on the staged one)
S_OUTSIDE_MAX = 0.05

# reports of this session's comparisons, for the per-configuration summaries
RECORDS = []


def record(report):
    """Keeps a comparison's report for the summaries that tests/conftest.py writes when the session ends."""
    RECORDS.append(dict(report))
    return report


ALGOS = {"block": (oracle.BLOCK, sv.spec_verify_block),
         "token": (oracle.TOKEN, sv.spec_verify_token),
         "greedy": (oracle.GREEDY, sv.spec_verify_greedy)}


def in_cell(weights, u, y):
    """Whether token y can be the draw at uniform u from these weights (float64): it has weight, and u lies in its cell of the
    normalised running sum or within MARGIN of it.  Decides about the uniforms next to an edge that `margins` excuses."""
    c = np.cumsum(weights, dtype=np.float64)
    below = c[y - 1] if y > 0 else 0.0
    return bool(weights[y] > 0) and below / c[-1] - MARGIN <= u <= c[y] / c[-1] + MARGIN


def run_gpu(algo, inputs, temperature, workspace=None):
    B, g1, V = inputs["target_logits"].shape
    dbg = torch.full((B, g1, 3), float("nan"), dtype=torch.float32, device=inputs["target_logits"].device)
    tau, y = ALGOS[algo][1](inputs["target_logits"], inputs["draft_logits"], inputs["draft_tokens"],
                            inputs["uniforms"], temperature, debug_out=dbg, workspace=workspace)
    # without the debug block the kernels leave out the residual masses that cannot matter (positions whose test
    # fails whatever S_i is): the decisions must be the same, bit for bit
    tau2, y2 = ALGOS[algo][1](inputs["target_logits"], inputs["draft_logits"], inputs["draft_tokens"],
                              inputs["uniforms"], temperature, workspace=workspace)
    torch.cuda.synchronize()
    assert torch.equal(tau, tau2) and torch.equal(y, y2), "results differ with and without the debug block"
    return {"accept_len": tau.cpu().numpy(), "next_token": y.cpu().numpy(), "dbg": dbg.cpu().numpy()}


def run_oracle(algo, inputs, temperature, rows=None, nthreads=0):
    """Oracle on all sequences, or on the subset `rows` (a list / array of sequence indices)."""
    if rows is not None:
        idx = torch.as_tensor(np.asarray(rows), device=inputs["target_logits"].device)
        inputs = {k: v.index_select(0, idx) for k, v in inputs.items()}
    host = workloads.to_numpy(inputs)
    dtype = oracle.BF16 if host["target_logits"].dtype == np.uint16 else oracle.F32
    return oracle.verify(ALGOS[algo][0], host["target_logits"], host["draft_logits"], host["draft_tokens"],
                         host["uniforms"], temperature, dtype=dtype, nthreads=nthreads)


def compare(gpu, ref, rows=None, label="", greedy=False):
    """Element-by-element comparison; returns a report dict and raises on a violation.

    `greedy`: h_i of greedy block verification is a ratio of two residual masses; where both are
    rounding noise (the two models agree on the row) it is 0/0 and is not compared."""
    g_tau, g_y, g_dbg = gpu["accept_len"], gpu["next_token"], gpu["dbg"]
    if rows is not None:
        rows = np.asarray(rows)
        g_tau, g_y, g_dbg = g_tau[rows], g_y[rows], g_dbg[rows]
    r_tau, r_y, r_dbg, marg = ref["accept_len"], ref["next_token"], ref["dbg"], ref["margins"]
    n = len(r_tau)
    tau_bad = g_tau != r_tau
    y_bad = (g_y != r_y) & ~tau_bad
    # a tau mismatch is excused by a uniform within MARGIN of its h; a Y mismatch (same tau)
    # by u within MARGIN of a CDF boundary
    excused = (tau_bad & (marg[:, 0] < MARGIN)) | (y_bad & (marg[:, 1] < MARGIN))
    unexcused = (tau_bad | y_bad) & ~excused
    w, S, h = r_dbg[..., 0], r_dbg[..., 1], r_dbg[..., 2]
    gw, gS, gh = g_dbg[..., 0].astype(np.float64), g_dbg[..., 1].astype(np.float64), g_dbg[..., 2].astype(np.float64)
    s_err = np.abs(gS - S)
    s_tol = S_RTOL * S + S_FLOOR * np.maximum(w, 1e-30)
    s_rel = s_err / np.maximum(S, 1e-300)
    # h_i = S_i / (S_i + 1 - w_i) is ill-conditioned where S_i and 1 - w_i are both small: its tolerance is 2e-5 plus
    # what the tolerance of S_i and an error of 5e-6 w_i in w_i can move it by (rows with w_i < 1 only; h_i = 1 otherwise,
    # and Alg. 1's h_i = min(r_i, 1) has w_i = 1 throughout)
    u = np.maximum(1.0 - w, 0.0)
    with np.errstate(invalid="ignore", over="ignore", divide="ignore"):
        h_tol = 2e-5 + np.where(u > 0, (u * s_tol + S * 5e-6 * w) / np.maximum(S + u, 1e-300) ** 2, 0.0)
    s_rows = S > 0            # (row gamma, where S = w, included)
    report = {
        "label": label, "n": int(n),
        "tau_mismatch": int(tau_bad.sum()), "y_mismatch": int(y_bad.sum()),
        "excused": int(excused.sum()), "unexcused": int(unexcused.sum()),
        "max_S_rel_err": float(np.max(np.where(S > 1e-12, s_rel, 0.0))),
        "frac_S_within_1e-5_rel": float(np.mean(s_rel[S > 0] <= S_RTOL)) if np.any(S > 0) else 1.0,
        "S_rows": int(s_rows.sum()),
        "S_rows_outside_1e-5_rel": int((s_rel[s_rows] > S_RTOL).sum()),
        # (positions below gamma: at gamma S is w itself)
        "max_dS_over_w": float(np.max((s_err / np.maximum(w, 1e-300))[:, :-1], initial=0.0, where=(w > 1e-30)[:, :-1])),
        # w below float32's normal range cannot be reported in the float32 debug block
        "max_w_rel_err": float(np.max(np.where(w > 1e-30, np.abs(gw - w) / np.maximum(w, 1e-300), 0.0))),
        "max_h_abs_err": float(np.max(np.where(greedy & (S < 1e-12), 0.0, np.abs(gh - h)))),
        "max_h_err_over_tol": float(np.max(np.where(greedy & (S < 1e-12), 0.0, np.abs(gh - h) / h_tol))),
        "mean_tau": float(np.mean(g_tau)),
        "n_fallback_oracle": int(ref["n_fallback"]),
    }
    assert report["unexcused"] == 0, f"unexcused (tau, Y) mismatches: {report}"
    assert np.all((g_tau >= 0) & (g_tau <= r_dbg.shape[1] - 1)), report
    assert np.all(s_err <= s_tol), f"residual mass out of tolerance: {report}"
    assert report["S_rows"] < 200 or report["S_rows_outside_1e-5_rel"] <= S_OUTSIDE_MAX * report["S_rows"], \
        f"too many residual masses outside 1e-5 relative: {report}"
    assert report["max_w_rel_err"] <= 2e-5, report
    assert report["max_h_err_over_tol"] <= 1.0, report
    return report
