"""Rows at any address: vocabularies that are no multiple of a sixteen-byte vector (and shorter than one), row strides and
base addresses at every offset of the element type.  The values are the same ones the oracle gets; everything around the
rows is NaN."""
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


def _placed(t, offset, pad):
    """The values of `t` [B, R, V] at rows V + pad elements apart, `offset` elements into a buffer of NaNs."""
    B, R, V = t.shape
    buf = torch.full((offset + B * R * (V + pad) + 16,), float("nan"), dtype=t.dtype, device=t.device)
    view = buf[offset:].as_strided((B, R, V), (R * (V + pad), V + pad, 1), offset)
    view.copy_(t)
    return view


# (V: below, at and around a vector of 4 / 8 logits, a wave chunk of 2048, a workgroup chunk of 8192)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [2, 3, 5, 7, 8, 9, 12, 2047, 2049, 2056, 8191, 8193, 10245])
def test_rows_at_any_address(V, dtype):
    cfg = workloads.Config("rows", 3, 3, V, dtype, 2.0, 0.8, 0.9, False, 1)
    inp = workloads.generate(cfg, seed=V, device=DEV)
    T, size = cfg.temperature, 4 if dtype == "f32" else 2
    probs = {k: torch.softmax(inp[k].float() / T, -1).to(inp[k].dtype) for k in ("target_logits", "draft_logits")}
    for n, (offset, pad) in enumerate([(0, 0), (1, 0), (16 // size - 1, 1), (0, -V % 8), (3, 5)]):
        algo = ("block", "token", "greedy")[n % 3]
        ref = parity.run_oracle(algo, inp, T)
        dbg = torch.full((cfg.B, cfg.gamma + 1, 3), float("nan"), dtype=torch.float32, device=DEV)
        t, d = _placed(inp["target_logits"], offset, pad), _placed(inp["draft_logits"], offset, pad)
        for path in (0, 1, 3, 8, 9):
            sv.spec_verify_debug_config(path, -1)
            try:
                tau, y = sv.spec_verify_ex(algo, t, d, inp["draft_tokens"], inp["uniforms"], T, debug_out=dbg)
            finally:
                sv.spec_verify_debug_config(0, -1)
            got = {"accept_len": tau.cpu().numpy(), "next_token": y.cpu().numpy(), "dbg": dbg.cpu().numpy()}
            parity.compare(got, ref, label=f"V{V}/{dtype}/offset{offset}/pad{pad}/path{path}", greedy=algo == "greedy")
        tau, y = sv.spec_verify_probs(algo, _placed(probs["target_logits"], offset, pad), _placed(probs["draft_logits"], offset, pad),
                                      inp["draft_tokens"], inp["uniforms"], debug_out=dbg)
        host = [workloads.logits_to_numpy(probs[k]) for k in ("target_logits", "draft_logits")]
        ref = oracle.verify_probs(parity.ALGOS[algo][0], *host, inp["draft_tokens"].cpu().numpy(), inp["uniforms"].cpu().numpy(),
                                  dtype=oracle.F32 if dtype == "f32" else oracle.BF16)
        bad = (tau.cpu().numpy() != ref["accept_len"]) | (y.cpu().numpy() != ref["next_token"])
        assert not np.any(bad & (ref["margins"].min(axis=1) >= parity.MARGIN)), (V, dtype, offset, pad)


# (the large kernel's draw takes a row's shares of the residual 64 at a time, and keeps the first 128: rows of 64 and 65, 128 and 129 wave
# chunks - they come in fours - and of more, of 2048 logits and of 4096)
@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("dtype,path,chunk", [("bf16", 3, 2048), ("f32", 3, 2048), ("bf16", 4, 4096)])
@pytest.mark.parametrize("chunks", [64, 68, 128, 132, 196])
def test_rows_of_many_shares(chunks, dtype, path, chunk, algo):
    for less, seed in ((0, 1), (4 * chunk - 3, 2)):                          # a last workgroup that is full, and one of three logits
        cfg = workloads.Config("shares", 3, 2, chunks * chunk - less, dtype, 2.0, 0.8 if seed == 1 else 3.0, 0.9, False, 1)
        inp = workloads.generate(cfg, seed=chunks + seed, device=DEV)
        sv.spec_verify_debug_config(path, -1)
        try:
            got = parity.run_gpu(algo, inp, cfg.temperature)
        finally:
            sv.spec_verify_debug_config(0, -1)
        parity.compare(got, parity.run_oracle(algo, inp, cfg.temperature), label=f"{cfg.V}/{dtype}/{algo}", greedy=algo == "greedy")
