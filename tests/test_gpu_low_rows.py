"""Rows whose logits all lie far below 0 (log-probabilities at a low temperature, or any logits with a constant taken off):
softmax does not see the constant, and neither may wave chunks that are masked out or lie beyond the row."""
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
# (temperature, what is added to the target's logits, to the draft's): scaled by log2(e) / T, from -58 to -4800
ADDED = [(1.0, -40, 0), (1.0, 0, -60), (1.0, -100, -100), (1.0, 300, -300), (1.0, -1000, 1000), (0.3, -40, -40), (0.3, -1000, -200)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,to_target,to_draft", ADDED)
def test_verification(T, to_target, to_draft, dtype):
    for V, masked in ((300, False), (3000, False), (9000, False), (9000, True), (40001, True)):
        cfg = workloads.Config(f"low_V{V}", 6, 2, V, dtype, 1.0, 0.8, T, False, 1)
        inp = workloads.generate(cfg, seed=V, device=DEV)
        inp["target_logits"] = (inp["target_logits"].float() + to_target).to(inp["target_logits"].dtype)
        inp["draft_logits"] = (inp["draft_logits"].float() + to_draft).to(inp["draft_logits"].dtype)
        if masked:                                                   # whole chunks, in one of the two rows only
            inp["draft_logits"][..., V // 2:] = -float("inf")
            inp["target_logits"][3:, :, : V // 3] = -float("inf")
        q = torch.softmax(inp["draft_logits"].double() / T, -1)
        inp["draft_tokens"] = torch.multinomial(q.view(-1, V), 1).view(cfg.B, cfg.gamma).to(torch.int32)
        for algo in ("block", "token", "greedy"):
            ref = parity.run_oracle(algo, inp, T)
            for path in (0, 1, 3, 4, 6, 8, 9):
                sv.spec_verify_debug_config(path, -1)
                try:
                    parity.compare(parity.run_gpu(algo, inp, T), ref, label=f"{to_target}/{to_draft}/T{T}/V{V}/{algo}/path{path}", greedy=algo == "greedy")
                finally:
                    sv.spec_verify_debug_config(0, -1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,added", [(1.0, -100), (1.0, -300), (0.3, -1000)])
def test_drafting(T, added, dtype):
    rows = 12
    for V in (20, 300, 1500, 3000, 9001, 60000):
        g = torch.Generator(device=DEV).manual_seed(V)
        x = (torch.randn((rows, V), generator=g, device=DEV) * 2.0 + added).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        x[6:, V // 2 + 1:] = -float("inf")
        u = workloads.philox_uniforms(V, (rows,))
        want, margins = oracle.sample_rows(workloads.logits_to_numpy(x), u, T, dtype=oracle.BF16 if dtype == "bf16" else oracle.F32)
        safe = margins >= parity.MARGIN
        assert safe.sum() >= 0.75 * rows
        ud = torch.as_tensor(u, device=DEV)
        side = torch.cuda.Stream().cuda_stream
        torch.cuda.synchronize()
        for stream in (None, side):
            got = sv.spec_sample_tokens(x, ud, T, tokens=torch.empty((rows,), dtype=torch.int32, device=DEV), stream=stream)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy()[safe], want[safe]), (V, stream)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_tokens_stay_inside_the_vocabulary_beyond_the_range_of_logits(dtype):
    # (a row's largest scaled logit beyond 2^31: its exponentials overflow, what is accepted is not defined)
    for V in (300, 2500, 5000, 50257):
        cfg = workloads.Config(f"beyond_V{V}", 12, 4, V, dtype, 1.0, 0.5, 1.0, False, 1)
        inp = workloads.generate(cfg, seed=V, device=DEV)
        inp["target_logits"][::2, :, 3] = 1e10
        inp["draft_logits"][::3, :, 5] = 1e10
        for algo in ("block", "token", "greedy"):
            for path in (0, 1, 3, 4, 6, 8, 9):
                sv.spec_verify_debug_config(path, -1)
                try:
                    tau, y = parity.ALGOS[algo][1](inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], 1.0)
                    torch.cuda.synchronize()
                finally:
                    sv.spec_verify_debug_config(0, -1)
                assert 0 <= int(tau.min()) and int(tau.max()) <= cfg.gamma, (V, algo, path)
                assert 0 <= int(y.min()) and int(y.max()) < V, (V, algo, path)
