"""Logits masked out with large negative numbers instead of -inf (-1e9, -1e10, half of or the whole lowest value of the type, at
temperatures that scale them differently): whole wave and workgroup chunks of a row then hold nothing else."""
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
MASKS = [(0.3, -1e9), (1.0, -1e9), (1.0, -1e10), (1.0, -1e20), (1.0, "half"), (1.0, "lowest"), (2.0, "lowest"), (0.3, "lowest")]


def _mask(dtype, value):
    lowest = torch.finfo(torch.bfloat16 if dtype == "bf16" else torch.float32).min
    return {"half": lowest / 2, "lowest": lowest}.get(value, value)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,value", MASKS)
def test_verification(T, value, dtype):
    low = _mask(dtype, value)
    for V in (1000, 3000, 9000, 40001):
        cfg = workloads.Config(f"masked_V{V}", 6, 2, V, dtype, 2.5, 0.8, T, False, 1)
        inp = workloads.generate(cfg, seed=V, device=DEV)
        keep = torch.arange(V, device=DEV) < V // 3
        inp["draft_logits"][3:, :, ~keep] = low                      # (the first sequences' drafts may come from what the target masks)
        inp["target_logits"][..., ~keep] = low
        q = torch.softmax(inp["draft_logits"].double() / T, -1)
        inp["draft_tokens"] = torch.multinomial(q.view(-1, V), 1).view(cfg.B, cfg.gamma).to(torch.int32)
        for algo in ("block", "token", "greedy"):
            ref = parity.run_oracle(algo, inp, T)
            for path in (0, 1, 3, 4, 6, 8, 9):
                sv.spec_verify_debug_config(path, -1)
                try:
                    parity.compare(parity.run_gpu(algo, inp, T), ref, label=f"{value}/T{T}/V{V}/{algo}/path{path}", greedy=algo == "greedy")
                finally:
                    sv.spec_verify_debug_config(0, -1)


# Rows that share a workgroup with others, and rows that have one each (which take calls of more sequences): lanes, waves and half workgroups that hold
# nothing but masked logits
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,value", MASKS)
def test_short_rows_and_rows_of_one_workgroup(T, value, dtype):
    low = _mask(dtype, value)
    for B, gamma, V, form in [(9, 3, 7, sv.binding.SV_FORM_SEQUENCES), (600, 2, 30, sv.binding.SV_FORM_SEQUENCES), (1030, 2, 100, sv.binding.SV_FORM_SEQUENCES),
                              (30, 3, 200, sv.binding.SV_FORM_SEQUENCES), (6, 17, 500, sv.binding.SV_FORM_SEQUENCES), (110, 2, 3000, sv.binding.SV_FORM_ROW),
                              (210, 2, 9000, sv.binding.SV_FORM_ROW), (210, 2, 17000, sv.binding.SV_FORM_ROW)]:
        cfg = workloads.Config(f"masked_short_V{V}", B, gamma, V, dtype, 2.5, 0.8, T, False, 1)
        inp = workloads.generate(cfg, seed=V, device=DEV)
        keep = torch.arange(V, device=DEV) % (V // 2) < V // 6 + 1
        inp["draft_logits"][B // 2:, :, ~keep] = low                 # (the first sequences' drafts may come from what the target masks)
        inp["target_logits"][..., ~keep] = low
        q = torch.softmax(inp["draft_logits"].double() / T, -1)
        gen = torch.Generator(device=DEV).manual_seed(V)
        inp["draft_tokens"] = torch.multinomial(q.view(-1, V), 1, generator=gen).view(B, gamma).to(torch.int32)
        some = sorted({0, B // 2 - 1, B // 2, B - 1, *range(0, B, B // 40 + 1)})
        for algo in ("block", "token", "greedy"):
            got = parity.run_gpu(algo, inp, T)
            assert sv.spec_verify_debug_last_form()[0] == form
            parity.compare(got, parity.run_oracle(algo, inp, T, rows=some), rows=some, label=f"{value}/T{T}/V{V}/{algo}", greedy=algo == "greedy")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,value", MASKS)
def test_drafting(T, value, dtype):
    low, rows = _mask(dtype, value), 12
    for V in (20, 300, 1500, 3000, 9001, 60000):
        g = torch.Generator(device=DEV).manual_seed(V)
        x = (torch.randn((rows, V), generator=g, device=DEV) * 3.0).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        x[:4, V // 2 + 1:] = low
        x[4:8, : V // 2] = low
        x[8:, : V // 3] = low
        x[8:, 2 * V // 3 + 1:] = low
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
