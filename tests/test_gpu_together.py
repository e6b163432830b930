"""The kernel for calls whose workgroups all run at once (every workgroup forms the ratios of all earlier rows itself) against the CPU
oracle, at the edges of its forms: rows of 4 / 5, 16 / 17 and 32 workgroups, drafts of one row more than its waves take in one pass and
of 64 tokens, and in turns with the kernels it shares a workspace with."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2403_10444_amd as sv
from paper_2403_10444_amd import binding
import workloads
from tests import parity

pytestmark = pytest.mark.gpu
DEV = "cuda"
CHUNK = 8192                 # logits of a row per workgroup


def _cfg(B, gamma, V, dtype, sigma_d=0.8, T=0.9):
    return workloads.Config(f"together_B{B}_g{gamma}_V{V}_{dtype}", B, gamma, V, dtype, 2.5, sigma_d, T, False, 1)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [
    (5, 3, 4 * CHUNK, "bf16"), (5, 3, 4 * CHUNK + 1, "f32"),                 # four workgroups and five: segments of 4 and 16 lanes
    (2, 5, 16 * CHUNK, "bf16"), (2, 5, 16 * CHUNK + 8, "bf16"),              # sixteen and seventeen: one and two words per lane
    (1, 8, 32 * CHUNK - 3, "f32"), (1, 4, 25 * CHUNK, "bf16"),
    (2, 16, 5 * CHUNK, "bf16"), (2, 17, 5 * CHUNK - 100, "f32"),             # sixteen rows to a pass
    (1, 64, 6 * CHUNK, "bf16"), (3, 64, 3001, "f32"), (1, 63, CHUNK + 1, "bf16"),
    (40, 4, 4 * CHUNK, "bf16"), (57, 8, 2 * CHUNK, "bf16"),                  # 800; 1026 workgroups: the last target rows come late
])
def test_forms(B, gamma, V, dtype, algo):
    cfg = _cfg(B, gamma, V, dtype)
    for seed, sigma_d in ((1, 0.8), (2, 0.05)):                              # (close models: most tokens are accepted)
        inp = workloads.generate(workloads.with_overrides(cfg, sigma_draft=sigma_d), seed=seed + gamma + V, device=DEV)
        got = parity.run_gpu(algo, inp, cfg.temperature)
        assert sv.spec_verify_debug_last_kernel() == binding.SV_KERNEL_RESIDENT and sv.spec_verify_debug_last_together() == 1
        parity.compare(got, parity.run_oracle(algo, inp, cfg.temperature), label=f"{cfg.name}/{algo}", greedy=algo == "greedy")


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
def test_equal_models_and_own_draft_lengths(algo):
    """q = p: no residual has any mass beyond rounding, everything is accepted or drawn from p."""
    cfg = _cfg(6, 9, 3 * CHUNK - 5, "bf16")
    inp = workloads.generate(cfg, seed=5, device=DEV)
    inp["draft_logits"] = inp["target_logits"][:, :-1].clone()
    lens = torch.tensor([1, 2, 5, 8, 9, 9], dtype=torch.int32, device=DEV)
    tau, y = sv.spec_verify_ex(algo, inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], cfg.temperature, draft_lens=lens)
    torch.cuda.synchronize()
    assert torch.equal(tau, lens)
    p = torch.softmax(inp["target_logits"].double() / cfg.temperature, -1).cpu().numpy()
    for b in range(cfg.B):
        g = int(lens[b])
        assert parity.in_cell(p[b, g], float(inp["uniforms"][b, g]), int(y[b]))


def test_in_turns_with_the_other_kernels_on_one_workspace():
    """Its three copies of the words lie where the large kernel keeps others: calls of all kernels follow each other on one
    workspace, drafts of the sequences' own lengths among them."""
    B, gamma, V = 24, 7, 30001                                               # (768 workgroups)
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    for n, path in enumerate([0, 0, 3, 0, 4, 0, 6, 4, 0, 0, 3, 4, 0, 9, 0, 9, 9, 3, 0, 9]):
        cfg = _cfg(B, gamma, V, "f32" if n % 3 == 2 else "bf16")
        inp = workloads.generate(cfg, seed=100 + n, device=DEV)
        sv.spec_verify_debug_config(path, -1)
        try:
            got = parity.run_gpu("block", inp, cfg.temperature, workspace=ws)
            lens = torch.tensor([1 + (b + n) % gamma for b in range(B)], dtype=torch.int32, device=DEV)
            own = sv.spec_verify_ex("greedy", inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], cfg.temperature,
                                    draft_lens=lens, workspace=ws)
        finally:
            sv.spec_verify_debug_config(0, -1)
        fresh = sv.spec_verify_ex("greedy", inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], cfg.temperature, draft_lens=lens)
        torch.cuda.synchronize()
        ref = parity.run_oracle("block", inp, cfg.temperature)
        parity.compare(got, ref, label=f"turn{n}/path{path}")
        assert (np.array([int((a != b).sum()) for a, b in zip(own, fresh)]) <= (0 if path == 0 else 1)).all()
        assert binding.spec_verify_workspace_check(ws, B, gamma, V) == binding.SV_OK


# Both sides of the lines between this kernel and the other one for calls of few resident sets (runs_together): what calls of 1024 resident workgroups
# are, by type, draft length and row width.
@pytest.mark.parametrize("B,gamma,V,dtype,together", [
    (1, 8, 140000, "bf16", 1), (1, 9, 140000, "bf16", 0), (1, 8, 140000, "f32", 1), (1, 9, 140000, "f32", 0),        # 18 workgroups a row: drafts of up to 8
    (8, 6, 140000, "bf16", 1), (9, 6, 140000, "bf16", 0), (11, 4, 140000, "bf16", 1), (13, 4, 140000, "bf16", 0),    # 1008, 1134; 990, 1170
    (8, 16, 40961, "f32", 1), (9, 16, 40961, "f32", 0), (11, 12, 40961, "f32", 1),                                    # 816, 918; drafts of up to 12: 858
    (32, 8, 30001, "bf16", 1), (33, 8, 30001, "bf16", 0), (64, 3, 30001, "bf16", 1), (65, 3, 30001, "bf16", 0),      # 1152, 1188; drafts of three 1024, 1040
    (70, 8, 16000, "f32", 1)])                                                                                        # 1260: float32 has no such line
def test_both_sides_of_its_lines(B, gamma, V, dtype, together):
    cfg = _cfg(B, gamma, V, dtype)
    inp = workloads.generate(cfg, seed=B + gamma, device=DEV)
    algo = ("block", "token", "greedy")[(B + gamma) % 3]
    got = parity.run_gpu(algo, inp, cfg.temperature)
    assert sv.spec_verify_debug_last_kernel() == binding.SV_KERNEL_RESIDENT and sv.spec_verify_debug_last_together() == together
    parity.compare(got, parity.run_oracle(algo, inp, cfg.temperature), label=f"{cfg.name}/{algo}", greedy=algo == "greedy")
