"""Calls of more than 2^32 threads: HIP runs such a launch's count modulo 2^32 and reports nothing, so the library cuts
them into several.  Rows are so simple that every result is known exactly (equal logits, or two tokens whose ratio of
probabilities is 1 / 2), and uniforms differ from row to row, so that a misplaced slice shows too."""
from __future__ import annotations

import pytest
import torch

import paper_2403_10444_amd as sv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(autouse=True)
def room():
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GiB of device memory")
    yield
    sv.spec_verify_debug_config(0, -1)
    torch.cuda.empty_cache()


def test_rows_to_draw_from():
    rows, V = (1 << 24) + 3, 2049                  # 256 threads per row
    logits = torch.zeros((rows, V), dtype=torch.bfloat16, device=DEV)
    u = (torch.arange(rows, device=DEV) % 61).float() / 64.0
    tokens = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    sv.spec_sample_tokens(logits, u, 1.0, tokens=tokens)
    assert torch.equal(tokens.long(), (u.double() * V).floor().long())


@pytest.mark.parametrize("path", ["default", "staged", "probs"])
def test_token_verification_of_two_tokens(path):
    # 2^24 chunks of rows and more; p = (1/4, 3/4), q = (1/2, 1/2), the drafted token is 0: a test passes below 1/2
    B, gamma, V = (1 << 20) + 77, 16, 2
    logits = path != "probs"
    p = torch.tensor([0.25, 0.75], device=DEV)
    target = (p.log() if logits else p).expand(B, gamma + 1, V).contiguous()
    draft = torch.full((B, gamma, V), 0.0 if logits else 0.5, device=DEV)
    drafted = torch.zeros((B, gamma), dtype=torch.int32, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(3)
    u = torch.randint(0, 16, (B, gamma + 1), generator=gen, device=DEV).float() / 16.0 + 1.0 / 32.0
    tau = torch.full((B,), -7, dtype=torch.int32, device=DEV)
    y = torch.full((B,), -7, dtype=torch.int32, device=DEV)
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    sv.spec_verify_debug_config(1 if path == "staged" else 0, -1)
    if logits:
        sv.spec_verify_token(target, draft, drafted, u, 1.0, workspace=ws, accept_len=tau, next_token=y)
    else:
        sv.spec_verify_probs("token", target, draft, drafted, u, workspace=ws, accept_len=tau, next_token=y)
    want = torch.cumprod((u[:, :gamma] < 0.5).int(), 1).sum(1).int()
    assert torch.equal(tau, want)
    # a residual of p - q holds token 1 only; after a whole draft p itself is drawn from
    assert torch.equal(y, torch.where(want == gamma, (u[:, gamma] >= 0.25).int(), 1).int())


def test_sequences_of_a_workgroup_each():
    B, gamma, V = (1 << 22) + 5, 15, 129           # 1024 threads per sequence
    target = torch.zeros((B, gamma + 1, V), dtype=torch.bfloat16, device=DEV)
    draft = torch.zeros((B, gamma, V), dtype=torch.bfloat16, device=DEV)
    drafted = torch.zeros((B, gamma), dtype=torch.int32, device=DEV)
    u = ((torch.arange(B, device=DEV) % 61).float() / 64.0)[:, None].expand(B, gamma + 1).contiguous()
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    tau, y = sv.spec_verify_block(target, draft, drafted, u, 1.0, workspace=ws)
    assert torch.equal(tau, torch.full_like(tau, gamma))
    assert torch.equal(y.long(), (u[:, 0].double() * V).floor().long())


def test_a_workspace_of_more_words_is_prepared_whole():
    B, gamma, V = 1 << 21, 64, 2
    n = sv.spec_verify_workspace_bytes(B, gamma, V)
    assert n > 1.2 * (1 << 34)
    ws = torch.full((n,), 255, dtype=torch.uint8, device=DEV)
    sv.spec_verify_workspace_init(ws, B, gamma, V)
    assert sv.spec_verify_workspace_check(ws, B, gamma, V) == 0
    # (what is left as it was is the scratch area behind the control words: row sums and row constants)
    rows = B * (2 * gamma + 1)
    left = sum(int((part == -1).sum()) for part in ws.view(torch.int64).split(1 << 28)) * 8
    assert left <= rows * 64 and left < 0.5 * n
    assert not bool(ws[64:1 << 20].any())
