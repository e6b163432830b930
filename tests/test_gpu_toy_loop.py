"""GPU: the drafting kernel against the oracle, and the outer loop (Alg. 3) on toy models run on the device
against the same loop around the oracle, fed the same uniforms."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2403_10444_amd as sv
import workloads
from paper_2403_10444_amd import specdec
from tests import parity, toy_loop

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MARGIN = 1e-6


@pytest.mark.parametrize("rows,V,dtype", [(64, 1, "f32"), (300, 2, "f32"), (100, 1000, "bf16"), (8, 8192, "f32"),
                                          (6, 8200, "bf16"), (4, 128256, "bf16"), (3, 50001, "f32")])
def test_sample_tokens_matches_the_oracle(rows, V, dtype):
    g = torch.Generator(device="cpu").manual_seed(rows * 7 + V)
    logits = torch.randn((rows, V), generator=g) * 3.0
    logits = logits.to(torch.bfloat16 if dtype == "bf16" else torch.float32).to(DEV)
    u = workloads.philox_uniforms(rows + V, (rows,))
    for T in (1.0, 0.6):
        got = sv.spec_sample_tokens(logits, torch.as_tensor(u, device=DEV), T).cpu().numpy()
        host = workloads.logits_to_numpy(logits)
        want, margins = oracle.sample_rows(host, u, T, dtype=oracle.BF16 if dtype == "bf16" else oracle.F32)
        bad = got != want
        assert not np.any(bad & (margins >= MARGIN)), (np.nonzero(bad)[0], margins[bad])
        assert bad.mean() < 0.02


def _rows_with_extremes(rows, V, dtype, seed, device):
    """At least six rows: the first holds its tail only and draws just below 1, the middle one its head only, the last one starts at
    V // 4 and draws at 0; ordinary rows and uniforms otherwise."""
    assert rows >= 6
    g = torch.Generator(device=device).manual_seed(seed)
    logits = torch.randn((rows, V), generator=g, device=device) * 4.0
    logits[0, : V - max(V // 2, 1) if V < 6000 else V - 3000] = float("-inf")
    logits[rows // 2, max(V // 3, 1):] = float("-inf")
    logits[-1, : V // 4] = float("-inf")
    u = workloads.philox_uniforms(rows + V, (rows,))
    u[-1], u[0] = 0.0, 1.0 - 2.0 ** -24
    return logits.to(torch.bfloat16 if dtype == "bf16" else torch.float32).to(DEV), u


def _check_rows(got, logits, u, T, dtype):
    rows, V = logits.shape
    want, margins = oracle.sample_rows(workloads.logits_to_numpy(logits), u, T, dtype=oracle.BF16 if dtype == "bf16" else oracle.F32)
    safe = margins >= MARGIN
    assert safe[1:-1].sum() >= 0.75 * (rows - 2), margins           # (what is compared below is not next to nothing)
    assert np.array_equal(got[safe], want[safe]), (np.nonzero(got != want)[0], margins)
    assert got[-1] == V // 4                                        # u = 0: the first token with weight
    for r in np.unique(np.concatenate([[0, rows // 2], np.nonzero(~safe)[0]])):
        x = logits[r].double().cpu().numpy() / T
        assert parity.in_cell(np.exp(x - x.max()), float(u[r]), int(got[r])), (r, u[r], got[r], want[r])


# (the edges of the kernels' ranges: one thread, sixteen lanes, a wave, four and sixteen waves per row, rows whose waves keep
# several units per lane; row counts that leave the last workgroup partly empty; rows at every alignment)
@pytest.mark.parametrize("rows,V,dtype", [(257, 32, "bf16"), (9, 33, "f32"), (37, 100, "bf16"), (18, 511, "f32"), (7, 512, "bf16"), (7, 513, "f32"),
                                          (6, 2047, "bf16"), (7, 2048, "f32"), (9, 2049, "bf16"), (8, 8191, "bf16"), (6, 8193, "f32"),
                                          (513, 8197, "bf16"), (600, 10001, "f32"), (8, 32768, "f32"), (9, 32769, "bf16"), (8, 2097153, "bf16")])
def test_sample_tokens_at_the_edges_of_its_kernels(rows, V, dtype):
    logits, u = _rows_with_extremes(rows, V, dtype, rows * 11 + V, "cpu")
    got = sv.spec_sample_tokens(logits, torch.as_tensor(u, device=DEV), 0.7).cpu().numpy()
    _check_rows(got, logits, u, 0.7, dtype)


# (rows spread over the device through scratch memory - the library's on the null stream, torch's on another current one -: the edges
# of the units and of the rule, a stretch of several units per lane; and the same rows by one workgroup each, on an explicit stream)
@pytest.mark.parametrize("rows,V,dtype", [(100, 49153, "bf16"), (101, 50257, "f32"), (104, 51200, "bf16"), (105, 51200, "f32"), (7, 131073, "bf16"),
                                          (64, 128256, "bf16"), (8, 262145, "f32"), (9, 1048576, "bf16"), (8, 1048577, "bf16")])
def test_sample_tokens_in_two_launches(rows, V, dtype):
    logits, u = _rows_with_extremes(rows, V, dtype, rows * 13 + V, DEV)
    ud = torch.as_tensor(u, device=DEV)
    units = (V + 2047) // 2048
    wanted = sv.load().spec_sample_workspace_bytes(rows, V)
    assert wanted == (rows * units * 16 if 24 < units <= 512 and rows <= 4 * units else 0)
    side = torch.cuda.Stream()
    assert torch.cuda.current_stream().cuda_stream == 0 and side.cuda_stream != 0
    torch.cuda.synchronize()
    null = sv.spec_sample_tokens(logits, ud, 0.7)
    with torch.cuda.stream(side):
        current = sv.spec_sample_tokens(logits, ud, 0.7)
    one_each = sv.spec_sample_tokens(logits, ud, 0.7, tokens=torch.empty_like(null), stream=side.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(null, current)                          # (the same kernels)
    for tokens in (null, one_each):
        _check_rows(tokens.cpu().numpy(), logits, u, 0.7, dtype)


def test_sample_tokens_from_several_threads_and_streams():
    """Threads that draw on the null stream at once share the library's scratch memory, call by call; others draw on streams
    and workspaces of their own."""
    import threading
    n, rows, V = 4, 48, 60000
    g = torch.Generator(device=DEV).manual_seed(17)
    logits = [torch.randn((rows, V), generator=g, device=DEV).mul_(4.0).to(torch.bfloat16) for _ in range(n)]
    uniforms = [torch.rand((rows,), generator=g, device=DEV) for _ in range(n)]
    want = [sv.spec_sample_tokens(x, u, 0.8).clone() for x, u in zip(logits, uniforms)]
    out = [torch.full((60, rows), -1, dtype=torch.int32, device=DEV) for _ in range(n)]
    streams = [0, 0, 0, torch.cuda.Stream().cuda_stream]
    ws = torch.empty(sv.spec_sample_workspace_bytes(rows, V), dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    start = threading.Barrier(n)

    def draw(i):
        start.wait()
        for k in range(60):
            sv.spec_sample_tokens(logits[i], uniforms[i], 0.8, tokens=out[i][k], stream=streams[i], workspace=ws if streams[i] else None)

    threads = [threading.Thread(target=draw, args=(i,)) for i in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(n):
        assert torch.equal(out[i], want[i].expand(60, rows)), i


def test_sample_tokens_into_given_tokens_allocates_nothing():
    """With the output handed over a call touches no allocator, with and without a workspace, on the current stream, on one
    handed over and under capture; the tokens are the same ones."""
    rows, V = 64, 50257
    g = torch.Generator(device=DEV).manual_seed(5)
    logits = torch.randn((3, rows, V), generator=g, device=DEV).mul_(4.0).to(torch.bfloat16)
    u = workloads.philox_uniforms(77, (3, rows))
    ud = torch.as_tensor(u, device=DEV)
    ws = torch.empty(sv.spec_sample_workspace_bytes(rows, V), dtype=torch.uint8, device=DEV)
    assert ws.numel() > 0
    want, margins = oracle.sample_rows(workloads.logits_to_numpy(logits.view(3 * rows, V)), u.reshape(-1), 0.7, dtype=oracle.BF16)
    want, safe = want.reshape(3, rows), margins.reshape(3, rows) >= MARGIN
    assert safe.sum() > 0.9 * safe.size
    tokens = torch.empty((rows,), dtype=torch.int32, device=DEV)
    side = torch.cuda.Stream()
    for workspace in (None, ws):
        for stream in (None, side.cuda_stream):
            tokens.fill_(-1)
            torch.cuda.synchronize()
            before = torch.cuda.memory_stats()["allocation.all.allocated"]
            out = sv.spec_sample_tokens(logits[0], ud[0], 0.7, tokens=tokens, stream=stream, workspace=workspace)
            assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
            torch.cuda.synchronize()
            assert out is tokens and np.array_equal(tokens.cpu().numpy()[safe[0]], want[0][safe[0]])
    with pytest.raises(sv.SpecVerifyError):
        sv.spec_sample_tokens(logits[0], ud[0], 0.7, tokens=tokens, workspace=ws[:-16])
    with pytest.raises(ValueError):
        sv.spec_sample_tokens(logits[0], ud[0], 0.7, tokens=tokens, workspace=ws.cpu())
    # (the two launches recorded, replayed on other rows, with eager work between the replays)
    rows_in, u_in = logits[0].clone(), ud[0].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sv.spec_sample_tokens(rows_in, u_in, 0.7, tokens=tokens, workspace=ws)
    for n in (1, 2, 0, 1):
        rows_in.copy_(logits[n])
        u_in.copy_(ud[n])
        tokens.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(tokens.cpu().numpy()[safe[n]], want[n][safe[n]]), n


def test_sample_tokens_of_rows_without_weight_is_token_0():
    for V in (2, 300, 1500, 9000, 40000, 60000):
        logits = torch.full((3, V), float("-inf"), device=DEV)
        assert sv.spec_sample_tokens(logits, torch.tensor([0.0, 0.5, 0.99], device=DEV), 1.0).tolist() == [0, 0, 0]


def test_sample_tokens_uniform_extremes():
    logits = torch.tensor([[0.0, -80.0, 1.0, -80.0]], device=DEV)
    assert int(sv.spec_sample_tokens(logits, torch.zeros(1, device=DEV), 1.0)[0]) == 0
    assert int(sv.spec_sample_tokens(logits, torch.full((1,), 1.0 - 2.0 ** -24, device=DEV), 1.0)[0]) == 2


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("gamma", [2, 10])
def test_toy_loop_on_the_device_equals_the_loop_around_the_oracle(algo, gamma):
    mb, ms = np.log(np.array([1 / 3, 2 / 3])), np.log(np.array([2 / 3, 1 / 3]))      # the paper's toy models
    B, iters, seed = 512, 4, 3
    ref = toy_loop.oracle_loop(algo, mb, ms, gamma, B, iters, 1.0, seed)
    got = specdec.toy_speculative_decoding(algo, mb, ms, gamma, B, iters, 1.0,
                                           lambda it: toy_loop.iteration_uniforms(seed, it, B, gamma), device=DEV)
    safe = ref["margin"] >= MARGIN
    assert safe.mean() > 0.99
    for key in ("tau", "y"):
        assert np.array_equal(got[key][safe], ref[key][safe]), key
    assert np.array_equal(got["x"][safe], ref["x"][safe])


def test_toy_loop_reproduces_the_ordering_of_the_ccdf():
    # the experiment of the paper's figure (gamma = 10): block verification accepts longer sub-blocks
    mb, ms = np.log(np.array([1 / 3, 2 / 3])), np.log(np.array([2 / 3, 1 / 3]))
    gamma, B, iters = 10, 4096, 8
    out = {}
    for algo in ("token", "block"):
        r = specdec.toy_speculative_decoding(algo, mb, ms, gamma, B, iters, 1.0,
                                             lambda it: toy_loop.iteration_uniforms(11, it, B, gamma), device=DEV)
        out[algo] = toy_loop.ccdf(r["tau"], gamma)
    exact_token = (2 / 3) ** np.arange(gamma + 1)
    assert np.abs(out["token"] - exact_token).max() < 4 * 0.5 / np.sqrt(B * iters)
    assert np.all(out["block"][2:] > out["token"][2:])         # Pr(tau >= 1) = 2/3 for both


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,V", [(1, 24 * 2048 + 1),                                # the narrowest rows that are spread: 25 units
                                    (3, 64 * 2048), (3, 64 * 2048 + 1), (2, 256 * 2048), (2, 256 * 2048 + 1),      # entries per lane; one launch and two
                                    (96, 61 * 2048 + 7), (97, 61 * 2048 + 7)])          # 1536 workgroups, one launch; 1552, two
def test_sample_tokens_on_the_null_stream(rows, V, dtype):
    """One launch where the call is small enough, call after call on the library's own words: the tokens of the one-workgroup-per-row
    kernel (another stream without scratch memory), which sums in another order: as the oracle says where the two differ."""
    from tests.parity import in_cell
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    x = (torch.randn((rows, V), generator=g, device="cuda") * 3.0).to(dtype)
    x[0, V // 3:] = -float("inf")                                     # (whole units without weight)
    side = torch.cuda.Stream()
    for turn in range(3):
        u = torch.rand((rows,), generator=g, device="cuda")
        if turn == 1:
            u[0], u[-1] = 0.0, 1.0 - 2.0 ** -24
        torch.cuda.synchronize()
        got = sv.spec_sample_tokens(x, u, 0.9, stream=0)
        want = sv.spec_sample_tokens(x, u, 0.9, tokens=torch.empty((rows,), dtype=torch.int32, device="cuda"), stream=side.cuda_stream)
        torch.cuda.synchronize()
        for r in (got != want).nonzero().flatten().tolist():
            p = torch.softmax(x[r].double() / 0.9, -1).cpu().numpy()
            assert in_cell(p, float(u[r]), int(got[r])), (turn, r)
        assert int((got != want).sum()) <= 1


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_sample_tokens_on_the_null_stream_after_waits_that_run_out(dtype):
    """A wave that stops waiting for the other units of its row forms what is missing itself: the same tokens, call after call, and what the
    others leave behind for it is nobody's: the calls that follow, of other rows, shapes and types, are right."""
    g = torch.Generator(device="cuda").manual_seed(5)
    calls = []
    for rows, V in ((64, 128256), (96, 61 * 2048 + 7), (1, 24 * 2048 + 1), (2, 256 * 2048 - 1), (64, 100001)):
        for dt in (dtype, torch.float32):
            x = (torch.randn((rows, V), generator=g, device="cuda") * 3.0).to(dt)
            u = torch.rand((rows,), generator=g, device="cuda")
            calls.append((x, u, sv.spec_sample_tokens(x, u, 0.9, stream=0)))
    for turn in range(3):
        for limit in (0, -1, 0, 0, -1):
            sv.spec_verify_debug_config(0, limit)
            try:
                for n in range(len(calls)):
                    x, u, want = calls[(n * 3 + turn) % len(calls)]
                    got = sv.spec_sample_tokens(x, u, 0.9, stream=0)
                    assert torch.equal(got, want), (turn, limit, tuple(x.shape), int((got != want).sum()), int(got.min()))
            finally:
                sv.spec_verify_debug_config(0, -1)
