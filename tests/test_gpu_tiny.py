"""The one-workgroup-per-sequence kernel (sequences whose 2 gamma + 1 rows fit into LDS together) against the CPU
oracle: forced through the testing hook, and as the library's own choice for such shapes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2403_10444_amd as sv
from paper_2403_10444_amd import binding
import oracle
import workloads
from tests import parity

pytestmark = pytest.mark.gpu
DEV = "cuda"
TINY = 5                     # spec_verify_debug_config path
MAX_FLOATS = 14336           # (2 gamma + 1) V that the kernel takes


@pytest.fixture(autouse=True)
def forced():
    sv.spec_verify_debug_config(TINY, -1)
    yield
    sv.spec_verify_debug_config(0, -1)


def _custom(B, gamma, V, dtype="f32", sigma_t=3.0, sigma_d=1.0, T=1.0, zipf=False):
    assert (2 * gamma + 1) * V <= MAX_FLOATS
    return workloads.Config(f"tiny_B{B}_g{gamma}_V{V}_{dtype}", B, gamma, V, dtype, sigma_t, sigma_d, T, zipf, 1)


SHAPES = [
    # B, gamma, V, dtype
    (1, 4, 1000, "f32"),        # configuration 1
    (300, 4, 1000, "f32"),
    (64, 8, 840, "bf16"),
    (33, 1, 4736, "bf16"),      # one position, the widest rows that fit
    (17, 2, 2816, "f32"),
    (40, 64, 111, "bf16"),      # the longest draft the library takes
    (25, 16, 64, "f32"),        # rows of one wave's width
    (9, 3, 3, "f32"),           # a vocabulary of three tokens
    (12, 5, 2, "bf16"),         # the worked example's vocabulary
    (50, 7, 777, "bf16"),       # nothing a multiple of anything
]


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", SHAPES)
def test_shapes(B, gamma, V, dtype, algo):
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=0.8, T=0.9)
    for seed in (31, 32):
        inp = workloads.generate(cfg, seed=seed + B + gamma, device=DEV)
        rep = parity.compare(parity.run_gpu(algo, inp, cfg.temperature), parity.run_oracle(algo, inp, cfg.temperature),
                             label=f"{cfg.name}/{algo}/tiny", greedy=algo == "greedy")
        parity.record(rep)


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
def test_the_librarys_own_choice_for_small_sequences_is_this_kernel(algo):
    """Without the hook the library takes this kernel for such shapes: same outputs, bit for bit, debug block included;
    the large kernel forced on the same inputs agrees with both on tau and Y."""
    cfg = _custom(200, 6, 1100, "bf16", sigma_t=3.0, sigma_d=1.0, T=0.8)
    inp = workloads.generate(cfg, seed=77, device=DEV)
    a = parity.run_gpu(algo, inp, cfg.temperature)
    sv.spec_verify_debug_config(0, -1)
    b = parity.run_gpu(algo, inp, cfg.temperature)
    assert sv.spec_verify_debug_last_kernel() == binding.SV_KERNEL_TINY
    sv.spec_verify_debug_config(3, -1)
    c = parity.run_gpu(algo, inp, cfg.temperature)
    assert sv.spec_verify_debug_last_kernel() == binding.SV_KERNEL_FUSED
    for key in ("accept_len", "next_token", "dbg"):
        assert np.array_equal(a[key], b[key], equal_nan=True), key
    ref = parity.run_oracle(algo, inp, cfg.temperature)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert np.array_equal(a["accept_len"][safe], c["accept_len"][safe]) and np.array_equal(a["next_token"][safe], c["next_token"][safe])


def test_shapes_beyond_its_limit_are_refused_when_forced():
    cfg = workloads.Config("too_wide", 2, 4, 2000, "f32", 2.0, 1.0, 1.0, False, 1)       # 9 x 2000 logits > the limit
    inp = workloads.generate(cfg, seed=1, device=DEV)
    with pytest.raises(sv.SpecVerifyError) as e:
        sv.spec_verify_block(inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], 1.0)
    assert e.value.code == binding.SV_ERR_UNSUPPORTED


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
def test_identical_models_accept_everything(algo):
    cfg = _custom(16, 5, 1200, "bf16", sigma_t=4.0)
    inp = workloads.generate(cfg, seed=5, device=DEV)
    inp["draft_logits"] = inp["target_logits"][:, :cfg.gamma].contiguous()
    gpu = parity.run_gpu(algo, inp, 0.7)
    assert np.all(gpu["accept_len"] == cfg.gamma)
    parity.compare(gpu, parity.run_oracle(algo, inp, 0.7), greedy=algo == "greedy")


@pytest.mark.parametrize("algo", ["block", "token"])
def test_disjoint_supports_reject_everything(algo):
    cfg = _custom(8, 4, 1024, "f32", sigma_t=1.0)
    inp = workloads.generate(cfg, seed=6, device=DEV)
    V = cfg.V
    inp["target_logits"][..., : V // 2] -= 60.0
    inp["draft_logits"][..., V // 2:] -= 60.0
    q = torch.softmax(inp["draft_logits"].double(), -1)
    inp["draft_tokens"] = torch.multinomial(q.view(-1, V), 1).view(cfg.B, cfg.gamma).to(torch.int32)
    gpu = parity.run_gpu(algo, inp, 1.0)
    assert np.all(gpu["accept_len"] == 0)
    assert np.all(gpu["next_token"] >= V // 2)
    parity.compare(gpu, parity.run_oracle(algo, inp, 1.0))


def test_uniform_extremes():
    cfg = _custom(6, 4, 1500, "bf16")
    inp = workloads.generate(cfg, seed=8, device=DEV)
    for value in (0.0, 1.0 - 2.0 ** -24):
        inp2 = dict(inp, uniforms=torch.full_like(inp["uniforms"], value))
        for algo in ("block", "token", "greedy"):
            parity.compare(parity.run_gpu(algo, inp2, 1.0), parity.run_oracle(algo, inp2, 1.0))


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("kt,kd", [(50, 50), (20, 200), (500, 5), (1, 40)])
def test_masked_logits_top_k(algo, kt, kd):
    cfg = _custom(16, 6, 1100, "bf16", sigma_t=3.0, sigma_d=1.0, T=0.9)
    inp = workloads.generate(cfg, seed=300 + kt + kd, device=DEV, top_k_target=kt, top_k_draft=kd)
    assert torch.isinf(inp["target_logits"]).any() and torch.isinf(inp["draft_logits"]).any()
    parity.compare(parity.run_gpu(algo, inp, cfg.temperature), parity.run_oracle(algo, inp, cfg.temperature),
                   greedy=(algo == "greedy"))


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(24, 8, 840, "bf16"), (9, 5, 1291, "f32"), (130, 16, 300, "bf16")])
def test_ragged_draft_lengths(algo, B, gamma, V, dtype):
    """Sequence b must come out exactly as a call with gamma = draft_lens[b] on its leading rows does; the rows beyond
    a sequence's length are poisoned with NaN to show that they are never read."""
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=1.0, T=0.8)
    inp = workloads.generate(cfg, seed=500 + B + gamma, device=DEV)
    rng = np.random.default_rng(B * gamma)
    lens = rng.integers(1, gamma + 1, size=B).astype(np.int32)
    lens[0], lens[-1] = gamma, 1
    tl, dl = inp["target_logits"].clone(), inp["draft_logits"].clone()
    for b in range(B):
        tl[b, lens[b] + 1:] = float("nan")
        dl[b, lens[b]:] = float("nan")
    tau, y = sv.spec_verify_ex(algo, tl, dl, inp["draft_tokens"], inp["uniforms"], cfg.temperature,
                               draft_lens=torch.as_tensor(lens, device=DEV))
    torch.cuda.synchronize()
    tau, y = tau.cpu().numpy(), y.cpu().numpy()
    host = workloads.to_numpy(inp)
    odt = oracle.BF16 if dtype == "bf16" else oracle.F32
    n_safe = 0
    for g in np.unique(lens):
        sel = np.nonzero(lens == g)[0]
        ref = oracle.verify(parity.ALGOS[algo][0], host["target_logits"][sel, :g + 1], host["draft_logits"][sel, :g],
                            host["draft_tokens"][sel, :g], host["uniforms"][sel, :g + 1], cfg.temperature, dtype=odt)
        safe = ref["margins"].min(axis=1) >= parity.MARGIN
        n_safe += int(safe.sum())
        assert np.array_equal(tau[sel][safe], ref["accept_len"][safe]), (g, algo)
        same_tau = safe & (tau[sel] == ref["accept_len"])
        assert np.array_equal(y[sel][same_tau], ref["next_token"][same_tau]), (g, algo)
        assert np.all(tau[sel] <= g)
    assert n_safe >= 0.8 * B


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype,pad_t,pad_d", [(16, 8, 800, "bf16", 96, 32), (7, 4, 1191, "f32", 1, 9),
                                                          (70, 2, 2800, "bf16", 3, 5)])
def test_padded_rows(algo, B, gamma, V, dtype, pad_t, pad_d):
    """Rows inside buffers whose last dimension is padded (stride > V); the padding is poisoned with NaN."""
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=1.0, T=0.8)
    inp = workloads.generate(cfg, seed=700 + B + gamma, device=DEV)
    tbuf = torch.full((B, gamma + 1, V + pad_t), float("nan"), dtype=inp["target_logits"].dtype, device=DEV)
    dbuf = torch.full((B, gamma, V + pad_d), float("nan"), dtype=inp["draft_logits"].dtype, device=DEV)
    tbuf[..., :V] = inp["target_logits"]
    dbuf[..., :V] = inp["draft_logits"]
    tau, y = sv.spec_verify_ex(algo, tbuf[..., :V], dbuf[..., :V], inp["draft_tokens"], inp["uniforms"], cfg.temperature)
    torch.cuda.synchronize()
    ref = parity.run_oracle(algo, inp, cfg.temperature)
    safe = ref["margins"].min(axis=1) >= parity.MARGIN
    assert safe.sum() >= 0.8 * B
    assert np.array_equal(tau.cpu().numpy()[safe], ref["accept_len"][safe])
    assert np.array_equal(y.cpu().numpy()[safe], ref["next_token"][safe])


def test_workspace_must_be_initialised_for_the_shape():
    """This kernel needs nothing of the workspace, but the contract is one: a workspace prepared for another shape
    gives -1 outputs."""
    cfg = _custom(4, 3, 500, "f32")
    inp = workloads.generate(cfg, seed=3, device=DEV)
    ws = sv.alloc_workspace(cfg.B, cfg.gamma + 1, cfg.V, DEV)
    tau, y = sv.spec_verify_block(inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], 1.0,
                                  workspace=ws)
    torch.cuda.synchronize()
    assert bool((tau == -1).all()) and bool((y == -1).all())


# ---- 24 logits of a row per lane: the edges of its range, drafts that fill the workgroup
@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(66, 4, 1025, "f32"), (65, 15, 1536, "bf16"), (65, 16, 1535, "f32"), (2, 2, 1533, "bf16"), (65, 3, 1537, "f32")])
def test_rows_of_24_logits_per_lane(B, gamma, V, dtype, algo):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"lane24_B{B}_g{gamma}_V{V}", B, gamma, V, dtype, 2.5, 0.8, 0.9, False, 1)
    for n, (lens, pad_t, pad_d, top_k) in enumerate([(False, 0, 0, 0), (True, 3, 8, 30)]):
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=top_k, use_lens=lens, pad_t=pad_t, pad_d=pad_d, lens_seed=n), 300 + n, False)
        assert sv.spec_verify_debug_last_form() == (binding.SV_FORM_SEQUENCE, 64, 24 if V <= 1536 else 32)


# ---- the kernel that keeps the rows in LDS, which rows of more than 2048 logits reach (shorter ones, above and below, stay in
# registers): the edges of its range, draft lengths, masked logits, padded rows, the degenerate inputs, the workspace's contract
LDS_SHAPES = [(40, 1, 2049, "f32"), (33, 1, 4778, "bf16"), (17, 2, 2867, "f32"), (24, 2, 2053, "bf16"), (1, 1, 3001, "bf16")]


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", LDS_SHAPES)
def test_rows_in_lds(B, gamma, V, dtype, algo):
    from tests.test_gpu_random_shapes import _check
    cfg = _custom(B, gamma, V, dtype, sigma_t=2.5, sigma_d=0.8, T=0.9)
    for n, (lens, pad_t, pad_d, top_k) in enumerate([(False, 0, 0, 0), (True, 3, 8, 0), (True, 16, 5, 20), (False, 0, 0, 3)]):
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=top_k, use_lens=lens, pad_t=pad_t, pad_d=pad_d, lens_seed=B + V), 10 * V + n, False)
        assert sv.spec_verify_debug_last_kernel() == binding.SV_KERNEL_TINY
        assert sv.spec_verify_debug_last_form() == (binding.SV_FORM_SEQUENCE_IN_LDS, 0, 0)
    sv.spec_verify_debug_config(TINY, -1)
    inp = workloads.generate(cfg, seed=V, device=DEV)
    for value in (0.0, 1.0 - 2.0 ** -24):
        inp2 = dict(inp, uniforms=torch.full_like(inp["uniforms"], value))
        parity.compare(parity.run_gpu(algo, inp2, 1.0), parity.run_oracle(algo, inp2, 1.0), greedy=algo == "greedy")
    # the same distributions: everything is accepted; disjoint ones: nothing is
    same = dict(inp, draft_logits=inp["target_logits"][:, :gamma].contiguous())
    got = parity.run_gpu(algo, same, 0.7)
    assert np.all(got["accept_len"] == gamma)
    parity.compare(got, parity.run_oracle(algo, same, 0.7), greedy=algo == "greedy")
    if algo != "greedy":
        apart = {k: v.clone() for k, v in inp.items()}
        apart["target_logits"][..., : V // 2] -= 60.0
        apart["draft_logits"][..., V // 2:] -= 60.0
        q = torch.softmax(apart["draft_logits"].double(), -1)
        apart["draft_tokens"] = torch.multinomial(q.view(-1, V), 1).view(B, gamma).to(torch.int32)
        got = parity.run_gpu(algo, apart, 1.0)
        assert np.all(got["accept_len"] == 0) and np.all(got["next_token"] >= V // 2)
        parity.compare(got, parity.run_oracle(algo, apart, 1.0))
    ws = sv.alloc_workspace(B + 1, gamma, V, DEV)                # prepared for another shape
    tau, y = parity.ALGOS[algo][1](inp["target_logits"], inp["draft_logits"], inp["draft_tokens"], inp["uniforms"], 1.0, workspace=ws)
    assert bool((tau == -1).all()) and bool((y == -1).all())


# ---- rows in the registers of groups of lanes: every group size and register count at its edges, drafts that fill a wave or
# the workgroup (the last target row then has no group of its own), sequences that leave a shared workgroup partly empty,
# draft lengths, padded and unaligned rows.  (The library's own choice: path 0.)
EDGES = [
    # B, gamma, V, dtype
    (5, 10, 2, "f32"), (6, 15, 32, "bf16"), (7, 16, 32, "f32"), (3, 64, 3, "bf16"),
    (5, 3, 33, "f32"), (9, 8, 128, "bf16"), (2, 63, 100, "f32"), (2, 64, 128, "bf16"),
    (5, 15, 129, "bf16"), (4, 16, 300, "f32"), (3, 4, 512, "f32"), (2, 64, 512, "f32"),
    (6, 4, 513, "bf16"), (5, 15, 1000, "f32"), (4, 16, 1024, "bf16"), (3, 16, 1023, "f32"),
    (5, 3, 2048, "f32"), (70, 8, 1025, "bf16"), (66, 15, 2047, "f32"), (65, 16, 2048, "bf16"), (66, 16, 2041, "f32"),
]


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", EDGES)
def test_groups_of_lanes_at_their_edges(B, gamma, V, dtype, algo):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"groups_B{B}_g{gamma}_V{V}_{dtype}", B, gamma, V, dtype, 2.0, 0.5, 0.9, False, 1)
    for n, (lens, pad_t, pad_d) in enumerate([(False, 0, 0), (True, 3, 8)]):
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=0, use_lens=lens, pad_t=pad_t, pad_d=pad_d, lens_seed=B + V), 10 * V + n, False)
        assert sv.spec_verify_debug_last_kernel() == binding.SV_KERNEL_TINY
    # the same distributions: everything is accepted, the token comes from the last target row
    sv.spec_verify_debug_config(0, -1)
    inp = workloads.generate(cfg, seed=V + gamma, device=DEV)
    inp["draft_logits"] = inp["target_logits"][:, :gamma].contiguous()
    got = parity.run_gpu(algo, inp, 0.9)
    assert np.all(got["accept_len"] == gamma)
    parity.compare(got, parity.run_oracle(algo, inp, 0.9), label=f"{cfg.name}/{algo}/identical", greedy=algo == "greedy")


# ---- rows of more than 2048 logits that fit LDS: both sides of the line from which they have workgroups of their own (600 target rows)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,gamma,V,in_lds", [(300, 1, 3000, True), (301, 1, 3000, False), (300, 1, 4778, True), (301, 1, 4778, False),
                                              (200, 2, 2049, True), (201, 2, 2049, False), (200, 2, 2867, True), (201, 2, 2867, False)])
def test_the_line_from_rows_in_lds(B, gamma, V, in_lds, dtype):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"lds_line_B{B}_g{gamma}_V{V}", B, gamma, V, dtype, 2.5, 0.8, 0.9, False, 1)
    for n, (algo, lens, pad_t, pad_d) in enumerate([("block", False, 0, 0), ("token", True, 3, 8), ("greedy", True, 0, 5)]):
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=0, use_lens=lens, pad_t=pad_t, pad_d=pad_d, lens_seed=B + V), 50 + n, False)
        form = sv.spec_verify_debug_last_form()
        # (602 workgroups of rows of 4778: the kernel for calls that run at once)
        assert form == ((binding.SV_FORM_SEQUENCE_IN_LDS, 0, 0) if in_lds else (binding.SV_FORM_ROW, 128, 24) if V <= 3072 else (0, 0, 0))


# ---- several sequences to a workgroup, logits and probabilities: every number of lanes per row pair and of sequences per workgroup at the
# edges of its range, a last workgroup that is partly empty, drafts of the most positions that a form holds
PACKED = [
    (9, 15, 8, "f32"), (7, 16, 7, "bf16"), (3, 17, 5, "f32"), (2, 64, 8, "bf16"),
    (513, 3, 9, "f32"), (515, 16, 32, "bf16"), (3, 33, 31, "f32"),
    (1025, 7, 33, "bf16"), (1026, 2, 128, "f32"), (5, 8, 127, "bf16"), (2, 64, 100, "f32"),
    (1537, 7, 129, "f32"), (1366, 8, 256, "bf16"), (6, 31, 255, "f32"), (2, 32, 200, "bf16"),
    (5, 16, 257, "f32"), (3, 31, 512, "bf16"), (1639, 4, 300, "bf16"), (2, 63, 400, "f32"), (2, 64, 300, "bf16"),
    (4, 15, 511, "f32"), (4, 12, 513, "bf16"), (240, 12, 1024, "f32"), (2, 31, 700, "bf16"), (5, 15, 1025, "bf16"), (66, 5, 2048, "f32"), (3, 16, 1500, "f32"),
]
# the forms that logits and probabilities of these calls take: (several sequences to a workgroup or one,) lanes of a row pair, logits of each (None: another kernel's)
_ONE, _SEVERAL = binding.SV_FORM_SEQUENCE, binding.SV_FORM_SEQUENCES
FORMS = dict(zip(PACKED, [
    ((_SEVERAL, 1, 8), (1, 8)), ((_SEVERAL, 1, 8), (1, 8)), ((_SEVERAL, 1, 8), (1, 8)), ((_SEVERAL, 1, 8), (1, 8)),
    ((_SEVERAL, 4, 8), (4, 8)), ((_SEVERAL, 4, 8), (4, 8)), ((_ONE, 4, 8), (4, 8)),
    ((_ONE, 16, 8), (16, 8)), ((_SEVERAL, 16, 8), (16, 8)), ((_ONE, 16, 8), (16, 8)), ((_ONE, 16, 8), (4, 32)),
    ((_SEVERAL, 16, 16), (16, 16)), ((_SEVERAL, 16, 16), (16, 16)), ((_SEVERAL, 32, 8), (32, 8)), ((_SEVERAL, 16, 16), (16, 16)),
    ((_SEVERAL, 32, 16), (32, 16)), ((_SEVERAL, 32, 16), (32, 16)), ((_ONE, 64, 8), (32, 16)), ((_ONE, 16, 32), (16, 32)), ((_ONE, 16, 32), None),
    ((_ONE, 64, 8), (64, 8)), ((_ONE, 64, 16), (64, 16)), ((_ONE, 64, 16), (32, 32)), (None, (32, 32)), (None, (64, 32)), ((_ONE, 64, 32), (64, 32)), (None, None),
]))


@pytest.mark.parametrize("probs", [False, True], ids=["logits", "probs"])
@pytest.mark.parametrize("B,gamma,V,dtype", PACKED)
def test_sequences_that_share_a_workgroup(B, gamma, V, dtype, probs):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"packed_B{B}_g{gamma}_V{V}_{dtype}", B, gamma, V, dtype, 2.0, 0.5, 0.9, False, 1)
    of_logits, of_probs = FORMS[B, gamma, V, dtype]
    for algo in ("block", "token", "greedy"):
        for n, (lens, pad_t, pad_d, top_k) in enumerate([(False, 0, 0, 0), (True, 3, 8, 0), (True, 16, 0, 3)]):
            ran = _check(dict(cfg=cfg, algo=algo, path="default", top_k=top_k, use_lens=lens, pad_t=pad_t, pad_d=pad_d, lens_seed=B + V), 10 * V + n, probs)
            form = (of_probs and (_SEVERAL, *of_probs)) if probs else of_logits
            assert not ran or sv.spec_verify_debug_last_form() == (form or (0, 0, 0))


# ---- both sides of the lines between the forms of short rows (logits)
@pytest.mark.parametrize("B,gamma,V,dtype,form", [
    (600, 16, 32, "f32", (_SEVERAL, 4, 8)), (600, 17, 32, "f32", (_ONE, 4, 8)), (5, 64, 9, "bf16", (_ONE, 4, 8)),
    (1024, 6, 128, "f32", (_SEVERAL, 16, 8)), (1023, 6, 128, "f32", (_ONE, 16, 8)), (2048, 7, 33, "f32", (_ONE, 16, 8)),
    (2048, 7, 33, "bf16", (_SEVERAL, 16, 8)), (2047, 7, 33, "bf16", (_ONE, 16, 8)), (1024, 8, 128, "bf16", (_ONE, 16, 8)), (3, 63, 128, "bf16", (_ONE, 16, 8)), (3, 64, 128, "f32", (_ONE, 16, 8)),
    (257, 24, 256, "f32", (_SEVERAL, 16, 16)), (256, 31, 256, "bf16", (_SEVERAL, 32, 8)), (300, 31, 129, "bf16", (_SEVERAL, 16, 16)), (300, 23, 200, "f32", (_SEVERAL, 32, 8)),
    (1366, 5, 512, "bf16", (_SEVERAL, 32, 16)), (1365, 5, 512, "bf16", (_ONE, 64, 8)), (1366, 5, 300, "f32", (_ONE, 64, 8)),
    (4916, 4, 257, "bf16", (_SEVERAL, 32, 16)), (4915, 4, 257, "bf16", (_ONE, 64, 8)), (1201, 16, 384, "bf16", (_ONE, 16, 32)), (1200, 16, 384, "bf16", (_SEVERAL, 32, 16)),
    (1201, 16, 385, "bf16", (_SEVERAL, 32, 16)), (1201, 16, 384, "f32", (_SEVERAL, 32, 16)), (257, 23, 512, "bf16", (_SEVERAL, 32, 16)),
    (256, 31, 300, "f32", (_SEVERAL, 32, 16)), (257, 31, 300, "bf16", (_ONE, 16, 32)), (257, 24, 300, "f32", (_ONE, 16, 32)), (3, 32, 512, "f32", (_ONE, 16, 32)),
])
def test_both_sides_of_the_lines_between_short_rows(B, gamma, V, dtype, form):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"lines_B{B}_g{gamma}_V{V}_{dtype}", B, gamma, V, dtype, 2.0, 0.5, 0.9, False, 1)
    for n, (algo, lens, pad_t, pad_d) in enumerate([("block", False, 0, 0), ("token", True, 3, 8), ("greedy", False, 0, 5)]):
        # (drafts of four over 257 ... 512 and of their own lengths have another line, below)
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=0, use_lens=lens and (gamma, V) != (4, 257), pad_t=pad_t, pad_d=pad_d, lens_seed=B + V), 7 * V + n, False)
        assert sv.spec_verify_debug_last_form() == form


@pytest.mark.parametrize("B,gamma,V,dtype,form", [
    (2047, 6, 128, "f32", (_SEVERAL, 16, 8)), (2048, 6, 33, "f32", (_ONE, 16, 8)), (2048, 5, 33, "f32", (_SEVERAL, 16, 8)), (4095, 7, 40, "bf16", (_SEVERAL, 16, 8)), (4096, 7, 40, "bf16", (_ONE, 16, 8)),
    (4096, 6, 33, "bf16", (_ONE, 16, 8)), (13107, 4, 257, "bf16", (_ONE, 64, 8)), (13108, 4, 257, "bf16", (_SEVERAL, 32, 16))])
def test_both_sides_of_the_lines_between_short_rows_of_own_lengths(B, gamma, V, dtype, form):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"own_lines_B{B}_g{gamma}_V{V}_{dtype}", B, gamma, V, dtype, 2.0, 0.5, 0.9, False, 1)
    for n, algo in enumerate(("block", "token", "greedy")):
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=0, use_lens=True, pad_t=3 * n, pad_d=8 * n, lens_seed=B + V), 9 * V + n, False)
        assert sv.spec_verify_debug_last_form() == form


@pytest.mark.parametrize("gamma,pad_t,dtype,form", [(17, 23, "f32", (_SEVERAL, 1, 8)), (17, 24, "f32", (_ONE, 4, 8)), (16, 24, "f32", (_SEVERAL, 1, 8)), (17, 24, "bf16", (_SEVERAL, 1, 8))])
def test_very_short_rows_that_lie_apart(gamma, pad_t, dtype, form):
    from tests.test_gpu_random_shapes import _check
    cfg = workloads.Config(f"apart_g{gamma}_{dtype}", 70, gamma, 8, dtype, 2.0, 0.5, 0.9, False, 1)
    for n, algo in enumerate(("block", "token", "greedy")):
        _check(dict(cfg=cfg, algo=algo, path="default", top_k=0, use_lens=n == 1, pad_t=pad_t, pad_d=7, lens_seed=n), 40 + n, False)
        assert sv.spec_verify_debug_last_form() == form
