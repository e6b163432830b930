"""Every exported verification call by its own name and signature, on real inputs: the same outputs, bit for bit, as the
packed call that the Python binding goes through."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2403_10444_amd as sv
import workloads
from paper_2403_10444_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = 0.8


class _Out:
    def __init__(self, B, gamma):
        self.tau = torch.full((B,), -7, dtype=torch.int32, device=DEV)
        self.y = torch.full((B,), -9, dtype=torch.int32, device=DEV)
        self.dbg = torch.full((B, gamma + 1, 3), float("nan"), dtype=torch.float32, device=DEV)

    def pointers(self):
        return self.tau.data_ptr(), self.y.data_ptr(), self.dbg.data_ptr()

    def host(self):
        torch.cuda.synchronize()
        return self.tau.cpu().numpy(), self.y.cpu().numpy(), self.dbg.cpu().numpy()


@pytest.mark.parametrize("algo", ["block", "token", "greedy"])
@pytest.mark.parametrize("B,gamma,V,dtype", [(37, 3, 900, "f32"), (29, 5, 20000, "bf16")])
def test_each_entry_point_by_its_own_signature(B, gamma, V, dtype, algo):
    cfg = workloads.Config("entry", B, gamma, V, dtype, 2.5, 0.9, T, False, 1)
    inp = workloads.generate(cfg, seed=B, device=DEV)
    target, draft = inp["target_logits"].contiguous(), inp["draft_logits"].contiguous()
    tokens, uniforms = inp["draft_tokens"], inp["uniforms"]
    pad_t, pad_d = 24, 8
    wide_t = torch.full((B, gamma + 1, V + pad_t), float("nan"), dtype=target.dtype, device=DEV)
    wide_d = torch.full((B, gamma, V + pad_d), float("nan"), dtype=target.dtype, device=DEV)
    wide_t[..., :V], wide_d[..., :V] = target, draft
    lens = torch.tensor([1 + (3 * b) % gamma for b in range(B)], dtype=torch.int32, device=DEV)
    p, q = torch.softmax(target.float(), -1).to(target.dtype), torch.softmax(draft.float(), -1).to(target.dtype)
    ws = sv.alloc_workspace(B, gamma, V, DEV)
    lib, code = sv.load(), binding.SV_ALGO[algo]
    dt = binding.SV_DTYPE_F32 if dtype == "f32" else binding.SV_DTYPE_BF16
    stream = torch.cuda.current_stream().cuda_stream
    tail = (ws.data_ptr(), ws.numel())
    one = lambda t: t.data_ptr()
    padded = (one(wide_t), one(wide_d), one(tokens), one(lens), V + pad_t, V + pad_d, one(uniforms), B, gamma, V, dt)

    def raw(call):
        out = _Out(B, gamma)
        assert call(out.pointers()) == binding.SV_OK
        return out.host()

    def packed(call):
        out = _Out(B, gamma)
        call(dict(accept_len=out.tau, next_token=out.y, debug_out=out.dbg))
        return out.host()

    dense = getattr(lib, f"spec_verify_{algo}")
    pairs = {
        "dense": (lambda o: dense(one(target), one(draft), one(tokens), one(uniforms), B, gamma, V, dt, T, *tail, *o, stream),
                  lambda o: getattr(sv, f"spec_verify_{algo}")(target, draft, tokens, uniforms, T, workspace=ws, **o)),
        "ex": (lambda o: lib.spec_verify_ex(code, *padded, T, *tail, *o, stream),
               lambda o: sv.spec_verify_ex(algo, wide_t[..., :V], wide_d[..., :V], tokens, uniforms, T, draft_lens=lens, workspace=ws, **o)),
        "noalloc": (lambda o: lib.spec_verify_ex_noalloc(code, *padded, T, *o, stream),
                    lambda o: sv.spec_verify_ex_noalloc(algo, wide_t[..., :V], wide_d[..., :V], tokens, uniforms, T, o["accept_len"],
                                                        o["next_token"], draft_lens=lens, debug_out=o["debug_out"])),
        "probs": (lambda o: lib.spec_verify_probs(code, one(p), one(q), one(tokens), None, 0, 0, one(uniforms), B, gamma, V, dt, *tail, *o, stream),
                  lambda o: sv.spec_verify_probs(algo, p, q, tokens, uniforms, workspace=ws, **o)),
    }
    results = {}
    for name, (by_name, by_struct) in pairs.items():
        a, b = raw(by_name), packed(by_struct)
        for x, z in zip(a, b):
            assert np.array_equal(x, z, equal_nan=True), name
        assert np.all((a[0] >= 0) & (a[0] <= gamma)) and np.all((a[1] >= 0) & (a[1] < V)) and np.isfinite(a[2][:, 0]).all(), name
        results[name] = a
    # (the calls are not one and the same: draft lengths shorten some sequences, and another algorithm is another answer)
    assert np.all(results["ex"][0] <= lens.cpu().numpy()) and not np.array_equal(results["dense"][2], results["ex"][2], equal_nan=True)
    assert all(np.array_equal(x, z, equal_nan=True) for x, z in zip(results["ex"], results["noalloc"]))
    other = getattr(lib, "spec_verify_token" if algo != "token" else "spec_verify_block")
    assert not np.array_equal(raw(lambda o: other(one(target), one(draft), one(tokens), one(uniforms), B, gamma, V, dt, T, *tail, *o, stream))[2],
                              results["dense"][2], equal_nan=True)
