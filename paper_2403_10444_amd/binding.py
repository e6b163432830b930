"""ctypes binding of libspecverify.so: argument marshalling only.

Every step of the verification path runs in the HIP kernels behind the C ABI declared
in ``include/specverify.h``.  PyTorch is used for device memory and streams, nothing
else.  There is no CPU fallback: if the library has not been built, loading fails.
"""
from __future__ import annotations

import ctypes
import os
import struct

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# the product library; SPECVERIFY_LIBRARY names another build of it in this folder (the tuning build
# libspecverify_profile.so, which adds spec_verify_debug_profile)
LIB_PATH = os.path.join(_HERE, os.environ.get("SPECVERIFY_LIBRARY", "libspecverify.so"))

SV_OK = 0
SV_ERR_INVALID_ARG = 1
SV_ERR_UNSUPPORTED = 2
SV_ERR_WORKSPACE_TOO_SMALL = 3
SV_ERR_HIP = 4
SV_ERR_INTERNAL = 5
SV_ERR_STATIC_SCRATCH_TOO_SMALL = 6
SV_STATIC_SCRATCH_BYTES = 32 << 20
SV_DTYPE_F32 = 0
SV_DTYPE_BF16 = 1

EXPORTED = (
    "spec_verify_workspace_bytes",
    "spec_verify_workspace_init",
    "spec_verify_workspace_check",
    "spec_verify_debug_config",
    "spec_verify_debug_last_kernel",
    "spec_verify_debug_last_chain",
    "spec_verify_debug_last_together",
    "spec_verify_debug_last_form",
    "spec_verify_debug_copy",
    "spec_verify_debug_stream_probe",
    "spec_sample_tokens",
    "spec_sample_tokens_ws",
    "spec_sample_workspace_bytes",
    "spec_verify_block",
    "spec_verify_token",
    "spec_verify_greedy",
    "spec_verify_ex",
    "spec_verify_ex_noalloc",
    "spec_verify_probs",
    "spec_verify_call",
    "spec_verify_status_string",
)

_VERIFY_ARGTYPES = [
    ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
    ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_int, ctypes.c_float,
    ctypes.c_void_p, ctypes.c_size_t,
    ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
]

# sv_call_t of the header: ten pointers, two strides, the workspace's size, the temperature, six integers.  (One packed
# argument instead of seventeen converted ones: with what else is spared below, 9.3 -> 6.1 us of host time per call)
_pack_call = struct.Struct("@10P2qQd6i").pack
_CALL_LOGITS, _CALL_PROBS, _CALL_LOGITS_NOALLOC = 0, 1, 2

_lib = None


def _current_stream(index: int) -> int:
    """The raw handle of torch's current stream on a device (the public call makes a Stream object around it: 1.5 us)."""
    return _raw_stream(index) if _raw_stream is not None else torch.cuda.current_stream(index).cuda_stream


_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


class SpecVerifyError(RuntimeError):
    def __init__(self, code: int, text: str):
        super().__init__(f"specverify: {text} (status {code})")
        self.code = code


def load() -> ctypes.CDLL:
    """Load the built library; raises if it is missing (build it with build.py)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(
                f"{LIB_PATH} is not built; run `python -m paper_2403_10444_amd.build` "
                "(there is no fallback implementation)")
        lib = ctypes.CDLL(LIB_PATH)
        lib.spec_verify_workspace_bytes.restype = ctypes.c_size_t
        lib.spec_verify_workspace_bytes.argtypes = [ctypes.c_int32] * 3
        for name in ("spec_verify_block", "spec_verify_token", "spec_verify_greedy"):
            fn = getattr(lib, name)
            fn.restype = ctypes.c_int
            fn.argtypes = _VERIFY_ARGTYPES
        lib.spec_verify_ex.restype = ctypes.c_int
        lib.spec_verify_ex.argtypes = ([ctypes.c_int] + _VERIFY_ARGTYPES[:3]
                                       + [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64] + _VERIFY_ARGTYPES[3:])
        lib.spec_verify_ex_noalloc.restype = ctypes.c_int
        lib.spec_verify_ex_noalloc.argtypes = [a for j, a in enumerate(lib.spec_verify_ex.argtypes) if j not in (13, 14)]   # no workspace
        lib.spec_verify_probs.restype = ctypes.c_int
        lib.spec_verify_probs.argtypes = [a for j, a in enumerate(lib.spec_verify_ex.argtypes) if j != 12]   # no temperature
        lib.spec_verify_call.restype = ctypes.c_int
        lib.spec_verify_call.argtypes = [ctypes.c_char_p]                     # (the packed struct's bytes)
        lib.spec_verify_workspace_init.restype = ctypes.c_int
        lib.spec_verify_workspace_init.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int32,
                                                   ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
        lib.spec_verify_workspace_check.restype = ctypes.c_int
        lib.spec_verify_workspace_check.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32,
                                                    ctypes.c_int32, ctypes.c_void_p]
        lib.spec_verify_debug_last_kernel.restype = ctypes.c_int32
        lib.spec_verify_debug_last_kernel.argtypes = []
        lib.spec_verify_debug_last_chain.restype = ctypes.c_int32
        lib.spec_verify_debug_last_chain.argtypes = []
        lib.spec_verify_debug_last_together.restype = ctypes.c_int32
        lib.spec_verify_debug_last_together.argtypes = []
        lib.spec_verify_debug_last_form.restype = ctypes.c_int32
        lib.spec_verify_debug_last_form.argtypes = []
        lib.spec_verify_debug_config.restype = None
        lib.spec_verify_debug_config.argtypes = [ctypes.c_int32, ctypes.c_int32]
        if hasattr(lib, "spec_verify_debug_profile"):          # tuning builds only
            lib.spec_verify_debug_profile.restype = None
            lib.spec_verify_debug_profile.argtypes = [ctypes.c_void_p]
        lib.spec_verify_debug_copy.restype = ctypes.c_int
        lib.spec_verify_debug_copy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
        lib.spec_verify_debug_stream_probe.restype = ctypes.c_int
        lib.spec_verify_debug_stream_probe.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p,
                                                       ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
        lib.spec_sample_tokens.restype = ctypes.c_int
        lib.spec_sample_tokens.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int, ctypes.c_float,
                                           ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
        lib.spec_sample_workspace_bytes.restype = ctypes.c_size_t
        lib.spec_sample_workspace_bytes.argtypes = [ctypes.c_int64, ctypes.c_int32]
        lib.spec_sample_tokens_ws.restype = ctypes.c_int
        lib.spec_sample_tokens_ws.argtypes = lib.spec_sample_tokens.argtypes[:-1] + [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
        lib.spec_verify_status_string.restype = ctypes.c_char_p
        lib.spec_verify_status_string.argtypes = [ctypes.c_int]
        _lib = lib
    return _lib


def status_string(code: int) -> str:
    return load().spec_verify_status_string(int(code)).decode()


def spec_verify_workspace_bytes(B: int, gamma: int, V: int) -> int:
    return int(load().spec_verify_workspace_bytes(int(B), int(gamma), int(V)))


def spec_verify_workspace_init(workspace: torch.Tensor, B: int, gamma: int, V: int, stream=None) -> None:
    if stream is None:
        stream = torch.cuda.current_stream(workspace.device).cuda_stream
    code = load().spec_verify_workspace_init(workspace.data_ptr(), workspace.numel() * workspace.element_size(),
                                             int(B), int(gamma), int(V), stream)
    if code != SV_OK:
        raise SpecVerifyError(code, status_string(code))


def spec_verify_workspace_check(workspace: torch.Tensor, B: int, gamma: int, V: int, stream=None) -> int:
    """Blocks on the stream and returns the workspace's status code (SV_OK when healthy)."""
    if stream is None:
        stream = torch.cuda.current_stream(workspace.device).cuda_stream
    return int(load().spec_verify_workspace_check(workspace.data_ptr(), int(B), int(gamma), int(V), stream))


def spec_verify_debug_config(path: int = 0, spin_limit: int = -1) -> None:
    load().spec_verify_debug_config(int(path), int(spin_limit))


SV_KERNEL_STAGED, SV_KERNEL_FUSED, SV_KERNEL_TINY, SV_KERNEL_RESIDENT, SV_KERNEL_PROBS = 1, 2, 5, 7, 8


def spec_verify_debug_last_kernel() -> int:
    """Which kernels the last verification call of this process launched (SV_KERNEL_*; 0 before the first)."""
    return int(load().spec_verify_debug_last_kernel())


def spec_verify_debug_last_chain() -> int:
    """Testing hook: whether the last call on the fused kernel handed w_i on in a chain (see the header)."""
    return int(load().spec_verify_debug_last_chain())


def spec_verify_debug_last_together() -> int:
    """Testing hook: which kernel the last call of few resident sets took: 1 the one of together.hpp, 0 that of resident.hpp."""
    return int(load().spec_verify_debug_last_together())


SV_FORM_SEQUENCE_IN_LDS, SV_FORM_SEQUENCE, SV_FORM_SEQUENCES, SV_FORM_ROW = 1, 2, 3, 4


def spec_verify_debug_last_form() -> tuple:
    """Testing hook: the form of its kernel that the last verification call took: (SV_FORM_*, lanes that share a row (pair), logits of a
    row per lane); zeros where the kernel has one form."""
    form = int(load().spec_verify_debug_last_form())
    return form // 1000000, form // 1000 % 1000, form % 1000


def spec_verify_debug_profile(buffer) -> None:
    """Tuning builds only (see build.py): per-workgroup timestamps of the fused kernel go to `buffer` (a zeroed
    int64 device tensor [B * (gamma + 1) * workgroups per row, 16]) until called again with None."""
    lib = load()
    if not hasattr(lib, "spec_verify_debug_profile"):
        raise RuntimeError("this build of the library has no profiling hook; build with build.py --profile and "
                           "set SPECVERIFY_LIBRARY=libspecverify_profile.so")
    lib.spec_verify_debug_profile(buffer.data_ptr() if buffer is not None else None)


def spec_verify_debug_copy(dst: torch.Tensor, src: torch.Tensor, stream=None) -> None:
    """The library's plain copy kernel (what memory-traffic counters are scaled against)."""
    nbytes = src.numel() * src.element_size()
    if dst.numel() * dst.element_size() != nbytes:
        raise ValueError("dst and src must have the same size in bytes")
    if stream is None:
        stream = torch.cuda.current_stream(src.device).cuda_stream
    code = load().spec_verify_debug_copy(dst.data_ptr(), src.data_ptr(), nbytes, stream)
    if code != SV_OK:
        raise SpecVerifyError(code, status_string(code))


def spec_verify_debug_stream_probe(a: torch.Tensor, b: torch.Tensor, out: torch.Tensor, short_waits: int = 0,
                                   long_waits: int = 0, stream=None) -> None:
    """The library's streaming probe (the floor of the verification kernel's launch shape) over two equally large
    device buffers; `out` takes one float per 4096 bytes of `a`.  `short_waits`, `long_waits` (units of 512 clocks):
    the modelled waits of a verifying kernel, see the header; 0, 0 is the floor."""
    nbytes = a.numel() * a.element_size()
    if b.numel() * b.element_size() != nbytes or out.numel() * 4096 < nbytes or out.dtype != torch.float32:
        raise ValueError("a and b must have the same size in bytes and out one float32 per 4096 bytes of a")
    if stream is None:
        stream = torch.cuda.current_stream(a.device).cuda_stream
    code = load().spec_verify_debug_stream_probe(a.data_ptr(), b.data_ptr(), nbytes, out.data_ptr(),
                                                 int(short_waits), int(long_waits), stream)
    if code != SV_OK:
        raise SpecVerifyError(code, status_string(code))


def spec_sample_workspace_bytes(rows: int, V: int) -> int:
    """Bytes of scratch memory that `spec_sample_tokens` can use for this many rows of V logits (0: none)."""
    return int(load().spec_sample_workspace_bytes(rows, V))


def spec_sample_tokens(logits: torch.Tensor, uniforms: torch.Tensor, temperature: float, tokens=None, stream=None,
                       workspace=None):
    """One token per row of ``logits`` [..., V] from softmax(logits / T) by the inverse CDF at ``uniforms``
    [...] (the drafting step of Alg. 3).  Returns int32 tokens of the shape of ``uniforms``.

    Rows too few to fill the device are spread over it where there is scratch memory: on the null stream (torch's default one)
    the library has its own; elsewhere ``workspace`` (contiguous uint8 device tensor of `spec_sample_workspace_bytes`; calls
    that overlap need one each), on any stream and under graph capture.  A call that hands over ``tokens`` allocates nothing;
    one that makes its own output on another current stream takes scratch memory from the same allocator."""
    V = logits.shape[-1]
    rows = logits.numel() // V
    if not logits.is_cuda or not logits.is_contiguous() or not uniforms.is_contiguous():
        raise ValueError("logits and uniforms must be contiguous cuda tensors")
    if uniforms.numel() != rows or uniforms.dtype is not torch.float32:
        raise ValueError("one float32 uniform per row")
    if workspace is not None and (workspace.get_device() != logits.get_device() or not workspace.is_contiguous()):
        raise ValueError("the workspace must be a contiguous tensor on the logits' device")
    lib = _lib or load()
    current = stream is None
    if current:
        stream = _current_stream(logits.get_device())
    if tokens is None:
        tokens = torch.empty(uniforms.shape, dtype=torch.int32, device=logits.device)
        if workspace is None and current and stream:
            # (the allocator keeps both for the current stream: a stream of the caller's own is not known to it)
            n = lib.spec_sample_workspace_bytes(rows, V)
            if n:
                workspace = torch.empty(n, dtype=torch.uint8, device=logits.device)
    code = lib.spec_sample_tokens_ws(logits.data_ptr(), rows, V, _dtype_code(logits), float(temperature), uniforms.data_ptr(),
                                     tokens.data_ptr(), None if workspace is None else workspace.data_ptr(),
                                     0 if workspace is None else workspace.nbytes, stream)
    if code != SV_OK:
        raise SpecVerifyError(code, status_string(code))
    return tokens


def alloc_workspace(B: int, gamma: int, V: int, device="cuda") -> torch.Tensor:
    """A device byte buffer of the size the library asks for, initialised for this shape."""
    n = spec_verify_workspace_bytes(B, gamma, V)
    if n == 0:
        raise SpecVerifyError(SV_ERR_UNSUPPORTED, "sizes not supported")
    ws = torch.empty(n, dtype=torch.uint8, device=device)
    with torch.cuda.device(ws.device):
        spec_verify_workspace_init(ws, B, gamma, V)
    return ws


def _dtype_code(t: torch.Tensor) -> int:
    dtype = t.dtype
    if dtype is torch.float32:
        return SV_DTYPE_F32
    if dtype is torch.bfloat16:
        return SV_DTYPE_BF16
    raise TypeError(f"logits must be float32 or bfloat16, got {t.dtype}")


SV_ALGO = {"block": 0, "token": 1, "greedy": 2}


def _row_stride(t: torch.Tensor, rows_per_seq: int) -> int:
    """Row stride in elements of a [B, rows_per_seq, V] tensor whose rows are dense and evenly spaced
    (a contiguous tensor, or the [..., :V] view of one with a padded last dimension)."""
    B, R, V = t.shape
    sb, sr, sv_ = t.stride()
    if sv_ != 1 or sr < V or (B > 1 and sb != sr * rows_per_seq):
        raise ValueError("logits must have unit stride along the vocabulary and evenly spaced rows")
    return sr


def _call(inputs, algo, dense, target_logits, draft_logits, draft_tokens, uniforms, temperature,
          workspace=None, accept_len=None, next_token=None, debug_out=None, stream=None, draft_lens=None):
    lib = _lib or load()
    B, g1, V = target_logits.shape
    gamma = g1 - 1
    if not target_logits.is_cuda:
        raise ValueError("specverify runs on the GPU only; tensors must live on a cuda device")
    if draft_logits.shape != (B, gamma, V) or draft_tokens.shape != (B, gamma) or uniforms.shape != (B, g1):
        raise ValueError("shape mismatch between the inputs")
    if draft_logits.dtype is not target_logits.dtype:
        raise TypeError("target and draft logits must share a dtype")
    if draft_tokens.dtype is not torch.int32:
        raise TypeError(f"expected {torch.int32}, got {draft_tokens.dtype}")
    if uniforms.dtype is not torch.float32:
        raise TypeError(f"expected {torch.float32}, got {uniforms.dtype}")
    index = target_logits.get_device()
    if draft_logits.get_device() != index or draft_tokens.get_device() != index or uniforms.get_device() != index:
        raise ValueError("inputs must be on one device")
    if not (draft_tokens.is_contiguous() and uniforms.is_contiguous()):
        raise ValueError("inputs must be contiguous")
    if dense:
        if not (target_logits.is_contiguous() and draft_logits.is_contiguous()):
            raise ValueError("inputs must be contiguous")
        tstride = dstride = 0
        draft_lens = None                             # (not an argument of the dense calls)
    if workspace is None and inputs != _CALL_LOGITS_NOALLOC:
        workspace = alloc_workspace(B, gamma, V, target_logits.device)
    if accept_len is None:
        accept_len = torch.empty(B, dtype=torch.int32, device=target_logits.device)
    if next_token is None:
        next_token = torch.empty(B, dtype=torch.int32, device=target_logits.device)
    if stream is None:
        stream = _current_stream(index)
    elif type(stream) is not int:
        stream = ctypes.cast(stream, ctypes.c_void_p).value
    if not dense:
        if draft_lens is not None and (draft_lens.shape != (B,) or draft_lens.dtype is not torch.int32
                                       or draft_lens.get_device() != index or not draft_lens.is_contiguous()):
            raise ValueError("draft_lens must be a contiguous int32 tensor [B] on the inputs' device")
        tstride, dstride = _row_stride(target_logits, g1), _row_stride(draft_logits, gamma)
    code = lib.spec_verify_call(_pack_call(
        target_logits.data_ptr(), draft_logits.data_ptr(), draft_tokens.data_ptr(),
        0 if draft_lens is None else draft_lens.data_ptr(), uniforms.data_ptr(),
        0 if workspace is None else workspace.data_ptr(), accept_len.data_ptr(), next_token.data_ptr(),
        0 if debug_out is None else debug_out.data_ptr(), stream or 0, tstride, dstride,
        0 if workspace is None else workspace.nbytes, 0.0 if temperature is None else float(temperature),
        inputs, algo, B, gamma, V, _dtype_code(target_logits)))
    if code != SV_OK:
        raise SpecVerifyError(code, status_string(code))
    return accept_len, next_token


def spec_verify_ex(algo, target_logits, draft_logits, draft_tokens, uniforms, temperature, draft_lens=None, **kw):
    """`algo` ("block", "token" or "greedy") with the input variants of `spec_verify_ex` in the header:
    ``draft_lens`` (int32 device tensor [B], values 1 .. gamma, or None) makes sequence b use only its first
    draft_lens[b] draft positions; the logits may be ``[..., :V]`` views of buffers whose last dimension is
    padded (the row strides are taken from the tensors)."""
    return _call(_CALL_LOGITS, SV_ALGO[algo], False, target_logits, draft_logits, draft_tokens, uniforms, temperature,
                 draft_lens=draft_lens, **kw)


def spec_verify_ex_noalloc(algo, target_logits, draft_logits, draft_tokens, uniforms, temperature, accept_len, next_token,
                           draft_lens=None, debug_out=None, stream=None):
    """`spec_verify_ex` on the library's built-in scratch memory instead of a workspace (see the header): the call
    allocates nothing, so the outputs must be preallocated int32 device tensors [B].  Calls on one GPU must not
    overlap."""
    return _call(_CALL_LOGITS_NOALLOC, SV_ALGO[algo], False, target_logits, draft_logits, draft_tokens, uniforms, temperature,
                 accept_len=accept_len, next_token=next_token, debug_out=debug_out, stream=stream, draft_lens=draft_lens)


def spec_verify_probs(algo, target_probs, draft_probs, draft_tokens, uniforms, draft_lens=None, **kw):
    """`algo` ("block", "token" or "greedy") on distributions handed over as probabilities (the arrays of the
    paper's App. A), used as given: see `spec_verify_probs` in the header.  ``draft_lens`` and padded rows as for
    `spec_verify_ex`."""
    return _call(_CALL_PROBS, SV_ALGO[algo], False, target_probs, draft_probs, draft_tokens, uniforms, None,
                 draft_lens=draft_lens, **kw)


def spec_verify_block(target_logits, draft_logits, draft_tokens, uniforms, temperature, **kw):
    """Block verification (Alg. 2): returns (accept_len [B], next_token [B]) int32 device tensors.

    Asynchronous on the current (or given) stream.  Optional keyword arguments: ``workspace``
    (uint8 device tensor from `alloc_workspace`), preallocated ``accept_len`` / ``next_token``,
    ``debug_out`` (float32 [B, gamma+1, 3] device tensor receiving w, S, h) and ``stream``
    (a raw hipStream_t handle)."""
    return _call(_CALL_LOGITS, SV_ALGO["block"], True, target_logits, draft_logits, draft_tokens, uniforms, temperature, **kw)


def spec_verify_token(target_logits, draft_logits, draft_tokens, uniforms, temperature, **kw):
    """Token verification (Alg. 1); same arguments and returns as `spec_verify_block`."""
    return _call(_CALL_LOGITS, SV_ALGO["token"], True, target_logits, draft_logits, draft_tokens, uniforms, temperature, **kw)


def spec_verify_greedy(target_logits, draft_logits, draft_tokens, uniforms, temperature, **kw):
    """Greedy block verification (Alg. 4); same arguments and returns as `spec_verify_block`."""
    return _call(_CALL_LOGITS, SV_ALGO["greedy"], True, target_logits, draft_logits, draft_tokens, uniforms, temperature, **kw)
