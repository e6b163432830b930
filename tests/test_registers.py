"""Registers of the kernels in the built library, from the metadata that the compiler left beside each: how many waves share a SIMD is what several
dispatch lines and launch sizes rest on, and one register more than a step of eight costs an eighth of it.  No GPU needed."""
from __future__ import annotations

import struct

import msgpack
import pytest

from paper_2403_10444_amd import binding

BUNDLE, TARGET = b"__CLANG_OFFLOAD_BUNDLE__", b"gfx950"


def _kernels():
    """Mangled name -> (vector registers, bytes of scratch memory per lane) of every kernel in the library."""
    data = open(binding.LIB_PATH, "rb").read()
    at = data.index(BUNDLE)
    entries, (count,) = at + 32, struct.unpack_from("<Q", data, at + 24)
    for _ in range(count):
        offset, size, length = struct.unpack_from("<3Q", data, entries)
        if TARGET in data[entries + 24:entries + 24 + length]:
            code = data[at + offset:at + offset + size]
            break
        entries += 24 + length
    # the ELF file's notes: name size, description size, type, name, description (msgpack)
    shoff, = struct.unpack_from("<Q", code, 40)
    shentsize, shnum = struct.unpack_from("<HH", code, 58)
    for n in range(shnum):
        kind, = struct.unpack_from("<I", code, shoff + n * shentsize + 4)
        if kind == 7:
            start, = struct.unpack_from("<Q", code, shoff + n * shentsize + 24)
            name_size, size, _ = struct.unpack_from("<3I", code, start)
            start += 12 + (name_size + 3) // 4 * 4
            meta = msgpack.unpackb(code[start:start + size], strict_map_key=False)
            return {k[".name"]: (k[".vgpr_count"], k[".private_segment_fixed_size"]) for k in meta["amdhsa.kernels"]}
    raise AssertionError("no kernel metadata")


@pytest.fixture(scope="module")
def kernels():
    return _kernels()


def _waves(registers):
    return min(8, 512 // ((registers + 7) // 8 * 8))


# a kernel's name with its element type and the start of its other parameters, and how many waves of it share a SIMD
@pytest.mark.parametrize("name,waves", [
    ("fused_verify_kernelINS_6bf16_tELb1ELi1ELi32E", 5), ("fused_verify_kernelIfLb1ELi1ELi32E", 4),
    ("resident_verify_kernelINS_6bf16_t", 5), ("together_verify_kernelINS_6bf16_t", 4), ("together_verify_kernelIf", 4),
    # rows of 513 to 1024 logits: at seven waves one sequence fewer shares a compute unit (three of nine waves, not two: 6153 sequences of 8 over 960 76 us, then 92)
    ("small_verify_kernelINS_6bf16_tELi64ELi16ELb0", 8),
    ("rows_verify_kernelINS_6bf16_tELb1ELi2ELi24E", 6), ("rows_verify_kernelINS_6bf16_tELb1ELi4ELi24E", 6), ("rows_verify_kernelINS_6bf16_tELb1ELi4ELi32E", 5),
    ("rows_verify_kernelINS_6bf16_tELb1ELi4ELi40E", 4), ("rows_verify_kernelIfLb1ELi4ELi48E", 4), ("rows_verify_kernelIfLb1ELi4ELi64E", 3),
])
def test_waves_per_simd(kernels, name, waves):
    found = {k: v for k, v in kernels.items() if name in k}
    assert found
    for kernel, (registers, scratch) in found.items():
        assert _waves(registers) >= waves, (kernel, registers)
        assert scratch == 0, (kernel, scratch)
