"""Host test of the built library: no kernel of the forward and backward passes needs scratch memory (spilled vector registers), from
the metadata that the compiler leaves beside every kernel (.private_segment_fixed_size, bytes a lane)."""
import os
import struct

import msgpack
import pytest

from paper_2510_04008_amd import build

EM_AMDGPU, NT_AMDGPU_METADATA, SHT_NOTE = 224, 32, 7


def _code_objects(data):
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            yield at
        at = data.find(b"\x7fELF", at + 4)


def _kernels(data, elf):
    shoff, = struct.unpack_from("<Q", data, elf + 40)
    shentsize, shnum = struct.unpack_from("<HH", data, elf + 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", data, elf + shoff + i * shentsize + 4)
        offset, size = struct.unpack_from("<QQ", data, elf + shoff + i * shentsize + 24)
        at, end = elf + offset, elf + offset + size
        while kind == SHT_NOTE and at + 12 <= end:
            name, desc, note = struct.unpack_from("<III", data, at)
            body = at + 12 + (name + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA:
                yield from msgpack.unpackb(data[body:body + desc], strict_map_key=False).get("amdhsa.kernels", [])
            at = body + (desc + 3) // 4 * 4


def _library():
    if not os.path.exists(build.LIB):
        pytest.skip("the library is not built")
    with open(build.LIB, "rb") as f:
        return f.read()


def test_no_kernel_of_the_passes_uses_scratch():
    data = _library()
    # (the decoding step of large tables is not among them: it holds its rows in registers up to 32 at a time, and some outside)
    kernels = [k for elf in _code_objects(data) for k in _kernels(data, elf) if "decode_step" not in k[".name"]]
    assert len(kernels) > 100
    assert [k[".name"] for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]] == []


def test_gradient_kernels_that_fit_a_cu_twice():
    # 512 threads: two wavefronts per SIMD and workgroup, of 512 registers a SIMD
    data = _library()
    kernels = [k for elf in _code_objects(data) for k in _kernels(data, elf) if "grad_kernelINS0_3CfgILi128ELi4ELi4E" in k[".name"]]
    assert len(kernels) == 8            # dQ and dK, with and without the unit-norm option, causal or not
    assert [(k[".name"], k[".vgpr_count"]) for k in kernels if k[".vgpr_count"] > 128] == []
