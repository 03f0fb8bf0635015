"""Registers of the compiled kernels, from the built library's own metadata:
the forms whose speed rests on how many waves a SIMD holds keep them.
"""
import os
import re
import struct

import msgpack
import pytest

from paper_2107_00555_amd import _lib


def _kernels(path):
    """{kernel symbol: metadata} of every gfx950 code object in a library."""
    blob = open(path, "rb").read()
    out = {}
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            off, size, namelen = struct.unpack_from("<QQQ", blob, entry)
            if blob[entry + 24:entry + 24 + namelen].endswith(b"gfx950"):
                for k in _metadata(blob[at + off:at + off + size]):
                    out[k[".name"]] = k
            entry += 24 + namelen
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


def _metadata(elf):
    """The kernels of an AMDGPU ELF's metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        end = off + size
        while kind == 7 and off < end:  # SHT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (namesz + 3) // 4 * 4
            if note == 32:  # NT_AMDGPU_METADATA
                return msgpack.unpackb(elf[desc:desc + descsz]).get("amdhsa.kernels", [])
            off = desc + (descsz + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2107_00555_amd import build
        build.build(verbose=False)
    return _kernels(_lib.LIB_PATH)


def _find(kernels, pattern):
    got = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert got, pattern
    return got


def _waves(k):
    """Waves a SIMD holds: 512 registers, given out in eights."""
    return 512 // ((k[".vgpr_count"] + k.get(".agpr_count", 0) + 7) // 8 * 8)


@pytest.mark.parametrize("op", [0, 1])  # forward, adjoint
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("lanes", ["dLi2E", "fLi4E"])
def test_one_step_kernel_with_sums_holds_four_waves(kernels, lanes, bc, op):
    # whole rows, two rows per lane
    for name, k in _find(kernels, rf"stencil_kernelI{lanes}Li1ELi4ELi2ELi{bc}ELi{op}ELb1E(Lb0E)?EE").items():
        assert _waves(k) >= 4 and k[".vgpr_spill_count"] == 0, (name, k[".vgpr_count"])


@pytest.mark.parametrize("bc", [0, 1])
def test_adjoint_step_with_running_sum_holds_four_waves(kernels, bc):
    # FP32, whole rows and ragged ones
    for name, k in _find(kernels, rf"stencil_kernelIfLi4ELi1ELi4ELi2ELi{bc}ELi3ELb1E").items():
        assert _waves(k) >= 4 and k[".vgpr_spill_count"] == 0, (name, k[".vgpr_count"])


def test_block_passes_spill_nothing(kernels):
    # (the loads of a block go out together only while every value has a register)
    for name, k in _find(kernels, r"12block_kernelI").items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name
