"""What the compiler gave the kernels of the built library: read from the metadata note of its gfx950 code objects."""
import os
import re
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2004_13940_amd", "libfm_mi355x.so")
EM_AMDGPU, NT_AMDGPU_METADATA = 224, 32


def _notes(obj):
    """Descriptors of the AMDGPU metadata notes of one ELF64 code object."""
    shoff, = struct.unpack_from("<Q", obj, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", obj, 0x3A)
    for i in range(shnum):
        typ, = struct.unpack_from("<I", obj, shoff + i * shentsize + 4)
        off, size = struct.unpack_from("<QQ", obj, shoff + i * shentsize + 0x18)
        at = off
        while typ == 7 and at < off + size:
            namesz, descsz, kind = struct.unpack_from("<III", obj, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if kind == NT_AMDGPU_METADATA and obj[at + 12:at + 12 + 6] == b"AMDGPU":
                yield msgpack.unpackb(obj[desc:desc + descsz])
            at = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        from paper_2004_13940_amd import build
        build.build()
    data = open(LIB, "rb").read()
    found, at = {}, data.find(b"\x7fELF", 1)
    while at >= 0:
        if data[at + 4] == 2 and struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            for note in _notes(memoryview(data)[at:].tobytes() if at else data):
                for k in note["amdhsa.kernels"]:
                    found[k[".name"]] = k
        at = data.find(b"\x7fELF", at + 1)
    assert len(found) > 250, "kernels of the library"
    return found


def test_no_kernel_spills(kernels):
    """Every instantiation is reached by some K: registers that spill to scratch memory make the small ones, which have
    the most lane groups to a workgroup, many times slower."""
    spilled = {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if k[".private_segment_fixed_size"] > 0}
    assert spilled == {}


def test_wide_groups_leave_room_for_eight_wavefronts(kernels):
    """Columns and refresh with 16 lanes to a group and more (K > 32) have few runs per wavefront and are bound by latency:
    up to 64 of the 512 registers per lane of a SIMD, so that eight wavefronts fit."""
    wide = {n: k[".vgpr_count"] for n, k in kernels.items()
            if re.search(r"k_colsILi[124]ELi(16|32|64)E|k_rowsILi[124]ELi(16|32|64)ELi1E", n)}
    assert len(wide) == 27, sorted(wide)
    assert {n: v for n, v in wide.items() if v > 64} == {}


def test_columns_of_large_aggregates_keep_to_four_wavefronts(kernels):
    """Column kernels for aggregates beyond the memory-side cache: more than a fifth and at most a quarter of the 512
    registers per lane of a SIMD, so that four wavefronts fit and not five."""
    few = {n: k[".vgpr_count"] for n, k in kernels.items() if re.search(r"k_colsILi4ELi8ELb[01]ELi[01]ELb1EE", n)}
    assert len(few) == 4, sorted(few)
    assert {n: v for n, v in few.items() if not 512 // 5 < (v + 7) // 8 * 8 <= 512 // 4} == {}


def test_wide_groups_with_short_runs_leave_room_for_eight_wavefronts(kernels):
    wide = {n: k[".vgpr_count"] for n, k in kernels.items() if re.search(r"k_cols_partILi[124]ELi(16|32|64)E", n)}
    assert len(wide) == 18, sorted(wide)
    assert {n: v for n, v in wide.items() if v > 64} == {}
