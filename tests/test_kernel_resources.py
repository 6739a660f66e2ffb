"""Registers, LDS and scratch memory of the kernels as built: what the placement beside the attention pass rests on.  No GPU needed:
the numbers are in the metadata of this library's own code objects."""
import os
import struct

import msgpack
import pytest

from paper_2601_13684_amd import binding
from paper_2601_13684_amd.build import LIB

CU_LDS, SIMD_REGS = 160 * 1024, 512
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 code objects of the offload bundles inside the shared library."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def notes(elf):
    """Descriptors of the AMDGPU metadata notes of an ELF64 file."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, num = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        if kind != 7:                                # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 0x18)
        p = off
        while p < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if ntype == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                yield elf[desc:desc + descsz]
            p = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    binding.lib()
    assert os.path.exists(LIB)
    found = {}
    with open(LIB, "rb") as f:
        blob = f.read()
    for obj in code_objects(blob):
        for desc in notes(obj):
            for k in msgpack.unpackb(desc)["amdhsa.kernels"]:
                found[k[".name"]] = dict(regs=-(-k[".vgpr_count"] // 8) * 8, lds=k[".group_segment_fixed_size"],
                                         scratch=k[".private_segment_fixed_size"], threads=k[".max_flat_workgroup_size"])
    assert len(found) > 40
    return found


def of(kernels, part):
    got = {n: k for n, k in kernels.items() if part in n}
    assert got, part
    return got


def test_no_scratch_memory(kernels):
    assert not [n for n, k in kernels.items() if k["scratch"]]


def test_attention_leaves_room_for_a_side_kernel(kernels):
    for part in ("attn_split_kernel", "attn_split8_kernel"):
        for n, k in of(kernels, part).items():
            assert k["threads"] == 256 and k["regs"] <= 216, (n, k)
    # LDS that two attention workgroups leave, as the launches of mon_select and the gather's plan count on it: 110 KB with
    # the filter and up to four heads to a group, 76 KB without, 56 KB in groups of eight
    for part, room in (("attn_split_kernelILi4ELb1", 110), ("attn_split_kernelILi4ELb0", 76), ("attn_split8_kernelILb1", 56), ("attn_split8_kernelILb0", 56)):
        for n, k in of(kernels, part).items():
            assert 2 * k["lds"] + room * 1024 <= CU_LDS, (n, k)


def test_side_kernels_fit_beside_two_attention_workgroups(kernels):
    left = SIMD_REGS - 2 * 216                       # registers per lane of a SIMD; a workgroup has threads / 256 waves on each
    small = ["mon_selectILi512E", "gather_plan_bitmap_kernelILi512E", "gather_plan_kernel", "gather_kernel", "rep_logits_kernel", "mon_score_hist",
             "mon_compact", "mon_hist", "mon_count", "mon_write", "mon_decide", "mon_sparse_score"]
    for part in small:
        for n, k in of(kernels, part).items():
            assert k["regs"] * k["threads"] // 256 <= left, (n, k)


def test_direct_selection_fits_beside_two_attention_workgroups(kernels):
    for n, k in of(kernels, "mon_directILi512E").items():
        assert k["regs"] * k["threads"] // 256 <= SIMD_REGS - 2 * 216, (n, k)
    for n, k in of(kernels, "mon_direct").items():               # what its launches allow for
        assert k["lds"] <= 14 * 1024, (n, k)
