"""Registers of kernel instances whose speed hangs on how many of their workgroups a compute unit holds, read from the code
object's metadata in the library built here (512 vector registers per SIMD lane: 64 a wave leave eight waves per SIMD, 80 six)."""
import re
import struct

import msgpack
import pytest

import paper_2604_25925_amd as sg
from paper_2604_25925_amd import binding


def _kernels():
    sg.load_library()
    blob = open(binding._LIB_PATH, "rb").read()
    found = {}
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:              # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", blob, at + 32)
            phentsize, phnum = struct.unpack_from("<HH", blob, at + 54)
            for p in range(phnum):
                kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", blob, at + phoff + p * phentsize)
                if kind != 4:                                              # PT_NOTE
                    continue
                pos, end = at + off, at + off + size
                while pos + 12 <= end:
                    nsz, dsz, typ = struct.unpack_from("<III", blob, pos)
                    data = pos + 12 + (nsz + 3 & ~3)
                    if typ == 32 and blob[pos + 12:pos + 12 + nsz] == b"AMDGPU\0":
                        for k in msgpack.unpackb(blob[data:data + dsz], strict_map_key=False)["amdhsa.kernels"]:
                            found[k[".name"]] = k
                    pos = data + (dsz + 3 & ~3)
        at = blob.find(b"\x7fELF", at + 4)
    return found


@pytest.fixture(scope="module")
def kernels():
    found = _kernels()
    assert len(found) > 50
    return found


def _instances(kernels, name, args):
    """The instances of a kernel template for bfloat16 (t) and float (f) with the given mangled arguments."""
    got = [kernels[k] for t in "tf" for k in kernels if re.search(r"\d%sI%s%sEE" % (name, t, args), k)]
    assert len(got) == 2, (name, args)
    return got


def test_rows_of_one_or_two_vectors_per_thread_do_not_spill(kernels):
    """Three workgroups of 512 threads per compute unit, at most 80 registers, and the kernel needs all of them."""
    for k in _instances(kernels, "k_rows", "Li512ELi2"):
        assert k[".vgpr_count"] <= 80 and k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, k[".name"]


def test_sums_in_parts_leave_room_for_four_workgroups(kernels):
    """Partial sums without pending levels: eight waves per SIMD of 512 threads, so that all parts of a small batch are resident at once."""
    for k in _instances(kernels, "k_ot_sum_parts", "Lb1ELb0"):
        assert k[".vgpr_count"] <= 64 and k[".vgpr_spill_count"] == 0, k[".name"]


def test_kseq_rows_from_memory_leave_room_for_three_workgroups(kernels):
    """One copy of the sweep; bfloat16 rows by vectors need a few more registers than that (85)."""
    for args in ("Lb0", "Lb1"):
        for k in _instances(kernels, "k_kseq_rows", args):
            assert k[".vgpr_count"] <= (88 if "k_kseq_rowsItLb1" in k[".name"] else 80) and k[".vgpr_spill_count"] == 0, k[".name"]
