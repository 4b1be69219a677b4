"""Registers per lane of kernels whose speed hangs on how many workgroups share a CU, from the metadata
of the library's own code object."""
import re
import struct

import pytest

from paper_2410_00161_amd import binding as B

msgpack = pytest.importorskip("msgpack")


def kernels():
    """{kernel name: metadata} of every gfx950 code object in the library."""
    blob = open(B.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(rb"\x7fELF\x02\x01", blob):
        at = m.start()
        if struct.unpack_from("<H", blob, at + 18)[0] != 224:   # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", blob, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", blob, at + 58)
        for i in range(shnum):
            kind, = struct.unpack_from("<I", blob, at + shoff + i * shentsize + 4)
            off, size = struct.unpack_from("<QQ", blob, at + shoff + i * shentsize + 24)
            if kind != 7:   # SHT_NOTE
                continue
            p, end = at + off, at + off + size
            while p + 12 <= end:
                namesz, descsz, typ = struct.unpack_from("<III", blob, p)
                desc = p + 12 + (namesz + 3) // 4 * 4
                if typ == 32:   # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(blob[desc:desc + descsz])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                p = desc + (descsz + 3) // 4 * 4
    return out


def test_window_sums_leave_room_for_their_workgroups():
    """A SIMD has 512 registers per lane: 128 let four workgroups of 256 share a CU (what the LDS holds of
    32 to 128 query rows), 168 let three (256 rows of 64 dimensions)."""
    seen = 0
    for name, k in kernels().items():
        m = re.search(r"window_sum_kernelILi\dELi(\d+)ELi(\d+)ELi\d", name)
        if not m:
            continue
        seen += 1
        most = 128 if m[2] == "16" else 168 if m[1] == "64" else 256
        assert k[".vgpr_count"] <= most, (name, k[".vgpr_count"])
        assert k[".vgpr_spill_count"] == 0, name
    assert seen == 32


def test_short_block_decodes_leave_room_for_their_workgroups():
    """8-bit rows, d = 128, four query heads, blocks shorter than 16 tokens: 168 registers let three workgroups
    of four wavefronts share a CU; 128 let four one-wavefront items share a SIMD (blocks of one token)."""
    seen = 0
    for name, k in kernels().items():
        m = re.search(r"decode_chunk_kernelILi1ELi128ELi4ELb0ELi(\d)ELb(\d)E", name)
        if not m or m[1] + m[2] == "11":
            continue
        seen += 1
        assert k[".vgpr_count"] <= (168 if m[1] == "4" else 128), (name, k[".vgpr_count"])
        assert k[".vgpr_spill_count"] == 0, name
    assert seen == 2


def test_decodes_leave_room_for_as_many_workgroups_as_share_the_lds():
    """Chunks sized for four workgroups a CU (8-bit rows of d = 64 with four or eight query heads) need 128
    registers, for three (16-bit ones; 8-bit rows of d = 128 with eight, which spill three) 168."""
    seen = 0
    for name, k in kernels().items():
        m = re.search(r"decode_chunk_kernelILi(\d)ELi(\d+)ELi([48])ELb(\d)ELi4E", name)
        if not m:
            continue
        shape = m.groups()
        if shape[1] == "64" and shape[0] in "12":
            most, spills = 128 if shape[0] == "1" else 168, 0
        elif shape == ("1", "128", "8", "1"):
            most, spills = 168, 3
        else:
            continue
        seen += 1
        assert k[".vgpr_count"] <= most, (name, k[".vgpr_count"])
        assert k[".vgpr_spill_count"] <= spills, (name, k[".vgpr_spill_count"])
    assert seen == 9


def test_held_windows_leave_room_for_their_workgroups():
    """256 registers let two workgroups of four wavefronts share a CU, as many as the LDS holds.  With 128 rows
    of d = 128 held in 128 of them the statistics spill a few (the constants of the groups that are done over),
    the sums of 16-bit keys one."""
    seen = 0
    for name, k in kernels().items():
        m = re.search(r"window_held_(stats|sum)_kernelILi(\d)ELi(\d+)ELi(\d)E", name)
        if not m:
            continue
        seen += 1
        spills = {("stats", "2"): 8, ("stats", "1"): 8, ("sum", "2"): 1}.get(m.groups()[:2], 0) if m[3] + m[4] == "1288" else 0
        assert k[".vgpr_count"] <= 256, (name, k[".vgpr_count"])
        assert k[".vgpr_spill_count"] <= spills, (name, k[".vgpr_spill_count"])
    assert seen == 36
