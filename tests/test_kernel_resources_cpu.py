"""Registers and scratch of the strip kernels, read from the code objects in the built library (no GPU): what bounds how many of
their workgroups share a compute unit."""
import re
import struct

import msgpack

import paper_2206_08869_amd as iodf
from paper_2206_08869_amd import binding


def _kernels():
    """Metadata of every kernel in the library: its code objects' notes."""
    iodf.load_library()
    with open(binding.LIB_PATH, "rb") as f:
        lib = f.read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    out, at = [], lib.find(magic)
    while at >= 0:
        entry = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", lib, entry - 8)[0]):
            offset, size, name_len = struct.unpack_from("<QQQ", lib, entry)
            target = lib[entry + 24:entry + 24 + name_len].decode()
            entry += 24 + name_len
            if "gfx950" in target and size:
                out += _notes(lib[at + offset:at + offset + size])
        at = lib.find(magic, at + 1)
    return out


def _notes(elf):
    sections, = struct.unpack_from("<Q", elf, 0x28)
    entry_size, n = struct.unpack_from("<HH", elf, 0x3A)
    for s in (sections + i * entry_size for i in range(n)):
        if struct.unpack_from("<I", elf, s + 4)[0] == 7:   # SHT_NOTE
            at = struct.unpack_from("<Q", elf, s + 0x18)[0]
            name_len, desc_len, _ = struct.unpack_from("<III", elf, at)
            at += 12 + (name_len + 3) // 4 * 4
            return msgpack.unpackb(elf[at:at + desc_len])["amdhsa.kernels"]
    return []


def _strip_blocks():
    """{(chunks outside, inside, second kernel's edge, tiles one, tiles two, takes runs): metadata}"""
    found = {}
    for k in _kernels():
        m = re.search(r"k_strip_blockILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E(?:Lb([01])E)?", k[".name"])
        if m:
            found[tuple(int(g or 0) for g in m.groups())] = k
    assert found
    return found


def test_one_strip_kernels_leave_room_for_a_third_workgroup():
    """512 registers to a SIMD's lane, in steps of eight: the largest kernels of 64 channels inside fit three times."""
    blocks = _strip_blocks()
    for kind in ((4, 2, 3, 6, 4, 0), (2, 2, 3, 6, 4, 0)):
        assert 512 // (-(-blocks[kind][".vgpr_count"] // 8) * 8) >= 3, blocks[kind]


def test_strip_kernels_use_no_scratch():
    """A register that spills goes through memory in the middle of the products' loops."""
    for kind, k in _strip_blocks().items():
        assert k[".private_segment_fixed_size"] == k[".vgpr_spill_count"] == k[".sgpr_spill_count"] == 0, (kind, k[".vgpr_spill_count"])
