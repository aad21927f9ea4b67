"""Registers of the kernels in the built library, read from the metadata its code objects carry."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")


def _kernels_of_elf(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        sec = shoff + i * shentsize
        if struct.unpack_from("<I", elf, sec + 4)[0] != 7:          # SHT_NOTE
            continue
        at, size = struct.unpack_from("<QQ", elf, sec + 24)
        end = at + size
        while at < end:
            n_name, n_desc, kind = struct.unpack_from("<III", elf, at)
            at += 12 + (n_name + 3) // 4 * 4
            if kind == 32:                                          # AMDGPU metadata
                yield from msgpack.unpackb(elf[at:at + n_desc])["amdhsa.kernels"]
            at += (n_desc + 3) // 4 * 4


def _kernels(path):
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                yield from _kernels_of_elf(data[at + off:at + off + size])
            p += 24 + n
        at = data.find(magic, at + len(magic))


def test_no_decode_variant_spills_vector_registers():
    """A spilled register that is reloaded inside the record loop waits for every record load in flight.  One variant
    (threshold policy, 16 four-bit and 16 fp16 places, value groups of 32, key groups of 64 or more) has 20 bytes of spills."""
    import paper_2512_19206_amd as M
    if not os.path.exists(M.LIB_PATH):
        from paper_2512_19206_amd.build import build_library
        build_library()
    spilled = {}
    names = set()
    for k in _kernels(M.LIB_PATH):
        names.add(k[".name"])
        if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]:
            spilled[k[".name"]] = k[".private_segment_fixed_size"]
    assert sum("decode_fused_kernel" in n for n in names) > 200
    left = {n: b for n, b in spilled.items() if "decode_fused_kernelILi16ELi16ELi4ELi11ELi0ELi1ELi0ELi2ELi0EE" not in n}
    assert not left, left
    assert all(b <= 20 for b in spilled.values()), spilled
