"""What the compiler made of the kernels, from the metadata of the library built here: no kernel spills vector registers."""
import struct

import pytest

from paper_2508_07101_amd import binding as cb

msgpack = pytest.importorskip("msgpack")
NT_AMDGPU_METADATA = 32


def _device_objects(data):
    """The gfx950 code objects bundled in a host library (offload bundle: magic, count, then offset, size and id each)."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24: p + 24 + id_len] and size:
                yield data[at + off: at + off + size]
            p += 24 + id_len
        at = data.find(magic, at + 32)


def _kernels(elf):
    """The kernels' metadata maps: the note of type NT_AMDGPU_METADATA of a 64-bit ELF object."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        if kind != 7:                                    # SHT_NOTE
            continue
        p = off
        while p < off + size:
            name_sz, desc_sz, note = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (name_sz + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA and elf[p + 12: p + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc: desc + desc_sz], raw=False)["amdhsa.kernels"]
            p = desc + (desc_sz + 3) // 4 * 4


def test_no_kernel_spills_vector_registers():
    cb.load()
    with open(cb.lib_path(), "rb") as fh:
        data = fh.read()
    kernels = [k for obj in _device_objects(data) for k in _kernels(obj)]
    assert len(kernels) > 50, "the library's kernels were not found"
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled, f"vector registers spilled, bytes of scratch per lane: {spilled}"
