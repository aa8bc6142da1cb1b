"""What the compiler made of the kernels, from the metadata of the library built here: no kernel spills vector registers, and the kernels whose
launches merge their own pieces leave room for others beside the workgroups that wait."""
import os
import re
import struct

import pytest

from paper_2508_07101_amd import binding as cb
from paper_2508_07101_amd import build as lib_build

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


def _all_kernels():
    cb.load()
    with open(cb.lib_path(), "rb") as fh:
        data = fh.read()
    return [k for obj in _device_objects(data) for k in _kernels(obj)]


def test_no_kernel_spills_vector_registers():
    kernels = _all_kernels()
    assert len(kernels) > 50, "the library's kernels were not found"
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled, f"vector registers spilled, bytes of scratch per lane: {spilled}"


def test_waiting_workgroups_leave_places_on_every_xcd():
    """Launches go to four hardware queues, so a launch's pieces share an XCD with the merging workgroups of three others of
    their kind at most (two to a row, an eighth of them on each XCD).  32 CUs of four SIMDs with 512 registers a lane, in eights, and 160 KB of LDS; a workgroup has a wave on every SIMD."""
    with open(os.path.join(lib_build.CSRC, "attn_plan.hpp")) as fh:
        cap = dict(re.findall(r"constexpr int (MERGE_ROWS_MAX\w*) = (\d+);", fh.read()))
    places = {}
    for k in _all_kernels():
        form = re.match(r"_ZN4cusa11attn_kernelILi(\d)ELi4ELb[01]ELb[01]ELb0ELb0ELb0EEE", k[".name"])   # tiles of 16 tokens, without scores
        if form:
            g = int(form.group(1))
            per_cu = min(512 // ((k[".vgpr_count"] + k[".agpr_count"] + 7) // 8 * 8), 160 * 1024 // k[".group_segment_fixed_size"])
            places[g] = min(32 * per_cu, places.get(g, 1 << 30))
    assert sorted(places) == [1, 2, 4, 8]
    for g, n in places.items():
        rows = int(cap["MERGE_ROWS_MAX_G8" if g == 8 else "MERGE_ROWS_MAX"])
        assert 3 * (2 * rows + 7) // 8 < n, f"groups of {g}: {3 * 2 * rows // 8} of {n} places"
