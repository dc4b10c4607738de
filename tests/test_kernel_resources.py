"""Registers of the built kernels (no GPU needed): the rescaled FP64 sweeps must not
spill, whatever they share a kernel with.  Reads the metadata notes that the compiler
left in the library that this repository built."""
import os
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2411_11547_amd", "libpairhmm.so")


def kernels(path):
    """{mangled name: metadata} of every kernel in a library's offload bundles."""
    msgpack = pytest.importorskip("msgpack")
    data = open(path, "rb").read()
    magic, found, at = b"__CLANG_OFFLOAD_BUNDLE__", {}, data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in name:
                found.update(notes(data[at + off:at + off + size], msgpack))
        at = data.find(magic, at + 1)
    return found


def notes(elf, msgpack):
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    out = {}
    for k in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + k * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + k * size + 24)
        end = off + length
        while kind == 7 and off + 12 <= end:  # SHT_NOTE
            n, d, t = struct.unpack_from("<III", elf, off)
            body = off + 12 + (n + 3) // 4 * 4
            if t == 32:  # NT_AMDGPU_METADATA
                meta = msgpack.unpackb(elf[body:body + d], strict_map_key=False)
                out.update({m[".name"]: m for m in meta["amdhsa.kernels"]})
            off = body + (d + 3) // 4 * 4
    return out


def test_rescaled_fp64_sweeps_do_not_spill():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    found = {n: m for n, m in kernels(LIB).items() if "k_rescue" in n}
    assert len(found) >= 6
    # (the plain states of 16 rows per lane have never fitted)
    plain16 = "k_rescueILi3ELi3ELb0ELi1ELi1E"
    spilled = {n: m[".vgpr_spill_count"] for n, m in found.items() if m[".vgpr_spill_count"] and plain16 not in n}
    assert not spilled, spilled


def test_fp64_sweep_of_short_reads_has_its_own_tables():
    """Reads of up to 127 bases alone: 2 rows per lane, 16 waves per CU, of 160 KB of
    LDS and 512 registers in each of four SIMDs."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    found = {n: m for n, m in kernels(LIB).items() if "k_rescueILi0ELi0E" in n}
    assert len(found) == 2
    for n, m in found.items():
        assert 16 * m[".group_segment_fixed_size"] <= 160 * 1024 and 4 * m[".vgpr_count"] <= 512, n
