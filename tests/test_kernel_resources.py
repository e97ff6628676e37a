"""Registers of the built kernels, read from the code objects in libhaze.so (CPU only)."""
import os
import struct

import msgpack
import pytest

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    """The gfx950 ELF images of the offload bundles (one per source file)."""
    at = lib.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", lib, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, idlen = struct.unpack_from("<QQQ", lib, entry)
            name = lib[entry + 24:entry + 24 + idlen]
            entry += 24 + idlen
            if b"gfx950" in name:
                yield lib[at + offset:at + offset + size]
        at = lib.find(MAGIC, entry)


def _kernels(elf):
    """The kernels' metadata: the msgpack note "AMDGPU" (type 32) of the ELF's note segments."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        ptype, _, offset, _, _, filesz = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        if ptype != 4:
            continue
        at, end = offset, offset + filesz
        while at + 12 <= end:
            namesz, descsz, kind = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if kind == 32 and elf[at + 12:at + 12 + namesz].rstrip(b"\0") == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            at = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    from paper_2603_02048_amd import haze
    if not os.path.exists(haze.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    with open(haze.LIB_PATH, "rb") as f:
        lib = f.read()
    found = {k[".name"]: k for elf in _code_objects(lib) for k in _kernels(elf)}
    assert len(found) > 40
    return found


@pytest.mark.parametrize("prefix,count", [
    ("_ZN4haze7k_marchILi1ELi0ELb0E", 2),      # F16, several fields in a launch: no scene (walking ahead or not)
    ("_ZN4haze7k_marchILi1ELi1ELb0E", 2),      # and boards outside the volume
    ("_ZN4haze14k_march_boardsILi1E", 1),      # F16, boards in the volume
    ("_ZN4haze12k_march_meshILi1E", 1)])       # F16, a triangle mesh
def test_f16_marches_without_row_bases_do_not_spill(kernels, prefix, count):
    """The march keeps its grid constants in vector registers only where there is
    room: with an address per view and row the F16 kernels spilled up to 21."""
    names = [n for n in kernels if n.startswith(prefix)]
    assert len(names) >= count
    assert {n: kernels[n][".vgpr_spill_count"] for n in names} == {n: 0 for n in names}


def test_tile_gather_does_not_spill(kernels):
    """Its particles' loop reloaded three or four registers, as many vector reads again."""
    names = [n for n in kernels if n.startswith("_ZN4haze13k_splat_tiles")]
    assert len(names) == 2
    assert {n: kernels[n][".vgpr_spill_count"] for n in names} == {n: 0 for n in names}
