"""Register use of the built kernels (CPU): the metadata of the code objects in libmclbm.so.

Values that are the same for all lattices of a node (store offsets at walls, the triplets of the species
source) cost registers from the first lattice to the last if the compiler keeps them; the kernels below then
spilled, or fell to one wave per SIMD, and took up to twice as long.
"""
import os
import re
import struct

import msgpack
import pytest

from paper_2004_11286_amd import build as B


def _code_objects(path):
    """The gfx950 ELF images of the offload bundles in a host library."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


def _metadata(elf):
    """The AMDGPU metadata note (type 32) of a code object."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for k in range(shnum):
        typ, = struct.unpack_from("<I", elf, shoff + k * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + k * shentsize + 24)
        if typ != 7:
            continue
        p = off
        while p < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                return msgpack.unpackb(elf[desc:desc + descsz])
            p = desc + (descsz + 3) // 4 * 4
    return {}


def kernels(path):
    return {m[".name"]: m for elf in _code_objects(path) for m in _metadata(elf).get("amdhsa.kernels", [])}


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(B.LIB):
        B.build_library()
    k = kernels(B.LIB)
    assert len(k) > 1000
    return k


def _check(built, pattern, count, vgprs):
    found = {n: m for n, m in built.items() if re.search(pattern, n)}
    assert len(found) == count, (pattern, len(found))
    for n, m in found.items():
        assert m[".vgpr_spill_count"] == 0 and m[".vgpr_count"] <= vgprs, (n, m[".vgpr_count"], m[".vgpr_spill_count"])


def test_16_bit_state_passes_at_x_walls(built):
    """Three and four species, strong coupling, both occupancy variants: two waves per SIMD, nothing spilled."""
    _check(built, r"k_state_speciesI(DF16_f|DF16bf|sf)fLi[34]ELi1ELi[01]ELb0E", 12, 256)


def test_split_species_collisions_of_the_property_step(built):
    """Temperature-dependent properties, FP32 storage, three and four species, every boundary, both couplings."""
    _check(built, r"k_collideIfdfLi[34]ELi[01245]ELi0ELi1ELb[01]ELb1E", 20, 256)


def test_fp64_state_passes_of_two_weakly_coupled_species(built):
    """Occupancy variant 1, every boundary: the whole register file of one wave per SIMD, nothing spilled."""
    _check(built, r"k_state_speciesIdddLi2ELi[01245]ELi1ELb1E", 5, 512)
