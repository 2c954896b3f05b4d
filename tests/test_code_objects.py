"""What the compiler reports about the kernels of the built library (the AMDGPU
metadata notes of libpxm.so's gfx950 code objects)."""
import re
import struct

import msgpack
import pytest

from paper_2307_03404_amd import pxm


def kernels():
    """Metadata of every kernel in the library, by mangled name."""
    pxm.lib()                                          # builds it if it is absent
    blob = open(pxm.LIB_PATH, "rb").read()
    out = {}
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + tlen]
            p += 24 + tlen
            if b"gfx950" in target:
                out.update(_notes(blob[at + off:at + off + size]))
        at = blob.find(magic, at + 1)
    return out


def _notes(elf):
    found = {}
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entsize)
        if kind != 7:                                  # SHT_NOTE
            continue
        namesz, descsz, _ = struct.unpack_from("<III", elf, off)
        desc = off + 12 + (namesz + 3) // 4 * 4
        for k in msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]:
            found[k[".name"]] = k
    return found


@pytest.fixture(scope="module")
def meta():
    m = kernels()
    assert any("k_fused" in n for n in m) and any("k_team" in n for n in m) and any("k_backward" in n for n in m)
    return m


def test_dynamic_lds_begins_on_16_bytes(meta):
    """The scatter reads and writes its LDS, which follows a kernel's static LDS,
    16 bytes at a time."""
    # k_fused<grid, ., ., one launch or backward>, k_team<., grid>, k_backward
    scatters = re.compile(r"k_fusedILb1ELb[01]ELb[01]ELi[02]E|k_teamILi\dELb1E|k_backward")
    lds = {n: k[".group_segment_fixed_size"] for n, k in meta.items() if scatters.search(n)}
    assert len(lds) > 40
    assert not {n: b for n, b in lds.items() if b % 16}
