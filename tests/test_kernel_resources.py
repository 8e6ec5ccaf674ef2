"""Registers of the built kernels against the residency that their launch rules count on.

The registers of a SIMD (512 per lane) are shared by its resident wavefronts, so a four-wavefront workgroup
leaves room for a second one on its CU only with at most 256 registers (vector and accumulation together).
The numbers are the ones that the compiler put into the code objects of the library built here.
"""
import os
import struct

import msgpack
import pytest


def _kernels(path):
    """Kernel name -> metadata of every code object bundled in the library."""
    out = {}
    blob = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in target:
                out.update(_notes(blob[at + off:at + off + size]))
        at = blob.find(magic, at + 24)
    return out


def _notes(elf):
    assert elf[:4] == b"\x7fELF"
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    found = {}
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        if kind != 4:                         # PT_NOTE
            continue
        p = off
        while p < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + namesz].rstrip(b"\0")
            d = p + 12 + (namesz + 3) // 4 * 4
            if name == b"AMDGPU" and ntype == 32:
                for k in msgpack.unpackb(elf[d:d + descsz]).get("amdhsa.kernels", []):
                    found[k[".name"]] = k
            p = d + (descsz + 3) // 4 * 4
    return found


@pytest.fixture(scope="module")
def kernels():
    from paper_1608_05794_amd import ck
    if not os.path.exists(ck.LIB_PATH):
        from paper_1608_05794_amd import build
        build.build()
    return _kernels(ck.LIB_PATH)


@pytest.mark.parametrize("np", [72, 80, 88, 96, 104, 112, 120])
def test_two_half_row_workgroups_per_cu(kernels, np):
    fit = [k[".vgpr_count"] for name, k in kernels.items() if f"Ros4CoopHalfILi{np}E" in name]
    print(np, fit)
    assert fit and min(fit) <= 256
