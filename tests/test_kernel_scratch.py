"""No kernel of the library keeps registers or arrays in scratch memory, but for the
persistent batch kernel, which holds every pass in one: read from the kernels'
metadata in the built library (amdhsa.kernels in the code objects' notes)."""
import struct

import pytest

from paper_2005_11806_amd import _abi

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of every offload bundle in blob."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, pos)
            triple = blob[pos + 24:pos + 24 + tlen]
            pos += 24 + tlen
            if triple.endswith(b"gfx950") and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def _kernels(elf, unpack):
    """The kernels' metadata: section type 7 (notes), note type 32 of AMDGPU."""
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    entsize, num = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(num):
        kind, _, _, off, size = struct.unpack_from("<IQQQQ", elf, shoff + i * entsize + 4)
        if kind != 7:
            continue
        pos = off
        while pos < off + size:
            nlen, dlen, typ = struct.unpack_from("<III", elf, pos)
            data = pos + 12 + (nlen + 3) // 4 * 4
            if typ == 32 and elf[pos + 12:pos + 18] == b"AMDGPU":
                yield from unpack(elf[data:data + dlen], raw=False)["amdhsa.kernels"]
            pos = data + (dlen + 3) // 4 * 4


def test_no_scratch():
    msgpack = pytest.importorskip("msgpack")
    with open(_abi.LIB_PATH, "rb") as f:
        blob = f.read()
    kernels = {k[".name"]: k[".private_segment_fixed_size"]
               for elf in _code_objects(blob) for k in _kernels(elf, msgpack.unpackb)}
    assert sum("k_yz" in n for n in kernels) > 100 and sum("k_inv_x" in n for n in kernels) > 50
    assert {n: s for n, s in kernels.items() if s and "k_batch_persistent" not in n} == {}
