"""Register use of the built kernels, from the metadata that the compiler
writes into the library's own gfx950 code objects (CPU, no GPU): a kernel
that spills pays for it in every pass of its loop, and in a loop that counts
its memory instructions a spill would shift the counts."""
import os
import struct

import msgpack
import pytest

from paper_2603_14806_amd import trimul as T

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA = 32


def code_objects(blob):
    """The device ELF images of the library's offload bundles."""
    at = blob.find(BUNDLE)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(BUNDLE))
        pos = at + len(BUNDLE) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "amdgcn" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(BUNDLE, pos)


def kernels(elf):
    """amdhsa.kernels of one 64-bit little-endian ELF's metadata notes."""
    (shoff,) = struct.unpack_from("<Q", elf, 40)
    entsize, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entsize)
        if kind != 7:   # SHT_NOTE
            continue
        pos, end = off, off + size
        while pos < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (namesz + 3) // 4 * 4
            if ntype == NT_AMDGPU_METADATA:
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            pos = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(T.LIB_PATH):
        from paper_2603_14806_amd import build
        build.build()
    with open(T.LIB_PATH, "rb") as f:
        found = {k[".name"]: k for elf in code_objects(f.read()) for k in kernels(elf)}
    assert len(found) > 30
    return found


def test_only_the_row_major_contractions_spill(built):
    """The contraction with a row-major result keeps 64-bit store addresses
    next to its 128 accumulators; every other kernel fits its registers."""
    spilling = {n for n, k in built.items() if k[".vgpr_spill_count"]}
    row_major_c = {n for n in built if "k2_contract_wsILb0E" in n or "k2_contract_wsILb1ELb0ELb0E" in n}
    assert row_major_c and spilling <= row_major_c, spilling - row_major_c
