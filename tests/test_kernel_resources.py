"""The built library's own resource figures: the code object metadata that the
compiler wrote for every kernel of this package."""
import os
import struct

import pytest

from paper_2602_07397_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(blob):
    """The gfx950 ELF images of the offload bundles in a host library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + tl]:
                yield blob[at + off:at + off + size]
            p += 24 + tl
        at = blob.find(magic, at + 24)


def _kernels(elf):
    """The kernels listed in an ELF image's metadata note (type 32)."""
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    es, n = struct.unpack_from("<HH", elf, 0x3a)
    for i in range(n):
        (kind,) = struct.unpack_from("<I", elf, shoff + i * es + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * es + 24)
        p = off
        while kind == 7 and p < off + size:
            ns, ds, t = struct.unpack_from("<III", elf, p)
            p += 12 + ((ns + 3) & ~3)
            if t == 32:
                yield from msgpack.unpackb(elf[p:p + ds])["amdhsa.kernels"]
            p += (ds + 3) & ~3


def test_no_kernel_spills():
    """No kernel keeps registers in scratch memory (all of them run many
    workgroups, whose scratch traffic goes through the caches of the streams)."""
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        blob = f.read()
    kernels = [k for e in _code_objects(blob) for k in _kernels(e)]
    assert len(kernels) > 50
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled, spilled
