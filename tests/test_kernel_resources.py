"""What the compiler reserved for the library's kernels, from the metadata in its own code objects (no GPU)."""
import struct

import pytest

from paper_2507_04123_amd import binding

msgpack = pytest.importorskip("msgpack")

_BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(_BUNDLE)
    while at >= 0:
        n, p = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + name]
            p += 24 + name
            if b"gfx950" in target and size:
                yield blob[at + off:at + off + size]
        at = blob.find(_BUNDLE, p)


def _kernels(obj):
    """The kernels' entries of an ELF's AMDGPU metadata note (type 32, MessagePack)."""
    phoff, phsize, phnum = struct.unpack_from("<Q", obj, 32)[0], *struct.unpack_from("<HH", obj, 54)
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", obj, phoff + i * phsize)
        end = off + size
        while kind == 4 and off < end:                                       # PT_NOTE
            name, desc, note = struct.unpack_from("<III", obj, off)
            body = off + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(obj[body:body + desc])["amdhsa.kernels"]
            off = body + (desc + 3) // 4 * 4


def test_no_kernel_uses_scratch_memory():
    """Registers that spill to memory cost a kernel its occupancy's worth: every form, those that read rows by address too,
    must fit the registers its launch bounds leave it."""
    found = {k[".name"]: k[".private_segment_fixed_size"] for o in _code_objects(open(binding.LIB_PATH, "rb").read()) for k in _kernels(o)}
    assert len(found) > 100
    assert {n: s for n, s in found.items() if s} == {}
