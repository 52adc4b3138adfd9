"""Properties of the kernels as they were built, read from the library's own code objects."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1610_02132_amd", "libqsgd.so")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 ELF images in a library (offload bundles: count, then offset, size, id length, id)."""
    at = data.find(BUNDLE)
    while at >= 0:
        count = struct.unpack_from("<Q", data, at + len(BUNDLE))[0]
        p = at + len(BUNDLE) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                yield data[at + off:at + off + size]
            p += 24 + n
        at = data.find(BUNDLE, at + len(BUNDLE))


def kernels(elf):
    """The kernels of a code object's metadata note (note type 32, owner AMDGPU)."""
    shoff, shentsize, shnum = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        end = off + size
        while kind == 7 and off < end:
            namesz, descsz, note = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (namesz + 3) // 4 * 4
            if note == 32 and elf[off + 12:off + 12 + 6] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            off = desc + (descsz + 3) // 4 * 4


def test_direct_encoder_keeps_its_values_in_registers():
    """(The team encoder's kernels for any data spill by choice: a budget of six waves per SIMD.)"""
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    seen, scratch = 0, []
    with open(LIB, "rb") as f:
        data = f.read()
    for elf in code_objects(data):
        for k in kernels(elf):
            if "k_encode_direct" not in k[".name"]:
                continue
            seen += 1
            if k[".private_segment_fixed_size"]:
                scratch.append((k[".name"], k[".private_segment_fixed_size"]))
    assert seen >= 40
    assert not scratch, f"{len(scratch)} of {seen} kernels: {scratch[:3]}"
