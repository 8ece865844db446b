"""The built library's device code holds kernels only.

A device function that the compiler leaves out of line is called through a return address
in a register pair, and branches across a very large function take that same pair for
their target: such a function does not return.  So everything is inlined, and every
function symbol of the code objects belongs to a kernel descriptor (name + ".kd")."""
import os
import struct

import pytest

from paper_1006_3340_amd import _build


def code_objects(data):
    """ELF images of the offload bundles in the library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" in triple and size:
                yield data[at + offset:at + offset + size]
        at = pos


def symbols(elf):
    """(name, type) of the image's symbol table entries that are defined."""
    assert elf[:5] == b"\x7fELF\x02"
    (shoff,) = struct.unpack_from("<Q", elf, 40)
    entsize, num = struct.unpack_from("<HH", elf, 58)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * entsize) for i in range(num)]
    for h in heads:
        if h[1] not in (2, 11):   # SHT_SYMTAB, SHT_DYNSYM
            continue
        names = heads[h[6]]
        for at in range(h[4], h[4] + h[5], 24):
            name, info, _, section, _, _ = struct.unpack_from("<IBBHQQ", elf, at)
            begin = names[4] + name
            if section:
                yield elf[begin:elf.index(b"\0", begin)].decode(), info & 15


def test_every_device_function_is_a_kernel():
    if not os.path.exists(_build.LIB):
        pytest.skip("library not built")
    with open(_build.LIB, "rb") as f:
        images = list(code_objects(f.read()))
    assert len(images) >= len(_build.SOURCES) // 2
    kernels, functions = set(), set()
    for elf in images:
        for name, kind in symbols(elf):
            if name.endswith(".kd"):
                kernels.add(name[:-3])
            elif kind == 2:       # STT_FUNC
                functions.add(name)
    assert kernels
    assert not functions - kernels, sorted(functions - kernels)
