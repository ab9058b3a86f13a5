"""Resources of the built kernels, read from the kernel descriptors of libnlpr.so's gfx950 code
object: no kernel keeps anything in scratch memory.  A register array whose index the compiler
does not know (a loop that it did not unroll) would go there: when that happened to the 9x9
branch-recording sweep, a gradient took twice its time."""
import os
import struct

import pytest

from paper_2210_04184_amd import nlpr

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    """The gfx950 ELF images of the offload bundles inside a shared library."""
    at = lib.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", lib, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", lib, pos)
            name = lib[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in name and size:
                yield lib[at + offset:at + offset + size]
        at = lib.find(MAGIC, at + 1)


def _descriptors(elf):
    """(name, scratch bytes per lane) of every kernel descriptor (the symbols NAME.kd; the
    private segment's size is the descriptor's second word)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    for _, kind, _, _, offset, size, link, _, _, entsize in sections:
        if kind != 2:                     # SHT_SYMTAB
            continue
        strings = sections[link][4]
        for at in range(offset, offset + size, entsize):
            name, _, _, shndx, value, _ = struct.unpack_from("<IBBHQQ", elf, at)
            end = elf.index(b"\0", strings + name)
            text = elf[strings + name:end].decode()
            if text.endswith(".kd") and 0 < shndx < shnum:
                _, _, _, base, start = sections[shndx][:5]
                yield text[:-3], struct.unpack_from("<I", elf, start + value - base + 4)[0]


def test_no_kernel_uses_scratch():
    if not os.path.exists(nlpr.LIB_PATH):
        pytest.skip("libnlpr.so is not built")
    with open(nlpr.LIB_PATH, "rb") as f:
        kernels = [k for elf in _code_objects(f.read()) for k in _descriptors(elf)]
    assert sum("sweep_kernel" in name for name, _ in kernels) >= 50     # the parser found them
    assert [k for k in kernels if k[1]] == []
