"""No kernel of the built library uses scratch memory: a spilled register is reloaded from there, and in the pipelined
loops such a reload waits for every load in flight.  Read from the kernel descriptors of the library's gfx950 code
(the 64-byte objects <kernel>.kd of an AMDGPU code object; their second 32-bit word is the scratch size per lane).  Scalar registers
that the compiler keeps in lanes of vector registers go to no memory and are not seen here."""
import os
import struct

from paper_1901_08227_amd import binding as B
from paper_1901_08227_amd import build

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    at = data.find(BUNDLE)
    while at >= 0:
        pos = at + len(BUNDLE) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(BUNDLE))[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(BUNDLE, at + len(BUNDLE))


def scratch_bytes(elf):
    """{kernel: scratch bytes per lane}"""
    table, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, table + k * entry) for k in range(count)]
    found = {}
    for _, kind, _, _, offset, size, link, _, _, step in sections:
        if kind != 11:  # the dynamic symbols
            continue
        strings = sections[link][4]
        for k in range(offset, offset + size, step):
            name, _, _, section, value, _ = struct.unpack_from("<IBBHQQ", elf, k)
            text = elf[strings + name:elf.index(b"\0", strings + name)]
            if text.endswith(b".kd"):
                home = sections[section]
                found[text[:-3].decode()] = struct.unpack_from("<I", elf, home[4] + value - home[3] + 4)[0]
    return found


def test_no_kernel_uses_scratch():
    B.lib()  # builds it where there is none
    assert os.path.exists(build.LIB)
    kernels = {}
    for elf in code_objects(open(build.LIB, "rb").read()):
        kernels.update(scratch_bytes(elf))
    assert len(kernels) > 100
    assert not {k: v for k, v in kernels.items() if v}
