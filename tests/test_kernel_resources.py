"""What the built kernels take of the hardware, read from the library's own code objects."""
import struct

import pytest

from paper_2503_22796_amd import build


def _code_objects(data):
    """The gfx950 ELF images of the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        p = at + len(magic)
        n, = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(n):
            offset, size, id_size = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + id_size]:
                yield data[at + offset:at + offset + size]
            p += 24 + id_size
        at = p


def _kernel_descriptors(elf):
    """{kernel: its 64-byte descriptor}: the objects behind the symbols that end in .kd."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    found = {}
    for _, kind, _, _, offset, size, link, _, _, entsize in sections:
        if kind != 2 and kind != 11:                                    # SHT_SYMTAB, SHT_DYNSYM
            continue
        names = sections[link][4]
        for at in range(offset, offset + size, entsize):
            name, _, _, section, value, _ = struct.unpack_from("<IBBHQQ", elf, at)
            text = elf[names + name:elf.index(b"\0", names + name)].decode()
            if text.endswith(".kd"):
                where = sections[section][4] + value - sections[section][3]
                found[text[:-3]] = elf[where:where + 64]
    return found


@pytest.fixture(scope="module")
def kernels():
    with open(build.LIB, "rb") as f:
        data = f.read()
    return {k: d for elf in _code_objects(data) for k, d in _kernel_descriptors(elf).items()}


def test_no_kernel_spills_to_scratch(kernels):
    # a reload waits for every memory operation in flight, the tiles requested ahead among them
    attention = [k for k in kernels if "attn_bf16_kernel" in k]
    assert len(attention) == 3 and sum("attn_f32_kernel" in k for k in kernels) == 4
    scratch = {k: struct.unpack_from("<I", d, 4)[0] for k, d in kernels.items()}      # private segment, bytes a lane
    assert all(n == 0 for n in scratch.values()), scratch
