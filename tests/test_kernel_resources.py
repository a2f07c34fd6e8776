"""Resources of the built kernels, read from the library's own code objects: no kernel keeps
registers in scratch memory (each access would be a trip to memory on the replay path)."""

import struct

from paper_2608_15533_amd import deltalog as D

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of the library's offload bundles."""
    at = blob.find(BUNDLE)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            name = blob[entry + 24:entry + 24 + name_len]
            entry += 24 + name_len
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(BUNDLE, at + 24)


def _descriptors(elf):
    """(kernel, bytes of its 64-byte descriptor) for every symbol NAME.kd."""
    sh_off, = struct.unpack_from("<Q", elf, 40)
    sh_size, sh_num = struct.unpack_from("<HH", elf, 58)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, sh_off + i * sh_size) for i in range(sh_num)]
    for _, kind, _, _, offset, size, link, _, _, ent in sections:
        if kind != 11:                                     # the dynamic symbols
            continue
        strings = sections[link][4]
        for sym in range(offset, offset + size, ent):
            name_at, _, _, shndx, value, _ = struct.unpack_from("<IBBHQQ", elf, sym)
            name = elf[strings + name_at:elf.index(b"\0", strings + name_at)].decode()
            if name.endswith(".kd"):
                at = value - sections[shndx][3] + sections[shndx][4]
                yield name[:-3], elf[at:at + 64]


def test_no_kernel_uses_scratch_memory():
    with open(D.LIB_PATH, "rb") as f:
        blob = f.read()
    scratch, seen = {}, 0
    for elf in _code_objects(blob):
        for name, kd in _descriptors(elf):
            seen += 1
            private, = struct.unpack_from("<I", kd, 4)
            if private:
                scratch[name] = private
    assert seen > 1000                                     # the parser found the kernels
    assert not scratch, f"scratch bytes per lane: {scratch}"
