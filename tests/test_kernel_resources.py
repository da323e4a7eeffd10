"""What the built kernels take of the chip, read from the metadata of the
library's own gfx950 code objects (no GPU needed)."""
import os
import struct

import pytest

from paper_2010_10131_amd import _lib

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 ELF images of a library's offload bundles."""
    at = data.find(BUNDLE)
    while at >= 0:
        o = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, o)
            if b"gfx950" in data[o + 24:o + 24 + n]:
                yield data[at + off:at + off + size]
            o += 24 + n
        at = data.find(BUNDLE, at + 24)


def kernels():
    """Kernel name -> metadata (the NT_AMDGPU_METADATA note, MessagePack)."""
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("the library is not built (paper_2010_10131_amd/build.py)")
    with open(_lib.LIB_PATH, "rb") as f:
        data = f.read()
    out = {}
    for elf in code_objects(data):
        table, = struct.unpack_from("<Q", elf, 0x28)
        size, count = struct.unpack_from("<HH", elf, 0x3A)
        for s in range(table, table + size * count, size):
            if struct.unpack_from("<I", elf, s + 4)[0] != 7:   # SHT_NOTE
                continue
            p, length = struct.unpack_from("<QQ", elf, s + 0x18)
            end = p + length
            while p < end:
                ns, ds, kind = struct.unpack_from("<III", elf, p)
                d = p + 12 + (ns + 3) // 4 * 4
                if kind == 32:
                    for k in msgpack.unpackb(elf[d:d + ds], strict_map_key=False)["amdhsa.kernels"]:
                        out[k[".name"]] = k
                p = d + (ds + 3) // 4 * 4
    assert out, "no kernel metadata found"
    return out


@pytest.mark.parametrize("part", ["gram"])
def test_no_scratch_memory(part):
    """Register arrays stay in registers: a kernel that keeps one in scratch
    memory sends its loads of the next chunk through memory and waits for them."""
    found = {n: k[".private_segment_fixed_size"] for n, k in kernels().items() if part in n}
    assert found
    assert not {n: b for n, b in found.items() if b}
