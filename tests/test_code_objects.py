"""What the compiler made of the kernels, read from the built library's own code objects: nothing in registers went to memory.  The
linear kernels keep up to 128 x 128 accumulators a wavefront and some use all but a few registers, where a spill would cost
more than any tile shape gains and no result would show it."""
import struct

import pytest

from paper_2604_15408_amd.build import LIB

msgpack = pytest.importorskip("msgpack")
_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    at = data.find(_MAGIC)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + n].decode()
            pos += 24 + n
            if "gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(_MAGIC, at + 1)


def _kernels(elf):
    """The kernels of the metadata note (type 32, msgpack) of an ELF file."""
    sections, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * entry + 4)
        offset, size = struct.unpack_from("<QQ", elf, sections + i * entry + 24)
        pos = offset if kind == 7 else offset + size           # SHT_NOTE
        while pos < offset + size:
            name, desc, note = struct.unpack_from("<III", elf, pos)
            body = pos + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            pos = body + (desc + 3) // 4 * 4


def test_no_kernel_spills():
    assert LIB.exists(), "build the library first"
    kernels = [k for elf in _code_objects(LIB.read_bytes()) for k in _kernels(elf)]
    names = [k[".name"] for k in kernels]
    assert sum("linear_kernel" in n for n in names) >= 2 * 2 * 16 and any("attn_kernel" in n for n in names)
    hot = ("linear_kernel", "attn_kernel", "layernorm_kernel")
    spilt = [(k[".name"], k[".vgpr_spill_count"], k[".sgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
             if k[".vgpr_spill_count"] or any(h in k[".name"] for h in hot) and (k[".sgpr_spill_count"] or k[".private_segment_fixed_size"])]
    assert not spilt, spilt
