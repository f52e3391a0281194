"""What the compiler left in the library's own code objects about the built kernels: none uses scratch memory
(a kernel that spills a register sets scratch up at every launch: 4 us a decode call when it happened), and the
arguments lie where the kernels take them to be."""
import os
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_15969_amd", "lib", "liblazyev.so")


def _code_objects(data):
    """The gfx950 ELF images of an uncompressed offload bundle, wherever one starts in `data`."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name_len] and size:
                yield data[at + off:at + off + size]
            p += 24 + name_len
        at += len(magic)


def _kernels(elf):
    """Kernel descriptions of the metadata note (type 32, name AMDGPU) of an ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, _, _, off, size = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
        p = off
        while kind == 7 and p < off + size:        # SHT_NOTE
            name_len, desc_len, note = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (name_len + 3) // 4 * 4
            if note == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + desc_len])["amdhsa.kernels"]
            p = desc + (desc_len + 3) // 4 * 4


def _built_kernels():
    if not os.path.exists(LIB):
        pytest.fail("the library is not built (python -m paper_2506_15969_amd.build)")
    with open(LIB, "rb") as f:
        return [k for obj in _code_objects(f.read()) for k in _kernels(obj)]


def test_argument_block_lies_where_the_decode_kernel_reads_it():
    """The kernel reads its last argument, the block, at a fixed place among its arguments: 56 bytes in, behind five pointers, two
    lengths and the shape."""
    fused = [k for k in _built_kernels() if "decode_fused_kernel" in k[".name"]]
    assert len(fused) > 20
    for k in fused:
        explicit = [x for x in k[".args"] if not x[".value_kind"].startswith("hidden_")]
        assert [x[".offset"] for x in explicit] == [0, 8, 16, 24, 32, 40, 44, 48, 56], (k[".name"], explicit)
        assert [x[".size"] for x in explicit[:8]] == [8] * 5 + [4] * 3 and explicit[8][".value_kind"] == "by_value", k[".name"]


def test_no_kernel_uses_scratch_memory():
    kernels = _built_kernels()
    fused = [k for k in kernels if "decode_fused_kernel" in k[".name"]]
    assert len(fused) > 20 and len(kernels) > len(fused)   # (the notes were found)
    bad = {k[".name"]: (k[".private_segment_fixed_size"], k.get(".vgpr_spill_count")) for k in kernels
           if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")}
    assert not bad, bad
