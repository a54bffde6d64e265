"""What the kernels of the built library take of a compute unit, from the metadata that the compiler writes beside the code (the
notes of the code objects inside the library)."""
import os
import struct

import msgpack
import pytest

from paper_2211_02048_amd import api


def _code_objects(path):
    """The gfx950 code objects of the library's bundles (one bundle per source file)."""
    data = open(path, "rb").read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + name_len].decode()
            pos += 24 + name_len
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at += len(magic)


def _kernels(elf):
    """The kernel records of the object's AMDGPU metadata note (type 32, MessagePack)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entry + 4)
        if kind != 7:                                       # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entry + 24)
        pos, end = off, off + size
        while pos + 12 <= end:
            name_len, desc_len, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (name_len + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc:desc + desc_len])["amdhsa.kernels"]
            pos = desc + (desc_len + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    api.lib()
    found = {k[".name"]: k for obj in _code_objects(api.LIB_PATH) for k in _kernels(obj)}
    assert len(found) > 200 and any("attn_kernel" in n for n in found) and any("conv_kernel" in n for n in found)
    return found


def _registers(k):
    """Vector registers per lane, of 512 that the waves of a SIMD share (handed out in eights)."""
    return (k[".vgpr_count"] + 7) // 8 * 8


def test_attention_registers_for_two_workgroups(kernels):
    """Four waves on the same chunks, heads of 97 to 128: two workgroups share a compute unit."""
    mine = {n: k for n, k in kernels.items() if "attn_kernelI" in n and "Li4ELi0ELi4ELi1E" in n or "Li4ELi1ELi4ELi1E" in n}
    assert len(mine) == 4
    for n, k in mine.items():
        assert _registers(k) <= 256, (n, _registers(k))


@pytest.mark.parametrize("name", ["conv_kernel", "conv_pair_kernel", "pointwise_kernel", "attn_kernel", "attn_f32_kernel", "attn_merge_kernel", "gn_"])
def test_no_scratch_memory(kernels, name):
    """Everything a kernel holds is in registers and LDS: no spills, no arrays in memory."""
    mine = {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if name in n}
    assert mine
    assert not any(mine.values()), [n for n, size in mine.items() if size]
