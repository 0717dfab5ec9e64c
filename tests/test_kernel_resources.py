"""What the compiler made of the attention kernels: none of them keeps anything in scratch memory.  A reload there waits for every load of the rings
that are counted by hand, and most calls are too short to hide it.  Read from the metadata of the library's own code objects."""
import os
import struct

import pytest

import __graft_entry__ as entry

msgpack = pytest.importorskip("msgpack")   # the metadata's format


def _kernels(path):
    """metadata of every kernel in the library's device code"""
    data, at, found = open(path, "rb").read(), 0, []
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, ids = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + ids]
            p += 24 + ids
            if b"gfx950" in target and size:
                found += _notes(data[at + off:at + off + size])
        at = p
    return found


def _notes(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    out = []
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + i * size + 24)
        end = off + length
        while kind == 7 and off < end:               # SHT_NOTE: name and description sizes, type
            name, desc, what = struct.unpack_from("<III", elf, off)
            at = off + 12 + (name + 3) // 4 * 4
            if what == 32:                           # the kernels' metadata
                out += msgpack.unpackb(elf[at:at + desc])["amdhsa.kernels"]
            off = at + (desc + 3) // 4 * 4
    return out


@pytest.mark.parametrize("kernel", ["decode_window_kernel", "decode_stream_kernel"])
def test_attention_kernels_use_no_scratch(kernel):
    if not os.path.exists(entry.LIB):
        entry.build()
    mine = [k for k in _kernels(entry.LIB) if kernel in k[".name"]]
    assert len(mine) == 16                           # head_dim, heads a group, statistic, format
    spilled = {k[".name"]: (k[".private_segment_fixed_size"], k.get(".vgpr_spill_count")) for k in mine
               if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")}
    assert not spilled
