"""Host-only checks of what the compiler made of the kernels, read from the code-object metadata in the built library."""
import re
import struct

import pytest

from paper_2112_15445_amd import binding as B


def _code_objects(data):
    """The gfx950 code objects of the offload bundles in the file."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(magic))
        q = at + len(magic) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, q)
            if b"gfx950" in data[q + 24:q + 24 + n] and size:
                yield data[at + off:at + off + size]
            q += 24 + n
        at = data.find(magic, at + len(magic))


def _kernels(elf):
    """The kernel entries of a code object's NT_AMDGPU_METADATA notes (type 32, msgpack)."""
    msgpack = pytest.importorskip("msgpack")
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    entry, count, _ = struct.unpack_from("<HHH", elf, 0x3A)
    for i in range(count):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entry)
        if kind != 7:                                        # SHT_NOTE
            continue
        o = off
        while o < off + size:
            name, desc, ntype = struct.unpack_from("<III", elf, o)
            d = o + 12 + (name + 3) // 4 * 4
            if ntype == 32:
                yield from msgpack.unpackb(elf[d:d + desc])["amdhsa.kernels"]
            o = d + (desc + 3) // 4 * 4


def _tile_kernels():
    """{(type, blocks along the channels, along the positions): metadata} of the one-shot matrix-core kernels."""
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    out = {}
    for elf in _code_objects(data):
        for k in _kernels(elf):
            m = re.search(r"mfma_tile_kernelIL\w*?10sc_dtype_t(\d)ELi(\d)ELi(\d)E", k[".name"])
            if m:
                out[tuple(map(int, m.groups()))] = k
    assert len(out) >= 26
    return out


def test_tile_kernels_use_no_scratch_memory():
    """The one-shot matrix-core kernels: no private segment.  (A workgroup index kept in memory costs every launch a
    store and a load before its first address, about 0.8 us.)"""
    tile = _tile_kernels().values()
    assert {k[".name"]: k[".private_segment_fixed_size"] for k in tile if k[".private_segment_fixed_size"]} == {}


def test_small_tile_kernels_leave_room_for_three_waves():
    """Wave tiles of up to four blocks: at most 168 of a SIMD's 512 registers a wave, so that three waves share it
    (what default_dense_tuning counts on); the larger ones two."""
    for (dtype, mw, nw), k in _tile_kernels().items():
        small = mw < 4 and mw * nw <= 4
        assert k[".vgpr_count"] + k.get(".agpr_count", 0) <= (168 if small else 256), (dtype, mw, nw)
