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


def _matrix_kernels():
    """({(type, blocks along the channels, along the positions, log2 of the columns a load, wide weights): metadata} of the one-shot
    matrix-core kernels, {(form, blocks along the channels, along the positions, groups, columns a load, eight products): metadata} of
    the fp32 split form's), every instantiation under a key of its own."""
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    tile, split = {}, {}
    for elf in _code_objects(data):
        for k in _kernels(elf):
            m = re.search(r"mfma_tile_kernelIL\w*?10sc_dtype_t(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)E", k[".name"])
            if m:
                out, key = tile, tuple(map(int, m.groups()))
            else:
                m = re.search(r"split_(conv|pipe)_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)E", k[".name"])
                if not m:
                    assert "mfma_tile_kernel" not in k[".name"] and "split_conv" not in k[".name"] and "split_pipe" not in k[".name"], k[".name"]
                    continue
                out, key = split, (m.group(1),) + tuple(map(int, m.groups()[1:]))
            assert key not in out
            out[key] = k
    return tile, split


def _registers(k):
    return k[".vgpr_count"] + k.get(".agpr_count", 0)


def test_every_instantiation_is_looked_at():
    """Two types x 13 wave tiles x four load widths and the one of wide weights; 9 wave tiles x two one-shot forms and 8 x two
    pipelined ones, each with three load widths and six or eight products."""
    tile, split = _matrix_kernels()
    waves = [(m, n) for m in (1, 2, 4) for n in (1, 2, 4, 7, 8) if not (m == 4 and n > 4)]
    assert set(tile) == {(t, m, n, c, w) for t in (1, 2) for m, n in waves for c, w in ((0, 0), (1, 0), (2, 0), (3, 0), (0, 1))}
    small = [(1, 1), (1, 2), (1, 4), (1, 7), (1, 8), (2, 1), (2, 2), (2, 4)]
    assert set(split) == {(f, m, n, g, c, full) for f, g, tiles in (("conv", 1, small + [(2, 7)]), ("conv", 2, small + [(2, 7)]), ("pipe", 2, small), ("pipe", 4, small))
                          for m, n in tiles for c in (1, 2, 4) for full in (0, 1)}


def test_tile_kernels_use_no_scratch_memory():
    """The one-shot matrix-core kernels: no private segment.  (A workgroup index kept in memory costs every launch a
    store and a load before its first address, about 0.8 us.)"""
    tile, _ = _matrix_kernels()
    assert {key: k[".private_segment_fixed_size"] for key, k in tile.items() if k[".private_segment_fixed_size"]} == {}


def test_small_tile_kernels_leave_room_for_three_waves():
    """Wave tiles of up to four blocks: at most 168 of a SIMD's 512 registers a wave, so that three waves share it
    (what default_dense_tuning counts on); the larger ones two."""
    tile, _ = _matrix_kernels()
    for (dtype, mw, nw, _, _), k in tile.items():
        small = mw < 4 and mw * nw <= 4
        assert _registers(k) <= (168 if small else 256), (dtype, mw, nw)


def test_split_kernels_spill_in_the_largest_wave_tiles_only():
    """The fp32 split form: the registers that its workgroups leave a wave (256; 168 in the pipelined form), and scratch memory only for
    2 x 7 blocks with two and four columns a load and for 2 x 4 with two groups in the pipelined form, at most 18 registers of it."""
    _, split = _matrix_kernels()
    for (form, mw, nw, groups, columns, full), k in split.items():
        assert _registers(k) <= (256 if form == "conv" else 168), (form, mw, nw, groups, columns, full)
        spills = (mw, nw) == (2, 7) and columns > 1 or form == "pipe" and (mw, nw, groups) == (2, 4, 2)
        assert k[".vgpr_spill_count"] <= (18 if spills else 0) and (spills or not k[".private_segment_fixed_size"]), (form, mw, nw, groups, columns, full)
