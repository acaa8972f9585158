"""The index arithmetic of csrc/geometry.hpp, compiled for the host: what the kernels read and write
stays inside the buffers they are given."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def geo(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("geo") / "host_geometry.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "host_geometry.cpp")], check=True)
    L = C.CDLL(so)
    for name, args, res in [("geo_tiles", [C.c_uint64], C.c_uint32), ("geo_tile_elems", [], C.c_uint32),
                            ("geo_row_elems", [], C.c_uint32), ("geo_row_in_record", [C.c_uint32, C.c_uint64], C.c_uint32)]:
        getattr(L, name).argtypes, getattr(L, name).restype = args, res
    return L


# kind, levels -> (elements a read covers, its bytes); the nibble kinds are read as 32-bit words by
# one kernel and as 16-bit ones by another: the wider read counts
READS = {"identity": (4, 16), "fp16": (4, 8), "sign": (8, 1), "dither": (8, 4), "natdither": (8, 4), "dither5": (8, 4)}


@pytest.mark.parametrize("kind", sorted(READS))
@pytest.mark.parametrize("pe", [1024, 2048, 3072, 4096, 5120, 9216, 12288, 1 << 20])
def test_update_and_decode_read_inside_the_record(geo, kind, pe):
    """A thread of the Adam-style update and of the dense decode reads 4 elements of every row of
    its tile; partitions are a multiple of 1024 elements and a tile is 4096, so the rows of the
    last tile may lie past the record (and, in the last partition, past the payload)."""
    import paper_2105_07829_amd as bpc
    levels = 15 if kind == "dither5" else 4
    code = {"identity": bpc.IDENTITY, "fp16": bpc.FP16, "sign": bpc.SIGN, "natdither": bpc.NATDITHER}.get(kind, bpc.DITHER)
    stride = bpc.partition_stride(bpc.make_params(code, pe, levels=levels))
    assert bpc.payload_bytes(bpc.make_params(code, pe, levels=levels), 2 * pe - 1) == 2 * stride
    tile, row, tiles = geo.geo_tile_elems(), geo.geo_row_elems(), geo.geo_tiles(pe)
    rows = np.array([t * tile + r for t in range(tiles) for r in range(0, tile, row)])
    read = np.array([geo.geo_row_in_record(int(r), pe) for r in rows])
    assert np.array_equal(read[rows < pe], rows[rows < pe])   # what exists is read where it is
    per, size = READS[kind]

    def last(first_elements):   # the byte after the last one read
        j = int(first_elements.max()) + row - 4
        end = 16 + (j // per) * size + size
        if kind == "dither5":   # one plane, behind the nibbles
            end = max(end, 16 + 4 * (pe // 8) + j // 8 + 1)
        return end

    assert last(read) <= stride
    if pe % tile:   # (the reads that this is about)
        assert last(rows) > stride
