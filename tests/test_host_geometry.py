"""The index arithmetic of csrc/geometry.hpp, compiled for the host: what the kernels read and write
stays inside the buffers they are given."""
import ctypes as C

import numpy as np
import pytest


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


def _offsets(name, D):
    rng = np.random.default_rng(5)
    inner = np.sort(rng.integers(0, D, 300))
    return {"as_stated": np.concatenate([[0], inner, [D]]), "one_block": [0, D],
            "starts_late": np.concatenate([[9000], 9000 + inner, [D + 9000]]),   # (its last one ends past D, too)
            "one_block_starts_late": [20000, D], "ends_late": np.concatenate([[0], inner, [D + 5 * 8192]]),
            "ends_early": [0, 100, D // 2], "ends_far_beyond": [0, 17, 1 << 60],
            "descending": np.arange(D, 0, -100), "any_words": rng.integers(0, 1 << 63, 200)}[name]


@pytest.mark.parametrize("name", ["as_stated", "one_block", "starts_late", "one_block_starts_late", "ends_late", "ends_early",
                                  "ends_far_beyond", "descending", "any_words"])
@pytest.mark.parametrize("D", [777, 40_000, 150_001])
def test_lans_blocks_stay_inside_their_pairs_whatever_the_offsets(geo, name, D):
    """LANS over caller-defined blocks: tile t and block b meet at pair t + b.  The workspace has
    room for tiles + blocks - 1 pairs; offsets are data of the caller's that no host code sees."""
    offs = np.ascontiguousarray(_offsets(name, D), dtype=np.uint64)
    n_blocks, T = len(offs) - 1, geo.geo_lans_tile()
    tiles = -(-D // T)
    touched = []
    t0, n = C.c_uint64(), C.c_uint64()
    for t in range(tiles):      # norms and step pass: the blocks of a tile, from the one that holds its first element
        tile_end = min(D, (t + 1) * T)
        b0 = geo.geo_find_block(offs.ctypes.data, n_blocks, t * T)
        assert 0 <= b0 < n_blocks
        if name in ("as_stated", "one_block", "ends_late"):
            assert b0 == np.searchsorted(offs, t * T, side="right") - 1
        for b in range(b0, n_blocks):
            if int(offs[b]) >= tile_end:
                break
            touched += [t + b, int(offs[b]) // T + b]
            # what the norms pass leaves unfinished is what the totals pass finishes
            geo.geo_block_tiles(int(offs[b]), int(offs[b + 1]), D, C.byref(t0), C.byref(n))
            if int(offs[b + 1]) > max(int(offs[b]), t * T):
                assert (int(offs[b]) < t * T or int(offs[b + 1]) > geo.geo_tile_edge(tile_end, D)) == (n.value > 1)
    for b in range(n_blocks):   # totals pass
        geo.geo_block_tiles(int(offs[b]), int(offs[b + 1]), D, C.byref(t0), C.byref(n))
        if n.value > 1:
            touched += [t0.value + b, t0.value + n.value - 1 + b]
    assert not touched or (min(touched) >= 0 and max(touched) <= tiles + n_blocks - 2)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16, 17, 20, 63, 64])
@pytest.mark.parametrize("d", [1, 9, 1024, 8192, 9000, 300_007, 1 << 20, (1 << 23) + 1024, 1 << 28])
@pytest.mark.parametrize("ratio", [1e-9, 1e-3, 0.01, 0.1, 1.0])
def test_rows_in_front_of_the_topk_server_cover_everything_and_fit_a_grid(geo, n, d, ratio):
    """Every sampled chunk and every entry of every message (and its end) belong to one row; a grid has at most
    65535 rows, however many entries the messages have."""
    k_cap, out = max(1, int(ratio * d)), (C.c_uint32 * 8)()
    for guesses in (0, 1):
        geo.geo_prep_rows(n, k_cap, d, guesses, out)
        threads, slots, chunks, sums, messages, pieces, roles, starts = out
        entries = 8 * threads
        assert sums + starts <= 65535 and 1 <= starts <= roles
        assert slots * chunks == threads and (slots >= n or slots == 16)
        assert sums * chunks >= geo.geo_sample_chunks(d) * guesses
        assert pieces * entries >= k_cap + 1
        if pieces > 1:
            assert messages == 1 and roles == n * pieces
        else:
            assert messages * (k_cap + 1) <= entries and roles * messages >= n > (roles - 1) * messages


@pytest.mark.parametrize("k,d,fits", [(3000, 300_007, 1), (10_485, 1 << 20, 1), (16_384, 1 << 20, 1), (2097, 1 << 21, 1), (14_000, 1 << 21, 1),
                                      (4194, 1 << 22, 1), (16_384, 1 << 22, 0), (8388, 1 << 23, 1), (9500, 1 << 23, 0), (838, 1 << 23, 1),
                                      (12_582, 12 << 20, 0), (16_384, 65_536, 1), (16_384, 32_768, 1), (16_000, 16_200, 1), (30, 100, 1), (1, 7, 1)])
def test_topk_lists_are_taken_where_they_fit(geo, k, d, fits):
    """The length of a list: how many elements of a partition lie at or above the key of a rank of the sample.  Where the
    rule says that it fits, it does, and holds at least k, in draws of a sample from elements in no order but
    for some 0.3 % on either side (2.75 standard deviations): 200 draws, five or fewer (mean 1.2)."""
    assert geo.geo_topk_list_fits(k, d) == fits
    m = 8 * geo.geo_sample_chunks(d)
    rank = geo.geo_sample_rank(k, m, d)
    assert rank * d >= k * m
    if not fits or rank >= m:
        return
    rs, cap = np.random.default_rng(k + d), geo.geo_topk_list_cap()
    # (elements numbered from the largest)
    lengths = np.array([np.sort(rs.choice(d, m, replace=False))[rank - 1] + 1 for _ in range(200)])
    assert np.count_nonzero((lengths < k) | (lengths > cap)) <= 5


@pytest.mark.parametrize("part,D,ratio,form", [(1024, 1 << 24, 0.001, 0), (1024, 1 << 24, 1.0, 0), (16_384, 1 << 24, 0.1, 0), (65_536, 1 << 24, 0.01, 0),
                                               (1 << 20, 1 << 24, 0.001, 0), (1 << 20, 300_007, 0.01, 0), (1 << 20, 1 << 24, 0.01, 1), (1 << 20, 1 << 22, 0.01, 1), (1 << 20, 50_000_000, 0.001, 0),
                                               (1 << 20, 138_357_544, 0.01, 1), (1 << 20, 1 << 24, 1.0, 1), (1 << 21, 1 << 24, 0.1, 1),
                                               (1 << 22, 1 << 24, 0.01, 2), (1 << 22, 1 << 24, 1.0, 2), (1 << 26, 1 << 26, 0.01, 2), (1 << 28, 1 << 28, 0.01, 2),
                                               (1 << 28, 1 << 28, 1.0, 2), (1 << 20, 1 << 20, 1.0, 2), (1 << 21, 1 << 21, 0.1, 2), (1 << 28, 300_007, 0.01, 0)])
def test_form_of_the_random_k_decode(geo, part, D, ratio, form):
    """The form that measured fastest (or within a few per cent of it) at these shapes: draws made again for
    stretches of 4096 or 32768 elements, or a fill and a scatter where that would grow with the square of the partition."""
    most = min(part, D)
    assert geo.geo_randk_decode_form(-(-D // part), most, max(1, int(ratio * most))) == form
