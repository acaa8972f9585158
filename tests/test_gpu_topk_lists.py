"""Top-k lists at the edges: keys at the top of the range, many messages of very many entries, equal magnitudes
beside the lists."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available()
    import gpu_util
    gpu_util.bpc.lib()
    return gpu_util


def same_records(orc, po, kind, got, ref, pe, D, ratio, nan=False):
    """Indices and values of every record."""
    stride, k_cap = orc.partition_stride(po), max(1, int(ratio * pe))
    for p in range(-(-D // pe)):
        k = max(1, int(ratio * min(pe, D - p * pe)))
        vals, size = 16 + 4 * (-(-k_cap // 4) * 4), 4 if kind == "topk" else 2
        a, b = got[p * stride:(p + 1) * stride], ref[p * stride:(p + 1) * stride]
        assert np.array_equal(a[:16 + 4 * k], b[:16 + 4 * k]), p
        va, vb = a[vals:vals + size * k], b[vals:vals + size * k]
        if nan:   # (which NaN is not said)
            t = np.float32 if kind == "topk" else np.float16
            assert np.array_equal(va.view(t), vb.view(t), equal_nan=True), p
        else:
            assert np.array_equal(va, vb), p


@pytest.mark.parametrize("kind", ["topk", "topk16"])
@pytest.mark.parametrize("ef", [True, False])
@pytest.mark.parametrize("pe,D,ratio,share", [(8192, 100, 0.05, 0.03), (8192, 8192 + 700, 1.0, 1.0), (32768, 32768, 0.25, 0.01), (32768, 32768, 0.25, 0.5)])
def test_topk_keys_at_the_top_of_the_range(gu, orc, kind, ef, pe, D, ratio, share):
    """Bit patterns 0x7fffffff and 0xffffffff in partitions whose guess is 0 (listed whole: all of a small one, or
    all but zeros).  They sort first like every NaN, and nothing is written past the records."""
    import torch
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio)
    rs = np.random.default_rng(D)
    bits = np.zeros(D, np.uint32)
    at = rs.choice(D, max(1, int(share * D)), replace=False)
    bits[at] = np.where(rs.random(at.size) < 0.5, 0x7fffffff, 0xffffffff)
    bits[rs.choice(D, 9, replace=False)] = np.float32(3.0).view(np.uint32)
    g, res = bits.view(np.float32), np.zeros(D, np.float32) if ef else None
    ref_res = None if res is None else res.copy()
    ref = orc.compress(po, g, ref_res)
    size, rd = bpc.payload_bytes(pb, D), gu.to_dev(res)
    pay, ws = torch.full((size + (1 << 20),), 0xA5, dtype=torch.uint8, device=gu.DEV), gu.new_ws(pb, D)
    bpc.bpc_compress(pb, gu.to_dev(g), rd, pay[:size], ws)
    bpc.workspace_check(pb, D, ws)
    assert bool((pay[size:] == 0xA5).all())
    same_records(orc, po, kind, gu.to_host(pay)[:size], ref, pe, D, ratio, nan=True)
    if ef:   # (a kept NaN leaves 0 behind, or what the difference of two NaNs is)
        assert np.array_equal(gu.to_host(rd)[~np.isnan(ref_res)], ref_res[~np.isnan(ref_res)])


@pytest.mark.parametrize("kind,pe,ratio,n,D", [("topk", 8_390_656, 1.0, 64, 3001), ("topk16", 8_390_656, 1.0, 63, 8193), ("topk", 8192, 0.01, 4, 300 * 8192 + 5),
                                               ("topk", 1024, 0.02, 64, 50 * 1024 + 77), ("topk16", 65536, 0.03, 17, 5 * 65536 + 9), ("topk", 1_048_576, 0.0019, 3, 1_048_576 + 8192)])
def test_topk_server_rows_of_sums_and_starts(gu, orc, kind, pe, ratio, n, D):
    """Messages of more entries than the rows of one launch take at once (64 messages of 8.4 M entries each at most; the
    gradient itself is short), of few entries (several to a row), and of just under and over a row's."""
    import torch
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio)
    rs = np.random.default_rng(n)
    kinds = [orc.compress(po, rs.standard_normal(D).astype(np.float32), None) for _ in range(min(n, 3))]
    dev = [gu.to_dev(m) for m in kinds]
    res = (rs.standard_normal(D) * 0.1).astype(np.float32)
    rd, pay = gu.to_dev(res), gu.new_payload(pb, D)
    ws = torch.empty(bpc.workspace_bytes(pb, D, n), dtype=torch.uint8, device=gu.DEV)
    bpc.bpc_server_aggregate([pb] * n, [dev[i % len(dev)] for i in range(n)], pb, rd, D, pay, ws)
    bpc.workspace_check(pb, D, ws)
    ref = orc.server_aggregate([po] * n, [kinds[i % len(kinds)] for i in range(n)], po, res, D)
    assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
    same_records(orc, po, kind, gu.to_host(pay), ref, pe, D, ratio)


def state_words(gu, geo, prm, D, ws):
    """Word 1 of every partition's selection state after a call on `ws`: non-zero where the list did not do."""
    at = int(geo.geo_topk_state(ctypes.byref(prm), D))
    return gu.to_host(ws[at:at + 32 * -(-D // prm.part_elems)]).view(np.uint32).reshape(-1, 8)[:, 1]


@pytest.mark.parametrize("kind,dtype,ef", [("topk", np.float32, True), ("topk16", np.float16, False)])
@pytest.mark.parametrize("pe,D,ratio", [(1 << 20, (1 << 20) + 77, 1 / 64), (1 << 21, 1 << 21, 14_000.5 / (1 << 21)), (1 << 22, (1 << 22) + 8193, 1 / 256),
                                        (1 << 23, 1 << 23, 0.001), (1 << 23, 1 << 23, 0.0015), (1 << 23, (1 << 23) + 1, 1e-4), (12 << 20, 12 << 20, 0.001), (1 << 26, 5_000_011, 2e-4)])
def test_topk_on_either_side_of_what_a_list_holds(gu, orc, geo, kind, dtype, ef, pe, D, ratio):
    """Ordinary vectors whose lists would be too long are not left to the fallback: they take another form."""
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio)
    rs = np.random.default_rng(int(1 / ratio))
    g = rs.standard_normal(D).astype(dtype)
    res = (rs.standard_normal(D) * 0.1).astype(np.float32) if ef else None
    rd, pay, ws = gu.to_dev(res), gu.new_payload(pb, D), gu.new_ws(pb, D)
    bpc.bpc_compress(pb, gu.to_dev(g), rd, pay, ws)
    bpc.workspace_check(pb, D, ws)
    ref = orc.compress(po, g, res)
    if ef:
        assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
    same_records(orc, po, kind, gu.to_host(pay), ref, pe, D, ratio)
    assert not state_words(gu, geo, pb, D, ws).any()


def few_magnitudes(what, D, rs, k, pe):
    """Vectors of which more elements share one key than a list has room for, and that key decides what is kept."""
    v = np.where(rs.random(D) < 0.5, -0.75, 0.75).astype(np.float32)
    if what == "zeros":
        v[:] = 0.0
        v[::7] = -0.0
    elif what == "sixteen":
        v = (rs.integers(1, 17, D) * 0.0625 * rs.choice([-1.0, 1.0], D)).astype(np.float32)
    elif what == "rows":      # of 64 elements, few of them touched: fewer non-zeros than k
        v = np.where(np.repeat(rs.random(-(-D // 64)) < 0.4 * k / pe, 64)[:D], rs.standard_normal(D), 0.0).astype(np.float32)
    elif what == "below":      # the deciding key is met well before the sample's rank: its elements are listed with lower ones
        v = np.where(rs.random(D) < 1.25 * k / pe, 0.5, 0.25).astype(np.float32) * rs.choice(np.float32([-1.0, 1.0]), D)
        v[rs.choice(D, 50, replace=False)] = 2.0
    elif what == "group end":  # the last of the k is the last element of a group, with larger ones before and behind
        larger = min(k // 2, 100)
        v[:] = 0.25
        at = (k // 8192 + 1) * 8192
        keep = rs.choice(at - 1, k - larger - 1, replace=False)
        v[:at] = 0.125
        v[keep] = 0.25
        v[at - 1] = -0.25
        v[rs.choice(np.setdiff1d(np.arange(at + 8192), np.append(keep, at - 1)), larger, replace=False)] = 3.0
    return v


@pytest.mark.parametrize("kind,dtype,ef", [("topk", np.float32, True), ("topk16", np.float16, True), ("topk", np.float16, False), ("topk16", np.float32, False)])
@pytest.mark.parametrize("pe,D,ratio", [(65536, 3 * 65536 + 40_777, 0.01), (1 << 20, (1 << 20) + 300_007, 0.01), (1 << 21, (1 << 21) + 9, 0.001),
                                        (1 << 20, (1 << 20) + 300_007, 0.03), (1 << 19, (1 << 19) + 8192 * 5, 0.0625), (1 << 23, 1 << 23, 0.0005)])
@pytest.mark.parametrize("what", ["equal", "zeros", "sixteen", "rows", "below", "group end"])
def test_topk_ties_beside_the_lists(gu, orc, geo, kind, dtype, ef, pe, D, ratio, what):
    """One list a partition and a list a group, partitions of one share of the select pass and of several, of more than 4 M
    elements; the same vector twice, so that the second call starts from what the first left in the workspace."""
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio)
    rs = np.random.default_rng(D)
    v = few_magnitudes(what, D, rs, int(ratio * pe), pe).astype(dtype)
    ref_res = np.zeros(D, np.float32) if ef else None
    ref = orc.compress(po, v, ref_res)
    g, ws = gu.to_dev(v), gu.new_ws(pb, D)
    ws.fill_(0xFF)
    for _ in range(2):
        rd, pay = gu.to_dev(np.zeros(D, np.float32)) if ef else None, gu.new_payload(pb, D)
        bpc.bpc_compress(pb, g, rd, pay, ws)
        bpc.workspace_check(pb, D, ws)
        same_records(orc, po, kind, gu.to_host(pay), ref, pe, D, ratio)
        if ef:
            assert np.array_equal(gu.to_host(rd).view(np.uint32), ref_res.view(np.uint32))
        # kept beside the list or lists, or on them; not left to the long form
        assert state_words(gu, geo, pb, D, ws)[0] in ((0, 2) if what in ("sixteen", "below") else (2,))


@pytest.mark.parametrize("pe,D,ratio", [(1 << 20, (1 << 20) + 300_007, 0.01), (1 << 20, (1 << 20) + 300_007, 0.03), (1 << 23, 1 << 23, 0.0005)])
@pytest.mark.parametrize("what", ["equal", "zeros", "sixteen"])
def test_topk_server_ties_beside_the_lists(gu, orc, geo, pe, D, ratio, what):
    """Delta of few magnitudes: two messages whose entries cancel, and the residual."""
    bpc = gu.bpc
    po, pb = gu.both_params(orc, "topk", pe, k_ratio=ratio)
    rs = np.random.default_rng(D)
    g = rs.standard_normal(D).astype(np.float32)
    msgs = [orc.compress(po, s * g, None) for s in (np.float32(1.0), np.float32(-1.0))]
    res = few_magnitudes(what, D, rs, int(ratio * pe), pe)
    rd, pay, ws = gu.to_dev(res), gu.new_payload(pb, D), gu.new_ws(pb, D, 2)
    bpc.bpc_server_aggregate([pb] * 2, [gu.to_dev(m) for m in msgs], pb, rd, D, pay, ws)
    bpc.workspace_check(pb, D, ws)
    ref = orc.server_aggregate([po] * 2, msgs, po, res, D)
    assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
    same_records(orc, po, "topk", gu.to_host(pay), ref, pe, D, ratio)
    assert state_words(gu, geo, pb, D, ws)[0] == 2
