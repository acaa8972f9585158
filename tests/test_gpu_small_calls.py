"""Calls of few tiles per workgroup go without the launch that presets the slots of the
single-pass kernels (the slots carry a tag of the launch instead); calls recorded into a graph and
large calls take the preset form.  Both give the same bits, whatever an earlier call left in the
workspace."""
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


# one tile; a partition and a ragged one; several tiles a workgroup; the sizes around the rule's
# line (512 or 768 workgroups of 8192 elements, four tiles each), where the large form begins
@pytest.mark.parametrize("D", [777, 140_001, 6_000_003, 16_777_216, 16_785_409, 25_170_000])
@pytest.mark.parametrize("kind,n,dtype", [("sign", 4, "float32"), ("sign", 3, "float16"), ("dither", 8, "float32"),
                                          ("dither", 3, "float16"), ("natdither", 16, "float32"), ("dither5", 4, "float32")])
def test_tagged_and_preset_forms_agree(gu, kind, n, dtype, D):
    import torch
    bpc, dev = gu.bpc, gu.DEV
    pe = 2_097_152 if dtype == "float16" else 1_048_576
    kw = dict(levels=15 if kind == "dither5" else 4, seed=5) if kind != "sign" else {}
    code = gu.KIND_B["dither" if kind == "dither5" else kind]
    D &= ~1   # (odd numbers of halves: test_odd_numbers_of_halves_in_the_single_pass_workers)
    prm = bpc.make_params(code, pe, **kw)
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + n)
    g = (torch.randn(D, generator=gen, device=dev) * 1e-3).to(getattr(torch, dtype))
    e0 = torch.randn(D, generator=gen, device=dev) * 1e-4
    s0 = torch.randn(D, generator=gen, device=dev) * 1e-4
    e, s = e0.clone(), s0.clone()
    pay = torch.zeros(bpc.payload_bytes(prm, D), dtype=torch.uint8, device=dev)
    out = torch.zeros_like(pay)
    ws = torch.full((bpc.workspace_bytes(prm, D, n),), 0xFF, dtype=torch.uint8, device=dev)

    def calls():
        bpc.bpc_compress(prm, g, e, pay, ws)
        bpc.bpc_server_aggregate([prm] * n, [pay] * n, prm, s, D, out, ws)

    def restore():
        e.copy_(e0); s.copy_(s0); pay.zero_(); out.zero_()

    def snapshot():
        torch.cuda.synchronize()
        bpc.workspace_check(prm, D, ws)
        return [t.clone() for t in (e, s, pay, out)]

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls()   # on a workspace of arbitrary bytes
    torch.cuda.current_stream().wait_stream(side)
    first = snapshot()
    restore()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for _ in range(2):
        restore()
        graph.replay()
        for a, b in zip(snapshot(), first):
            assert torch.equal(a, b)
    for _ in range(2):   # eager again, over slots that hold the very values to come
        restore()
        calls()
        for a, b in zip(snapshot(), first):
            assert torch.equal(a, b)


# tiles of 8192 elements over 768 resident workgroups (16 workers) or 512 (8 workers, bit planes)
@pytest.mark.parametrize("kind,n,D,tagged", [("sign", 16, 6_291_456, True), ("sign", 16, 16_000_000, True), ("sign", 16, 17_000_000, False),
                                             ("sign", 4, 17_000_000, True), ("sign", 4, 25_165_825, False),
                                             ("natdither", 16, 16_000_000, True), ("natdither", 16, 17_000_000, False),
                                             ("dither", 16, 24_000_000, False), ("dither5", 16, 16_000_000, True),
                                             ("dither", 8, 16_777_216, True), ("dither", 8, 16_777_217, False)])
def test_server_calls_that_go_without_the_preset(gu, kind, n, D, tagged):
    """The launch tag stands in the second status word of a call that goes without the preset; the
    preset form leaves that word alone."""
    import torch
    bpc, dev = gu.bpc, gu.DEV
    kw = dict(levels=15 if kind == "dither5" else 4, seed=5) if kind != "sign" else {}
    prm = bpc.make_params(gu.KIND_B["dither" if kind == "dither5" else kind], 1_048_576, **kw)
    pay = torch.zeros(bpc.payload_bytes(prm, D), dtype=torch.uint8, device=dev)
    out = torch.zeros_like(pay)
    ws = torch.zeros(bpc.workspace_bytes(prm, D, n), dtype=torch.uint8, device=dev)
    s = torch.randn(D, device=dev) * 1e-4
    bpc.bpc_server_aggregate([prm] * n, [pay] * n, prm, s, D, out, ws)
    bpc.workspace_check(prm, D, ws)
    at = int(bpc.lib().bpc_workspace_status_offset(ctypes.byref(prm), D))
    assert bool(ws[at + 4:at + 8].any()) == tagged


def _long_form(gu, geo, prm, D, ws):
    """For which partitions of the last top-k call on `ws` the list alone did not do (ties are kept beside it, or the
    partition was left to the long form)."""
    at = int(geo.geo_topk_state(ctypes.byref(prm), D))
    words = gu.to_host(ws[at:at + 32 * -(-D // prm.part_elems)]).view(np.uint32).reshape(-1, 8)
    return words[:, 1] != 0


@pytest.mark.parametrize("kind", ["topk", "topk16"])
@pytest.mark.parametrize("pe,P,overrun", [(4096, 1301, ()), (65536, 131, (3, 40, 77, 129)), (65536, 70, (0, 41, 69)), (65536, 20, (7, 8))])
def test_topk_many_partitions(gu, orc, geo, kind, pe, P, overrun):
    """The select pass with one, two and four workgroups a partition (more than 128 partitions, 65 to
    128, fewer), and with more partitions than the device holds of its workgroups.  Partitions of equal
    magnitudes have more tied keys than the short list has room (32768), so their list alone does not
    do, that of the others of the same call does; in partitions of 4096 elements even equal
    magnitudes or zeros fit the list."""
    bpc = gu.bpc
    D = (P - 1) * pe + 1001
    po, pb = gu.both_params(orc, kind, pe, k_ratio=0.01)
    rs = np.random.default_rng(23)
    g = rs.standard_normal(D).astype(np.float32)
    e = (0.3 * rs.standard_normal(D)).astype(np.float32)
    for p in overrun if overrun else (3, 200, 257, 700, 1299):
        n = min(pe, D - p * pe)
        g[p * pe:(p + 1) * pe] = np.where(rs.random(n) < 0.5, -0.5, 0.5)
        e[p * pe:(p + 1) * pe] = 0.0
    zeros = 800 if not overrun else 10
    g[zeros * pe:(zeros + 1) * pe] = 0.0
    e[zeros * pe:(zeros + 1) * pe] = 0.0
    full = [p for p in overrun if min(pe, D - p * pe) > 32768] + ([zeros] if overrun else [])
    res_ref = e.copy()
    pay_ref = orc.compress(po, g, res_ref)
    rd, pay, ws = gu.to_dev(e), gu.new_payload(pb, D), gu.new_ws(pb, D)
    bpc.bpc_compress(pb, gu.to_dev(g), rd, pay, ws)
    bpc.workspace_check(pb, D, ws)
    pay_gpu = gu.to_host(pay)
    assert np.array_equal(gu.to_host(rd).view(np.uint32), res_ref.view(np.uint32))
    stride = orc.partition_stride(po)
    for p in range(P):
        k = max(1, int(0.01 * min(pe, D - p * pe)))
        a, b = pay_gpu[p * stride:(p + 1) * stride], pay_ref[p * stride:(p + 1) * stride]
        assert np.array_equal(a[:16 + 4 * k], b[:16 + 4 * k]), p
    assert np.flatnonzero(_long_form(gu, geo, pb, D, ws)).tolist() == sorted(full)


@pytest.mark.parametrize("n,dtype", [(1, np.float16), (4, np.float32), (8, np.float16), (16, np.float32)])
@pytest.mark.parametrize("pe", [1024, 5120])
def test_fp16_with_the_most_runs_in_one_launch(gu, orc, n, dtype, pe):
    """64 runs of alternating class (partitions smaller than a tile and of a tile and a remainder, an
    odd last one): messages, residuals and an Adam-style step against the oracle, bit for bit."""
    import torch
    bpc = gu.bpc
    D = 70 * pe - 3
    mask = np.array([0] * 4 + [1] * 4 + [0, 1] * 31, np.uint8)
    assert len(mask) == 70 and 1 + np.count_nonzero(np.diff(mask)) == 64
    po, pb = gu.both_params(orc, "fp16", pe, bypass=mask)
    rs = np.random.default_rng(pe + n)
    ws = gu.new_ws(pb, D, n)
    ws.fill_(0xFF)
    pays_ref, pays = [], []
    for i in range(n):
        g = (rs.standard_t(3.0, D) * 1e-3).astype(dtype)
        e = (rs.standard_normal(D) * 3e-4).astype(np.float32)
        rd = gu.to_dev(e)
        pays.append(gu.new_payload(pb, D))
        bpc.bpc_compress(pb, gu.to_dev(g), rd, pays[i], ws)
        bpc.workspace_check(pb, D, ws)
        pays_ref.append(orc.compress_bypass(po, mask, g, e))
        assert np.array_equal(gu.to_host(rd), e)
    s = (rs.standard_normal(D) * 1e-4).astype(np.float32)
    sd, out = gu.to_dev(s), gu.new_payload(pb, D)
    bpc.bpc_server_aggregate([pb] * n, pays, pb, sd, D, out, ws)
    bpc.workspace_check(pb, D, ws)
    out_ref = orc.server_aggregate_bypass([po] * n, pays_ref, po, mask, s, D)
    assert np.array_equal(gu.to_host(sd), s)
    dense = torch.zeros(D, device=gu.DEV)
    bpc.bpc_decompress(pb, out, dense)
    assert np.array_equal(gu.to_host(dense), orc.decompress_bypass(po, mask, out_ref, D))
    x, m, v = [(rs.standard_normal(D) * c).astype(np.float32) for c in (0.02, 3e-4, 1e-3)]
    v = v * v
    dx, dm, dv = gu.to_dev(x), gu.to_dev(m), gu.to_dev(v)
    hyper = (1e-3, 0.9, 0.999, 1e-8, 0.01, 3)
    bpc.bpc_adaptive_update(pb, out, dx, dm, dv, bpc.make_opt(bpc.OPT_ADAM, *hyper), ws)
    bpc.workspace_check(pb, D, ws)
    orc.adaptive_update_bypass(po, mask, out_ref, D, x, m, v, orc.make_opt(orc.OPT_ADAM, *hyper))
    for a, b in ((dx, x), (dm, m), (dv, v)):
        assert np.array_equal(gu.to_host(a), b)


@pytest.mark.parametrize("kind,n", [("topk", 1), ("topk16", 1), ("topk", 3)])
@pytest.mark.parametrize("pe,D", [(65536, 5 * 65536 + 40_001), (1_048_576, 1_048_576 + 300_007)])
def test_topk_of_magnitudes_close_together_stays_on_the_short_list(gu, orc, geo, kind, n, pe, D):
    """Magnitudes within 2^-14 of each other share one bin of the first two radix levels, with far more
    of them in it than the short list holds; the guess then goes down to the key itself."""
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=0.01)
    rs = np.random.default_rng(D + n)
    v = ((1.0 + rs.random(D) * 2.0 ** -14) * rs.choice([-1.0, 1.0], D)).astype(np.float32)
    keys = v.view(np.uint32) & 0x7fffffff
    assert np.unique(keys >> 10).size <= 2 and pe > 32768
    ws = gu.new_ws(pb, D, n)
    res = np.zeros(D, np.float32)
    pay = gu.new_payload(pb, D)
    rd = gu.to_dev(res)
    if n == 1:
        ref = orc.compress(po, v, res)
        bpc.bpc_compress(pb, gu.to_dev(v), rd, pay, ws)
    else:   # server: everything but the last bits of Delta comes from the residual
        res = v.copy()
        rd = gu.to_dev(res)
        zero = orc.compress(po, np.zeros(D, np.float32), None)
        ref = orc.server_aggregate([po] * n, [zero] * n, po, res, D)
        bpc.bpc_server_aggregate([pb] * n, [gu.to_dev(zero)] * n, pb, rd, D, pay, ws)
    bpc.workspace_check(pb, D, ws)
    assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
    stride = orc.partition_stride(po)
    got = gu.to_host(pay)
    for p in range(-(-D // pe)):
        k = max(1, int(0.01 * min(pe, D - p * pe)))
        assert np.array_equal(got[p * stride:p * stride + 16 + 4 * k], ref[p * stride:p * stride + 16 + 4 * k]), p
    assert not _long_form(gu, geo, pb, D, ws).any()


# partitions of one share and of several, larger than one workgroup takes alone (more than 4 M elements); values on
# a grid give a few entries equal to the threshold (up to 64 are ranked one by one) or hundreds
@pytest.mark.parametrize("kind", ["topk", "topk16"])
@pytest.mark.parametrize("pe,D,grid", [(65536, 3 * 65536 + 777, 512.0), (65536, 40 * 65536 + 9, 16.0), (1_048_576, 1_048_576 + 70_001, 4096.0),
                                       (1_048_576, 300_007, 64.0), (8_388_608, 8_388_608 + 5000, None)])
def test_topk_select_ties_and_shares(gu, orc, geo, kind, pe, D, grid):
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=0.001)
    rs = np.random.default_rng(D)
    g = rs.standard_normal(D).astype(np.float32)
    if grid is not None:
        g = np.round(g * grid) / np.float32(grid)
    else:
        g[pe:] = 0.0   # the ragged last partition: zeros that fit its list
    big = grid is None
    for zeros in ((False, True) if big else (False,)):
        if zeros:
            g[:pe] = np.where(np.arange(pe) % 1000 == 0, g[:pe], 0.0)   # fewer non-zeros than k: too long for the list
            g[:: 2000] = 0.0
        res = np.zeros(D, np.float32)
        ref = orc.compress(po, g, res)
        rd, pay, ws = gu.to_dev(np.zeros(D, np.float32)), gu.new_payload(pb, D), gu.new_ws(pb, D)
        ws.fill_(0xFF)
        bpc.bpc_compress(pb, gu.to_dev(g), rd, pay, ws)
        bpc.workspace_check(pb, D, ws)
        assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
        stride, got = orc.partition_stride(po), gu.to_host(pay)
        k_cap = max(1, int(0.001 * pe))
        for p in range(-(-D // pe)):
            k = max(1, int(0.001 * min(pe, D - p * pe)))
            vals = 16 + 4 * (-(-k_cap // 4) * 4)
            size = 4 if kind == "topk" else 2
            for a, b in ((0, 16 + 4 * k), (vals, vals + size * k)):
                assert np.array_equal(got[p * stride + a:p * stride + b], ref[p * stride + a:p * stride + b]), p
        if big:
            assert _long_form(gu, geo, pb, D, ws).tolist() == [zeros, False]


# the last half alone in a tile, at the start and in the middle of a thread's four, in each row of a tile
@pytest.mark.parametrize("kind,kw", [("sign", {}), ("dither", dict(levels=4)), ("dither", dict(levels=7, norm=1)), ("dither", dict(levels=31)),
                                     ("dither", dict(levels=15, norm=1)), ("natdither", dict(levels=4)), ("natdither", dict(levels=7, norm=1))])
@pytest.mark.parametrize("ef", [True, False])
def test_odd_numbers_of_halves_in_the_single_pass_workers(gu, orc, kind, kw, ef):
    import fmt
    bpc, pe = gu.bpc, 131072
    po, pb = gu.both_params(orc, kind, pe, seed=9, stream_id=3, **kw)
    rs = np.random.default_rng(17)
    for D in (1, 3, 2047, 2049, 4099, 8191, 8193, 16387, 131071, 131073, 2 * 131072 + 8192 * 3 + 6147):
        g = (rs.standard_t(3.0, D) * 1e-3).astype(np.float16)
        g[-1] = np.float16(0.25)   # (the largest by far: its loss would show in every norm)
        res = (rs.standard_normal(D) * 3e-4).astype(np.float32) if ef else None
        rd = gu.to_dev(res) if ef else None
        ref = orc.compress(po, g, res)
        pay, ws = gu.new_payload(pb, D), gu.new_ws(pb, D)
        bpc.bpc_compress(pb, gu.to_dev(g), rd, pay, ws)
        bpc.workspace_check(pb, D, ws)
        got, stride = gu.to_host(pay), orc.partition_stride(po)
        for p, d in enumerate(fmt.part_sizes(D, pe)):
            size = 16 + 4 * (-(-d // 32) if kind == "sign" else -(-d // 8))
            spans = [(0, size)]
            for t in range(bpc_planes(kind, kw)):
                at = 16 + 4 * (pe // 8) + t * 4 * (pe // 32)
                spans.append((at, at + 4 * -(-d // 32)))
            for a, b in spans:
                assert np.array_equal(got[p * stride + a:p * stride + b], ref[p * stride + a:p * stride + b]), (D, p, a)
        if ef:
            assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32)), D


def bpc_planes(kind, kw):
    return 0 if kind != "dither" else sum(kw["levels"] >> (3 + t) != 0 for t in range(3))


# stretches of 8192 (top-k) and 32768 elements (random-k): ends inside, at and just past one, in full and ragged partitions
@pytest.mark.parametrize("kind,ratio", [("topk", 0.01), ("topk", 1.0), ("topk", 1e-6), ("topk16", 0.03), ("randk", 0.01), ("randk", 0.3), ("randk", 1e-6)])
@pytest.mark.parametrize("pe,D", [(1024, 5 * 1024 + 1), (40960, 40960 + 8191), (65536, 2 * 65536 + 8193), (131072, 131072 + 32768), (131072, 32769)])
def test_decompress_of_the_sparse_kinds(gu, orc, kind, ratio, pe, D):
    import torch
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio, seed=11, stream_id=5, value_scale=-1.0)
    rs = np.random.default_rng(D)
    g = rs.standard_normal(D).astype(np.float32)
    pay = orc.compress(po, g, None)
    out = torch.full((D + 64,), 7.0, device=gu.DEV)
    bpc.bpc_decompress(pb, gu.to_dev(pay), out[:D])
    got, ref = gu.to_host(out), orc.decompress(po, pay, D)
    assert np.all(got[D:] == 7.0)
    if kind == "randk":   # (the adds of repeated draws come in any order: a few roundings of the sum)
        assert np.allclose(got[:D], ref, rtol=1e-6, atol=1e-6 * np.abs(ref).max())
    else:
        assert np.array_equal(got[:D], ref)


@pytest.mark.parametrize("kind", ["topk", "topk16"])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("pe,D,equal", [(65536, 3 * 65536 + 777, False), (65536, 3 * 65536 + 40_001, True), (1_048_576, 300_007, True)])
def test_topk_without_error_feedback(gu, orc, geo, kind, dtype, pe, D, equal):
    """Nothing but the lists is stored; a list that fails (equal magnitudes) is made up for from the gradient."""
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=0.01)
    rs = np.random.default_rng(D)
    g = rs.standard_normal(D).astype(dtype)
    if equal:
        g = np.where(rs.random(D) < 0.5, -0.75, 0.75).astype(dtype)
        g[-1] = 2.0
    ref = orc.compress(po, g, None)
    pay, ws = gu.new_payload(pb, D), gu.new_ws(pb, D)
    ws.fill_(0xFF)
    bpc.bpc_compress(pb, gu.to_dev(g), None, pay, ws)
    bpc.workspace_check(pb, D, ws)
    stride, got, k_cap = orc.partition_stride(po), gu.to_host(pay), max(1, int(0.01 * pe))
    for p in range(-(-D // pe)):
        k = max(1, int(0.01 * min(pe, D - p * pe)))
        vals, size = 16 + 4 * (-(-k_cap // 4) * 4), 4 if kind == "topk" else 2
        for a, b in ((0, 16 + 4 * k), (vals, vals + size * k)):
            assert np.array_equal(got[p * stride + a:p * stride + b], ref[p * stride + a:p * stride + b]), p
    assert _long_form(gu, geo, pb, D, ws).any() == equal


# k above 16384 with an error-feedback buffer or a plain gradient: a list for every 8192 elements
@pytest.mark.parametrize("kind,ef,n", [("topk", True, 1), ("topk16", True, 1), ("topk", False, 1), ("topk", True, 3)])
@pytest.mark.parametrize("pe,D,ratio", [(524288, 524288 + 1, 0.04), (524288, 2 * 524288 - 8192 + 5, 0.0625), (1_048_576, 300_007, 0.03), (1_048_576, 1_048_576 + 8192 * 9, 0.03)])
@pytest.mark.parametrize("what", ["normal", "ties", "narrow", "equal", "one layer"])
def test_topk_group_lists(gu, orc, geo, kind, ef, n, pe, D, ratio, what):
    """Forms of the distribution: ties at the threshold, magnitudes within 2^-14 of each other, all equal (kept
    beside the lists), and a stretch of a partition that holds most of what is listed (more than its groups'
    lists have room for)."""
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio)
    rs = np.random.default_rng(D)
    v = rs.standard_normal(D).astype(np.float32)
    if what == "ties":
        v = np.round(v * 64.0) / np.float32(64.0)
    elif what == "narrow":
        v = ((1.0 + rs.random(D) * 2.0 ** -14) * rs.choice([-1.0, 1.0], D)).astype(np.float32)
    elif what == "equal":
        v = np.where(rs.random(D) < 0.5, -0.75, 0.75).astype(np.float32)
    elif what == "one layer":
        v[30_000:46_384] *= np.float32(100.0)
    ws = gu.new_ws(pb, D, n)
    ws.fill_(0xFF)
    pay = gu.new_payload(pb, D)
    if n == 1:
        g = (v.astype(np.float16) if not ef and D % 2 else v)
        res = (rs.standard_normal(D) * 1e-3).astype(np.float32) if ef and what == "normal" else np.zeros(D, np.float32) if ef else None
        rd = gu.to_dev(res) if ef else None
        ref = orc.compress(po, g, res)
        bpc.bpc_compress(pb, gu.to_dev(g), rd, pay, ws)
    else:
        msgs = [orc.compress(po, (v * np.float32(0.5 + i)).astype(np.float32), None) for i in range(n)]
        res = v.copy()
        rd = gu.to_dev(res)
        ref = orc.server_aggregate([po] * n, msgs, po, res, D)
        bpc.bpc_server_aggregate([pb] * n, [gu.to_dev(m) for m in msgs], pb, rd, D, pay, ws)
    bpc.workspace_check(pb, D, ws)
    if ef:
        assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
    stride, got, k_cap = orc.partition_stride(po), gu.to_host(pay), int(ratio * pe)
    assert k_cap > 16384
    for p in range(-(-D // pe)):
        k = max(1, int(ratio * min(pe, D - p * pe)))
        vals, size = 16 + 4 * (-(-k_cap // 4) * 4), 4 if kind == "topk" else 2
        for a, b in ((0, 16 + 4 * k), (vals, vals + size * k)):
            assert np.array_equal(got[p * stride + a:p * stride + b], ref[p * stride + a:p * stride + b]), p
    if n == 1 and what != "ties" and not (what == "narrow" and not ef):
        assert bool(_long_form(gu, geo, pb, D, ws)[0]) == (what == "equal")


# small random-k calls make their draws again in every workgroup: one tile and several partitions, more hits in a
# tile than its list has room (k = d / 2), and sizes on either side of the rule (2 M / 4 M elements)
@pytest.mark.parametrize("pe,D,ratio,n", [(1024, 1000, 0.01, 2), (16384, 5 * 16384 + 4099, 0.5, 2), (16384, 8193, 1.0, 1), (131072, 131072 + 8192 * 3 + 1, 0.03, 8),
                                          (1_048_576, 1_048_576 + 70_001, 0.01, 3), (1_048_576, 4 * 1_048_576 + 3, 0.01, 3)])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_randk_small_and_large_calls(gu, orc, pe, D, ratio, n, dtype):
    import torch
    bpc = gu.bpc
    rs = np.random.default_rng(D)
    prm = [gu.both_params(orc, "randk", pe, k_ratio=ratio, seed=3, stream_id=100 + i, value_scale=1.0 if i == n else -1.0) for i in range(n + 1)]
    ws = gu.new_ws(prm[0][1], D, n)
    ws.fill_(0xFF)
    pays, close = [], lambda a, b: np.all(np.abs(a - b) <= 1e-6 * (np.abs(b) + np.abs(b).mean()))
    for i in range(n):
        g = (rs.standard_normal(D) * 1e-2).astype(dtype)
        res = (rs.standard_normal(D) * 1e-3).astype(np.float32)
        res0 = res.copy()
        rd, pay = gu.to_dev(res), gu.new_payload(prm[i][1], D)
        bpc.bpc_compress(prm[i][1], gu.to_dev(g), rd, pay, ws)
        bpc.workspace_check(prm[i][1], D, ws)
        ref = orc.compress(prm[i][0], g, res)
        pays.append(ref)
        _equal_randk(orc, prm[i][0], gu.to_host(pay), ref, pe, D, ratio, exact=True)
        assert _randk_residual_close(g.astype(np.float32) + res0, gu.to_host(rd), res, pe, ratio)
    s = (rs.standard_normal(D) * 1e-3).astype(np.float32)
    sd, out = gu.to_dev(s), gu.new_payload(prm[n][1], D)
    bpc.bpc_server_aggregate([p[1] for p in prm[:n]], [gu.to_dev(p) for p in pays], prm[n][1], sd, D, out, ws)
    bpc.workspace_check(prm[n][1], D, ws)
    ref = orc.server_aggregate([p[0] for p in prm[:n]], pays, prm[n][0], s, D)
    _equal_randk(orc, prm[n][0], gu.to_host(out), ref, pe, D, ratio, exact=False)
    assert np.abs(gu.to_host(sd) - s).max() <= 1e-6 * 40 * np.abs(s).max()
    x, m, v = [(rs.standard_normal(D) * c).astype(np.float32) for c in (0.02, 3e-4, 1e-3)]
    v = v * v
    dx, dm, dv = gu.to_dev(x), gu.to_dev(m), gu.to_dev(v)
    hyper = (1e-3, 0.9, 0.999, 1e-8, 0.01, 3)
    bpc.bpc_adaptive_update(prm[n][1], gu.to_dev(ref), dx, dm, dv, bpc.make_opt(bpc.OPT_ADAM, *hyper), ws)
    bpc.workspace_check(prm[n][1], D, ws)
    orc.adaptive_update(prm[n][0], ref, D, x, m, v, orc.make_opt(orc.OPT_ADAM, *hyper))
    for a, b in ((dx, x), (dm, m), (dv, v)):
        assert close(gu.to_host(a), b)


def _randk_residual_close(q, got, ref, pe, ratio):
    """The residual of random-k with scale d / k, got and the oracle's.  An element drawn m times has scale * q taken off
    it m times, on either side in some order: each difference rounds at 2^-24 of a partial result, of which none is
    larger than |q| + m scale |q|, and so does the product (2^-24 of scale |q|, m times the same)."""
    q = q.astype(np.float64)
    sizes = np.array([min(pe, q.size - p) for p in range(0, q.size, pe)])
    scale = np.repeat([d / max(1, int(ratio * d)) for d in sizes], sizes)
    off = np.abs(q - ref)                                   # m scale |q|
    m = np.round(off / np.maximum(scale * np.abs(q), 1e-45))
    bound = 2.0 ** -24 * (2 * m * (np.abs(q) + off) + off + np.abs(q)) * 1.01 + 1e-45
    return bool(np.all(np.abs(got.astype(np.float64) - ref) <= bound))


# k from a quarter of the partition on: tiles with more hits than their list has room for, which make their draws three
# times where that is worth it, and sizes that take the launch in front instead
@pytest.mark.parametrize("pe,D,ratio", [(8192, 9 * 8192 + 7, 1.0), (16384, 3 * 16384 + 5, 1.0), (16384, 40 * 16384 + 1, 1.0), (32768, 2 * 32768 + 100, 0.25),
                                        (4096, 5 * 4096 + 4095, 0.3)])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_randk_tiles_with_many_hits(gu, orc, pe, D, ratio, dtype):
    bpc = gu.bpc
    rs = np.random.default_rng(D)
    po, pb = gu.both_params(orc, "randk", pe, k_ratio=ratio, seed=3, stream_id=9, value_scale=-1.0)
    g, res = (rs.standard_normal(D) * 1e-2).astype(dtype), (rs.standard_normal(D) * 1e-3).astype(np.float32)
    q, rd, pay, ws = g.astype(np.float32) + res, gu.to_dev(res), gu.new_payload(pb, D), gu.new_ws(pb, D)
    bpc.bpc_compress(pb, gu.to_dev(g), rd, pay, ws)
    bpc.workspace_check(pb, D, ws)
    ref = orc.compress(po, g, res)
    _equal_randk(orc, po, gu.to_host(pay), ref, pe, D, ratio, exact=True)
    assert _randk_residual_close(q, gu.to_host(rd), res, pe, ratio)


def _equal_randk(orc, po, got, ref, pe, D, ratio, exact):
    stride = orc.partition_stride(po)
    for p in range(-(-D // pe)):
        k = max(1, int(ratio * min(pe, D - p * pe)))
        a, b = got[p * stride:p * stride + 16 + 4 * k], ref[p * stride:p * stride + 16 + 4 * k]
        assert np.array_equal(a[:16], b[:16]), p
        va, vb = a[16:].view(np.float32), b[16:].view(np.float32)
        assert np.array_equal(va, vb) if exact else np.abs(va - vb).max() <= 1e-6 * 40 * np.abs(vb).max(), p


# the search of an update call without a table, tiles of 4096 and 8192 elements: ends inside and on a tile, and a call
# of more tiles than the rule takes
@pytest.mark.parametrize("kind,ratio", [("topk", 0.01), ("topk16", 0.03), ("topk", 1.0), ("randk", 0.02)])
@pytest.mark.parametrize("pe,D", [(8192, 3 * 8192 + 1), (131072, 131072 + 4096), (131072, 32769), (1_048_576, 5 * 1_048_576 + 77)])
@pytest.mark.parametrize("opt", ["adam", "lans", "blocks"])
def test_sparse_updates_with_and_without_a_table(gu, orc, kind, ratio, pe, D, opt):
    import torch
    bpc = gu.bpc
    if ratio == 1.0 and D > 10 ** 6:
        pytest.skip("a message as large as the gradient adds nothing here")
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio, seed=2, stream_id=7)
    rs = np.random.default_rng(D)
    pay = orc.compress(po, rs.standard_normal(D).astype(np.float32), None)
    x, m, v = [(rs.standard_normal(D) * c).astype(np.float32) for c in (0.02, 3e-4, 1e-3)]
    v = v * v
    x0 = x.copy()
    dx, dm, dv = gu.to_dev(x), gu.to_dev(m), gu.to_dev(v)
    offs = np.unique(np.array([0, 1000, 9000, 9001, 30000, D], dtype=np.uint64).clip(0, D)) if opt == "blocks" else None
    nb = 0 if offs is None else len(offs) - 1
    hyper = (1e-3, 0.9, 0.999, 1e-8, 0.01, 3)
    kind_b, kind_o = (bpc.OPT_ADAM, orc.OPT_ADAM) if opt == "adam" else (bpc.OPT_LANS, orc.OPT_LANS)
    ob = bpc.make_opt(kind_b, *hyper, block_offsets=None if offs is None else torch.from_numpy(offs.astype("int64")).to(gu.DEV))
    oo = orc.make_opt(kind_o, *hyper) if offs is None else orc.make_opt(kind_o, *hyper, block_offsets=offs)
    ws = torch.full((max(bpc.workspace_bytes(pb, D, 1), bpc.update_workspace_bytes(pb, D, nb)),), 0xFF, dtype=torch.uint8, device=gu.DEV)
    bpc.bpc_adaptive_update(pb, gu.to_dev(pay), dx, dm, dv, ob, ws)
    bpc.workspace_check(pb, D, ws)
    orc.adaptive_update(po, pay, D, x, m, v, oo)
    tol = lambda a, b: np.all(np.abs(gu.to_host(a) - b) <= 1e-6 * (np.abs(b) + np.abs(b).mean()))
    assert tol(dm, m) and tol(dv, v) and tol(dx, x)
    if opt != "adam":
        edges = offs if offs is not None else np.unique(np.append(np.arange(0, D, pe), D))
        assert gu.lans_step_close(gu.to_host(dx), x, x0, blocks=edges)


# bit planes on the server: one to three planes, worker counts below, at and above the groups of four, ragged
# ends inside a thread's eight elements; the same call recorded into a graph (preset form) gives the same bytes
@pytest.mark.parametrize("n", [1, 3, 5, 16, 64])
@pytest.mark.parametrize("kw", [dict(levels=8), dict(levels=15, norm=1), dict(levels=16, norm=1), dict(levels=31), dict(levels=32), dict(levels=63, norm=1)])
@pytest.mark.parametrize("ef", [True, False])
def test_bit_planes_in_the_single_pass_server(gu, orc, n, kw, ef):
    import fmt
    import torch
    bpc, pe = gu.bpc, 16384
    po, pb = gu.both_params(orc, "dither", pe, seed=21, stream_id=4, **kw)
    rs = np.random.default_rng(n)
    for D in (1, 8191, 8193, 2 * 16384 + 8192 + 4099):
        msgs = [orc.compress(po, (rs.standard_normal(D) * 1e-3 * (i + 1)).astype(np.float32), None) for i in range(n)]
        res = (rs.standard_normal(D) * 3e-4).astype(np.float32) if ef else None
        rd, pays = gu.to_dev(res) if ef else None, [gu.to_dev(m) for m in msgs]
        res0 = rd.clone() if ef else None
        pay, ws = gu.new_payload(pb, D), gu.new_ws(pb, D, n)
        ws.fill_(0xFF)
        bpc.bpc_server_aggregate([pb] * n, pays, pb, rd, D, pay, ws)
        bpc.workspace_check(pb, D, ws)
        ref = orc.server_aggregate([po] * n, msgs, po, res, D)
        got, stride = gu.to_host(pay), orc.partition_stride(po)
        for p, d in enumerate(fmt.part_sizes(D, pe)):
            spans = [(0, 16 + 4 * -(-d // 8))] + [(16 + 4 * (pe // 8) + t * 4 * (pe // 32),) * 2 for t in range(bpc_planes("dither", kw))]
            for a, b in [spans[0]] + [(a, a + 4 * -(-d // 32)) for a, _ in spans[1:]]:
                assert np.array_equal(got[p * stride + a:p * stride + b], ref[p * stride + a:p * stride + b]), (D, p, a)
        if ef:
            assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32)), D
    res1, pay1 = rd.clone() if ef else None, pay.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bpc.bpc_server_aggregate([pb] * n, pays, pb, rd, D, pay, ws)
    for _ in range(3):
        if ef:
            rd.copy_(res0)
        pay.copy_(gu.new_payload(pb, D))
        graph.replay()
        torch.cuda.synchronize()
        bpc.workspace_check(pb, D, ws)
        assert torch.equal(pay, pay1) and (not ef or torch.equal(rd, res1))


# every form of the decode, on either side of its rules: partitions of 1024 to 4 M elements, few draws and many
@pytest.mark.parametrize("kind,ratio,pe,D", [("topk", 0.02, 1024, 9 * 1024 + 77), ("topk16", 0.5, 2048, 5 * 2048 + 1025), ("topk", 0.01, 3072, 3072 + 2049),
                                             ("randk", 0.01, 1024, 9 * 1024 + 77), ("randk", 0.01, 1 << 20, (1 << 20) + 4097), ("randk", 1.0, 5120, 3 * 5120 + 4095),
                                             ("randk", 0.01, 1 << 20, 5 * (1 << 20) + 77), ("randk", 0.1, 1 << 18, 9 * (1 << 18) + 32769),
                                             ("randk", 0.01, 1 << 22, 2 * (1 << 22) + 5), ("randk", 1.0, 1 << 20, (1 << 20) + 1), ("randk", 0.001, 1 << 26, 5_000_003)])
def test_decompress_forms(gu, orc, kind, ratio, pe, D):
    import torch
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio, seed=13, stream_id=6, value_scale=-1.0)
    g = np.random.default_rng(D).standard_normal(D).astype(np.float32)
    pay = orc.compress(po, g, None)
    out = torch.full((D + 64,), 7.0, device=gu.DEV)
    bpc.bpc_decompress(pb, gu.to_dev(pay), out[:D])
    got, ref = gu.to_host(out), orc.decompress(po, pay, D)
    assert np.all(got[D:] == 7.0)
    if kind == "randk":   # (repeated draws add in any order)
        assert np.allclose(got[:D], ref, rtol=1e-6, atol=1e-6 * np.abs(ref).max())
    else:
        assert np.array_equal(got[:D], ref)
