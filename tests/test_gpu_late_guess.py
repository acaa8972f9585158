"""Top-k calls whose guesses do not come.  The workgroups of the load pass wait for the guess of the key that lists
start from; the workgroup that is there to make it may be kept from running by another kernel that waits on
another stream.  Here the passes are compiled without those workgroups (late_guess.hip), so that every
partition is left to the long form by a workgroup that waited: the calls end, nothing gives up, and what they
give is the oracle's."""
import ctypes as C
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "_build", "liblate_guess.so")


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available()
    import gpu_util
    gpu_util.bpc.lib()
    return gpu_util


@pytest.fixture(scope="module")
def late():
    assert os.path.exists(LIB), "run __graft_entry__.build() first"
    L = C.CDLL(LIB)
    p = C.c_void_p
    L.late_compress.argtypes = [p, p, C.c_int, p, C.c_uint64, p, p, p]
    L.late_aggregate.argtypes = [p, p, C.c_int, p, C.c_uint64, p, p, p]
    return L


# one group and many, several partitions, a ragged last one; short lists, lists a group (k above 16384), a
# partition of more than 4 M elements
@pytest.mark.parametrize("kind,dtype,ef,n", [("topk", np.float32, True, 1), ("topk16", np.float16, True, 1), ("topk", np.float16, False, 1),
                                             ("topk", np.float32, True, 3), ("topk16", np.float32, False, 2)])
@pytest.mark.parametrize("pe,D,ratio", [(8192, 5000, 0.02), (65536, 40 * 65536 + 777, 0.01), (1_048_576, 2 * 1_048_576 + 70_001, 0.01),
                                        (1_048_576, 1_048_576 + 8192 * 9 + 1, 0.03), (8_388_608, 8_388_608 + 5001, 0.001)])
def test_calls_whose_guesses_do_not_come(gu, orc, late, kind, dtype, ef, n, pe, D, ratio):
    import torch
    bpc = gu.bpc
    po, pb = gu.both_params(orc, kind, pe, k_ratio=ratio)
    rs = np.random.default_rng(D + n)
    ws = gu.new_ws(pb, D, n)
    ws.fill_(0xFF)
    pay = gu.new_payload(pb, D)
    res = (rs.standard_normal(D) * 0.1).astype(np.float32) if ef else None
    rd = gu.to_dev(res)
    stream = torch.cuda.current_stream().cuda_stream
    ptr = lambda t: None if t is None else t.data_ptr()
    if n == 1:
        g = rs.standard_normal(D).astype(dtype)
        gd = gu.to_dev(g)
        err = late.late_compress(C.byref(pb), gd.data_ptr(), bpc.F16 if dtype == np.float16 else bpc.F32, ptr(rd), D, pay.data_ptr(), ws.data_ptr(), stream)
        ref = orc.compress(po, g, res)
    else:
        msgs = [orc.compress(po, rs.standard_normal(D).astype(np.float32), None) for _ in range(n)]
        pays = [gu.to_dev(m) for m in msgs]
        err = late.late_aggregate(C.byref(pb), (C.c_void_p * n)(*[p.data_ptr() for p in pays]), n, ptr(rd), D, pay.data_ptr(), ws.data_ptr(), stream)
        ref = orc.server_aggregate([po] * n, msgs, po, res, D)
    assert err == 0
    bpc.workspace_check(pb, D, ws)
    if ef:
        assert np.array_equal(gu.to_host(rd).view(np.uint32), res.view(np.uint32))
    stride, got, k_cap = orc.partition_stride(po), gu.to_host(pay), max(1, int(ratio * pe))
    for p in range(-(-D // pe)):
        k = max(1, int(ratio * min(pe, D - p * pe)))
        vals, size = 16 + 4 * (-(-k_cap // 4) * 4), 4 if kind == "topk" else 2
        for a, b in ((0, 16 + 4 * k), (vals, vals + size * k)):
            assert np.array_equal(got[p * stride + a:p * stride + b], ref[p * stride + a:p * stride + b]), p
