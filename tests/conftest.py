import ctypes as C
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def orc():
    import oracle
    oracle.build()
    return oracle


@pytest.fixture(scope="session")
def geo(tmp_path_factory):
    """csrc/geometry.hpp compiled for the host."""
    so = str(tmp_path_factory.mktemp("geo") / "host_geometry.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-o", so,
                    os.path.join(ROOT, "tests", "host_geometry.cpp")], check=True)
    L = C.CDLL(so)
    for name, args, res in [("geo_tiles", [C.c_uint64], C.c_uint32), ("geo_tile_elems", [], C.c_uint32),
                            ("geo_row_elems", [], C.c_uint32), ("geo_row_in_record", [C.c_uint32, C.c_uint64], C.c_uint32),
                            ("geo_lans_tile", [], C.c_uint32), ("geo_find_block", [C.c_void_p, C.c_uint64, C.c_uint64], C.c_int64),
                            ("geo_tile_edge", [C.c_uint64, C.c_uint64], C.c_uint64),
                            ("geo_block_tiles", [C.c_uint64, C.c_uint64, C.c_uint64, C.c_void_p, C.c_void_p], None),
                            ("geo_topk_state", [C.c_void_p, C.c_uint64], C.c_uint64),
                            ("geo_prep_rows", [C.c_uint32, C.c_uint32, C.c_uint32, C.c_int, C.c_void_p], None),
                            ("geo_sample_chunks", [C.c_uint32], C.c_uint32),
                            ("geo_topk_list_fits", [C.c_uint64, C.c_uint32], C.c_int),
                            ("geo_randk_decode_form", [C.c_uint64, C.c_uint64, C.c_uint64], C.c_int),
                            ("geo_sample_rank", [C.c_uint64, C.c_uint32, C.c_uint32], C.c_uint32), ("geo_topk_list_cap", [], C.c_uint32)]:
        getattr(L, name).argtypes, getattr(L, name).restype = args, res
    return L
