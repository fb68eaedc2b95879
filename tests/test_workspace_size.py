"""The rule that sizes a context's DCT tile lists up front, against the number of
tiles that every smaller map takes (host arithmetic of the library, no GPU)."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2203_13675_amd", "liblp_unwrap.so")


@pytest.fixture(scope="module")
def rules():
    if not os.path.exists(LIB):
        from paper_2203_13675_amd import build_lib
        build_lib.build()
    lib = ctypes.CDLL(LIB)
    side = lib["_ZN3lpu8dct_sideEiib"]  # lpu::dct_side(int, int, bool)
    side.argtypes, side.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_bool], ctypes.c_int
    most = lib["_ZN3lpu14dct_tiles_mostEii"]  # lpu::dct_tiles_most(int, int)
    most.argtypes, most.restype = [ctypes.c_int, ctypes.c_int], ctypes.c_int
    return side, most


@pytest.mark.parametrize("M,N", [(1, 1), (40, 7000), (31, 33), (480, 640), (512, 384), (768, 768),
                                 (1024, 1024), (900, 1100), (2050, 1000), (64, 20000)])
def test_reserved_tiles_cover_every_smaller_map(rules, M, N):
    side, most = rules
    have = most(M, N)
    cut = lambda n: sorted({v for k in range(0, n + 33, 32) for v in (k, k + 1) if 1 <= v <= n} | {n})
    for m in cut(M):
        for n in cut(N):
            for fp64 in (False, True):
                t = side(m, n, fp64)
                assert t in (32, 64)
                assert -(-m // t) * -(-n // t) <= have, (m, n, fp64, t)
            assert -(-m // 64) * -(-n // 64) <= have, (m, n)
