"""Rules that choose between launches of the tiled kernels, at sizes where the choice was timed.  Needs no GPU."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def L():
    from paper_2506_02024_amd import binding, build

    if build.is_stale():
        build.build_library()
    return binding.lib()


def through_lds(L, bm, bn, M, K, split):
    f = L._ZN3nfp16rows_through_ldsEiillli                    # nfp::rows_through_lds
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 2 + [ctypes.c_int64] * 3 + [ctypes.c_int]
    return f(bm, bn, M, K, K, split)


@pytest.mark.parametrize("bm,bn,M,K,split,lds", [
    # odd slices of rows on lines, microseconds through LDS and straight into registers: 170.7 / 158.7, 165.7 / 152.4, 339.7 / 318.7
    (256, 256, 1024, 14336, 3, False), (256, 256, 900, 14336, 3, False), (256, 256, 900, 32768, 3, False),
    # even ones and whole rows: 181.0 / more, 171.8 / 169.1 (2048 tokens: one of the few that lose 2 %); smaller tiles: 184.2 / 192.8
    (256, 256, 1024, 14336, 2, True), (256, 256, 2048, 6400, 1, True), (256, 128, 1024, 14336, 3, True),
])
def test_how_row_major_planes_reach_a_tile(L, bm, bn, M, K, split, lds):
    assert through_lds(L, bm, bn, M, K, split) == lds
