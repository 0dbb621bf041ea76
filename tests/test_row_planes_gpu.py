"""GPU parity of the tiled kernel that brings row-major planes through LDS (pairs of K-tiles)."""
import ctypes

import pytest

from paper_2506_02024_amd import workloads
from test_gemm_gpu import run_both_modes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfp():
    from paper_2506_02024_amd import binding

    return binding


def through_lds(nfp, bm, bn, M, K, split):
    f = nfp.lib()._ZN3nfp16rows_through_ldsEiillli          # nfp::rows_through_lds
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 2 + [ctypes.c_int64] * 3 + [ctypes.c_int]
    return f(bm, bn, M, K, K, split)


@pytest.mark.parametrize("M,N,K,bm,bn,split,lds", [
    # rows on lines: one K-tile (half a pair), one pair, odd and even counts, N and M that end inside a tile
    (200, 260, 64 * 2, 256, 256, 1, True), (257, 250, 64 * 4, 256, 128, 1, True), (129, 300, 64 * 6, 128, 256, 1, True),
    (70, 130, 64 * 12, 128, 128, 1, True), (130, 130, 64 * 10, 128, 128, 1, False),
    # slices of a split: even, odd (a pair that is half past the slice; K-tile by K-tile), a shorter last one
    (300, 264, 64 * 24, 256, 256, 2, True), (260, 264, 64 * 26, 256, 128, 2, True), (100, 520, 64 * 6, 128, 256, 2, False),
    (90, 264, 64 * 40, 128, 128, 3, True), (256, 512, 64 * 10, 256, 256, 4, False),
    # rows that start inside lines, K that ends inside a chunk of a pair: 16, 48 and 80 columns past the last pair
    (250, 270, 64 * 20 + 16, 256, 256, 1, True), (512, 140, 64 * 36 + 48, 256, 128, 1, True), (128, 270, 64 * 28 + 80, 128, 256, 2, True),
    (65, 150, 64 * 24, 128, 128, 1, True), (77, 150, 64 * 25, 128, 128, 1, True), (300, 150, 64 * 19 + 16, 256, 128, 1, False),
])
def test_row_planes_through_lds(nfp, M, N, K, bm, bn, split, lds):
    # against the oracle, and bit for bit against packed planes, which no kernel of this kind reads
    assert through_lds(nfp, bm, bn, M, K, split) == lds
    knobs = {"small_max_m": 0, "large_bm": bm, "large_bn": bn, "large_split": split}
    try:
        for k, v in knobs.items():
            nfp.tune(k, v)
        run_both_modes(nfp, workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M),
                       "%d x %d, M=%d %s" % (N, K, M, knobs), check_plain=False)
    finally:
        for k in knobs:
            nfp.tune(k, -1)
