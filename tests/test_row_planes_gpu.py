"""GPU parity of the tiled kernels: row-major planes through LDS, token tiles cut down to the batch."""
import ctypes

import numpy as np
import pytest

from paper_2506_02024_amd import workloads
from helpers import NESTED_ROWS, bits, tile_height, to_dev
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
    knobs = {"small_max_m": 0, "large_bm": bm, "large_bn": bn, "large_split": split, "large_height": 256 if M > 256 else -1}
    try:
        for k, v in knobs.items():
            nfp.tune(k, v)
        assert M <= 256 or tile_height(nfp, NESTED_ROWS, M, N, K) == bm
        run_both_modes(nfp, workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M),
                       "%d x %d, M=%d %s" % (N, K, M, knobs), check_plain=False)
    finally:
        for k in knobs:
            nfp.tune(k, -1)


@pytest.mark.parametrize("M,N,K,bn,split,height", [
    # token tiles of 256 cut down to 160, 192 and 224 tokens: first and last batch of each, several tiles, K-tails
    (97, 260, 64 * 3 + 16, 256, 1, 160), (160, 140, 64 * 5, 128, 1, 160), (161, 140, 64 * 8, 128, 2, 192), (192, 270, 64 * 4, 256, 1, 192),
    (193, 130, 64 * 21 + 32, 128, 1, 224), (224, 520, 64 * 12, 256, 2, 224), (225, 264, 64 * 4, 256, 1, 256),
    (257, 264, 64 * 6, 256, 1, 160), (385, 264, 64 * 9 + 48, 256, 1, 224), (449, 136, 64 * 4, 128, 1, 256), (620, 264, 64 * 22, 128, 2, 224), (777, 300, 64 * 2, 256, 1, 224),
])
def test_token_tiles_cut_down_to_the_batch(nfp, M, N, K, bn, split, height):
    # (up to 256 tokens by themselves, above pinned: there the height is the one that is priced lowest)
    knobs = {"small_max_m": 0, "large_bm": 256, "large_bn": bn, "large_split": split, "large_height": height if M > 256 else -1}
    try:
        for k, v in knobs.items():
            nfp.tune(k, v)
        assert tile_height(nfp, NESTED_ROWS, M, N, K) == height
        X, W = workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M)
        run_both_modes(nfp, X, W, "%d x %d, M=%d %s" % (N, K, M, knobs), check_plain=False)
        # the same tiles without the merge
        Xd, Wd = to_dev(X), to_dev(W)
        up, lo = nfp.decompose(Wd)
        assert np.array_equal(bits(nfp.gemm(Xd, up, lo, nfp.MODE_FP16)), bits(nfp.plain_gemm_fp16(Xd, nfp.pack_fp16(Wd))))
    finally:
        for k in knobs:
            nfp.tune(k, -1)


@pytest.mark.parametrize("M,N,K", [(65, 4096, 1024), (66, 300, 640), (128, 1536, 2064), (129, 640, 4096), (200, 2056, 1040), (255, 130, 5120), (256, 3000, 768)])
def test_short_batches_in_their_own_launch_shapes(nfp, M, N, K):
    # 65 ... 256 tokens with no knob set: every shape the launch may take fits the fixed scratch
    assert nfp.gemm_workspace_size(M, N, K, nfp.MODE_FP16) <= nfp.STATIC_SCRATCH_BYTES
    run_both_modes(nfp, workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M), "%d x %d, M=%d" % (N, K, M))


@pytest.mark.parametrize("M,N,K,split", [(65, 130, 64 * 3 + 16, 1), (130, 264, 64 * 9, 2), (192, 560, 64 * 20 + 48, 1), (200, 136, 64 * 16, 3), (256, 1040, 64 * 5, 1)])
def test_several_token_tiles_of_64(nfp, M, N, K, split):
    # packed weights that are not marked non-temporal: against the oracle, the row-major planes and packed FP16 weights
    knobs = {"large_bm": 64, "large_split": split}
    try:
        for k, v in knobs.items():
            nfp.tune(k, v)
        X, W = workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M)
        run_both_modes(nfp, X, W, "%d x %d, M=%d %s" % (N, K, M, knobs), check_plain=False)
        Xd, Wd = to_dev(X), to_dev(W)
        up, lo = nfp.decompose(Wd)
        assert np.array_equal(bits(nfp.gemm(Xd, up, lo, nfp.MODE_FP16)), bits(nfp.plain_gemm_fp16(Xd, nfp.pack_fp16(Wd))))
    finally:
        for k in knobs:
            nfp.tune(k, -1)
