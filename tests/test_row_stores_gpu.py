"""GPU parity of the tiled kernels' stores to output rows that start anywhere: every distance of a row's start from 16
bytes, rows that end inside the last 16 bytes, at them, and in the first 16 of a tile."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_02024_amd import workloads
from helpers import NESTED_ROWS, assert_gemm_close, bits, tile_height, to_dev

pytestmark = pytest.mark.gpu

FILL = 7.0


@pytest.fixture(scope="module")
def nfp():
    from paper_2506_02024_amd import binding

    return binding


@pytest.mark.parametrize("M,N,bm,bn", [(130, 257, 256, 256), (70, 255, 128, 256), (65, 131, 256, 128), (129, 250, 128, 128),
                                       (64, 385, 64, 128), (385, 519, 256, 256), (200, 3, 256, 128)])
@pytest.mark.parametrize("mode", ["fp16", "fp8", "plain"])
def test_rows_that_start_anywhere(nfp, M, N, bm, bn, mode):
    # against the oracle, and the same bits whatever 16 bytes the rows start in; nothing beside the rows is written
    K = 144
    X, W = workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M)
    up, lo, bad = oracle.decompose(W)
    assert bad == 0
    Xd, Wd, upd, lod = to_dev(X), to_dev(W), to_dev(up), to_dev(lo)
    if mode == "fp8":
        Xq, s = oracle.quantize_act(X)
        ref = oracle.gemm_fp8(Xq, s, up)
    else:
        ref = oracle.gemm_fp16(X, W)
    knobs = {"small_max_m": 0, "large_bm": bm, "large_bn": bn, "large_split": 1, "large_height": 256 if M > 256 else -1}
    try:
        for k, v in knobs.items():
            nfp.tune(k, v)
        assert M <= 256 or tile_height(nfp, NESTED_ROWS, M, N, K) == bm
        first = None
        for offset in (0, 1, 2, 4, 7):
            for ld in (N, (N + 7) // 8 * 8, N + 3):
                buf = torch.full((M * ld + 16,), FILL, dtype=torch.float16, device="cuda:0")
                y = torch.as_strided(buf, (M, N), (ld, 1), offset)
                if mode == "plain":
                    nfp.plain_gemm_fp16(Xd, Wd, out=y)
                else:
                    nfp.gemm(Xd, upd, lod, nfp.MODE_FP8 if mode == "fp8" else nfp.MODE_FP16, out=y)
                got = bits(y)
                if first is None:
                    first = got
                    assert_gemm_close(y.cpu().numpy(), ref, "%s M=%d N=%d %s" % (mode, M, N, knobs))
                assert np.array_equal(got, first), (offset, ld)
                y.fill_(FILL)
                assert bool((buf == FILL).all()), (offset, ld)
    finally:
        for k in knobs:
            nfp.tune(k, -1)
