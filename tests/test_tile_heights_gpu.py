"""GPU: token tiles of every height give the same bits, in all kinds, with batches that end in every part of a tile."""
import numpy as np
import pytest

import oracle
from paper_2506_02024_amd import workloads
from helpers import assert_gemm_close, bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfp():
    from paper_2506_02024_amd import binding

    return binding


# the last tile of each height: one token, all but one, whole, one 16- or 32-token block and a bit
@pytest.mark.parametrize("M,N,K,bn,split", [(321, 300, 448, 256, 1), (479, 257, 208, 256, 1), (672, 520, 1040, 256, 3), (561, 131, 272, 256, 1),
                                            (385, 140, 704, 128, 2), (449, 389, 144, 128, 1), (960, 256, 128, 256, 1)])
def test_heights_of_token_tiles_change_nothing(nfp, M, N, K, bn, split):
    X, W = workloads.act_host(M, K, seed=N), workloads.weight_host(N, K, seed=M)
    Xd, Wd = to_dev(X), to_dev(W)
    up, lo = nfp.decompose(Wd)
    packed, wp = nfp.decompose(Wd, packed=True), nfp.pack_fp16(Wd)
    pins = {"large_bm": 256, "large_bn": bn, "large_split": split}
    first = None
    for height in (256, 224, 192, 160):
        for k, v in dict(pins, large_height=height).items():
            nfp.tune(k, v)
        try:
            got = [bits(nfp.gemm(Xd, up, lo, nfp.MODE_FP16)), bits(nfp.gemm(Xd, packed[0], packed[1], nfp.MODE_FP16)),
                   bits(nfp.plain_gemm_fp16(Xd, Wd)), bits(nfp.plain_gemm_fp16(Xd, wp)),
                   bits(nfp.gemm(Xd, up, None, nfp.MODE_FP8)), bits(nfp.gemm(Xd, packed[0], None, nfp.MODE_FP8))]
        finally:
            for k in list(pins) + ["large_height"]:
                nfp.tune(k, -1)
        if first is None:
            first = got
            assert_gemm_close(got[0].view(np.float16), oracle.gemm_fp16(X, W), "FP16 mode")
            Xq, s = oracle.quantize_act(X)
            assert_gemm_close(got[4].view(np.float16), oracle.gemm_fp8(Xq, s, oracle.decompose(W)[0]), "FP8 mode")
        for a, b in zip(got, first):
            assert np.array_equal(a, b), height
    for a in first[1:4]:
        assert np.array_equal(a, first[0])                 # both orders of the planes, and the plain weights
    assert np.array_equal(first[4], first[5])
