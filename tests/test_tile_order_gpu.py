"""GPU: the order in which workgroups take the tiles of eight and more token tiles (an eighth of them per XCD, by groups of
token tiles) computes every tile once: the bits of the plain launch order."""
import numpy as np
import pytest
import torch

from paper_2506_02024_amd import workloads
from helpers import NESTED_ROWS, bits, tile_height, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfp():
    from paper_2506_02024_amd import binding

    return binding


# token tiles x weight tiles: 8 x 1, 9 x 1 (eighths of 1 and 2 tiles), 9 x 3, 13 x 9, 17 x 2, 8 x 5 and 12 x 3 in slices of K, 25 x 1, and in
# tiles of 224, 192 and 160 tokens 9 x 5 (slices of K), 9 x 3, 11 x 2, 15 x 3
@pytest.mark.parametrize("M,N,bm,bn,split,tiles", [
    (1024, 100, 128, 128, 1, 8), (1025, 128, 128, 128, 1, 9), (1100, 300, 128, 128, 1, 9), (1600, 1100, 128, 128, 1, 13), (2049, 512, 128, 256, 1, 17),
    (2000, 1050, 256, 256, 2, 8), (3070, 300, 256, 128, 3, 12), (6400, 200, 256, 256, 1, 25),
    (2000, 1050, 224, 256, 2, 9), (1600, 600, 192, 256, 1, 9), (1700, 500, 160, 256, 1, 11), (2700, 300, 192, 128, 1, 15)])
def test_order_of_eight_and_more_token_tiles(nfp, M, N, bm, bn, split, tiles):
    K = 512
    Wd, Xd = to_dev(workloads.weight_host(N, K, seed=N)), to_dev(workloads.act_host(M, K, seed=M))
    up, lo = nfp.decompose(Wd)
    packed = nfp.decompose(Wd, packed=True)
    pins = {"large_bm": 256 if bm > 128 else 128, "large_bn": bn, "large_split": split, "large_height": bm if bm > 128 else -1}
    outs = {}
    for order in (0, -1):
        for k, v in dict(pins, large_xcd_map=order).items():
            nfp.tune(k, v)
        try:
            assert -(-M // tile_height(nfp, NESTED_ROWS, M, N, K)) == tiles
            outs[order] = [bits(nfp.gemm(Xd, up, lo, nfp.MODE_FP16)), bits(nfp.gemm(Xd, packed[0], packed[1], nfp.MODE_FP16)),
                           bits(nfp.plain_gemm_fp16(Xd, Wd)), bits(nfp.gemm(Xd, up, None, nfp.MODE_FP8))]
        finally:
            for k in list(pins) + ["large_xcd_map"]:
                nfp.tune(k, -1)
    for a, b in zip(outs[0], outs[-1]):
        assert np.array_equal(a, b)
    assert not (outs[0][0] == 0).all(axis=1).any()     # (and no row is left out)
