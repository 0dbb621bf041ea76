"""GPU: the short conversion of rows with their own scale gives the codes of the division, in the stand-alone kernels and in
the streaming kernel at 9 to 16 tokens."""
import numpy as np
import pytest
import torch

from paper_2506_02024_amd import workloads
from helpers import bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfp():
    from paper_2506_02024_amd import binding

    return binding


# one wave and 16, one chunk per lane and two, both kernels; rows of 8 chunks
@pytest.mark.parametrize("M,K,onepass", [(700, 2048, -1), (700, 2048, 0), (64, 16384, 1), (33, 16, -1), (90, 9232, -1)])
def test_codes_of_many_row_maxima(nfp, M, K, onepass):
    # correctly rounded binary32 quotients, so the codes are equal, not close
    rng = np.random.default_rng(K + M)
    top = rng.integers(1, 0x7c00, size=(M, 1))
    top[0, 0], top[1, 0], top[2, 0] = 0x7bff, 1, 0x5f00    # 65504, the smallest subnormal, 448 (a scale of one: ties)
    x = rng.integers(0, 0x10000, size=(M, K)) % (top + 1) | rng.integers(0, 2, size=(M, K)) << 15
    x[:, K // 2] = top[:, 0]
    x[3, :] = 0x8000                                       # no more than negative zeros
    X = torch.from_numpy(x.astype(np.uint16).view(np.float16))
    amax = X.float().abs().amax(dim=1, keepdim=True)
    scale = torch.where(amax == 0, torch.ones_like(amax), amax / 448.0)
    want = (X.float() / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    nfp.tune("quant_onepass", onepass)
    try:
        q, s = nfp.quantize_act(X.to("cuda:0"))
    finally:
        nfp.tune("quant_onepass", -1)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), scale.reshape(-1).numpy().view(np.uint32))
    assert np.array_equal(q.cpu().view(torch.uint8).numpy(), want.view(torch.uint8).numpy())


@pytest.mark.parametrize("M,N,K", [(9, 12304, 1296), (12, 12290, 2064), (16, 16400, 3584)])
@pytest.mark.parametrize("packed", [False, True], ids=["rowmajor", "packed"])
def test_streaming_kernel_quantises_9_to_16_tokens(nfp, M, N, K, packed):
    up, _ = nfp.decompose(to_dev(workloads.weight_host(N, K, seed=M)), packed=packed)
    X = workloads.act_host(M, K, seed=N)
    X[0] *= np.float16(300.0)
    X[M - 1, 5] = np.float16(65504.0)
    other = X.copy()
    other[8, K - 1], other[M // 2, 0] = np.float16(np.inf), np.float16(np.nan)
    for x in (X, other):
        got = {}
        for knob in (0, -1):
            nfp.tune("small_fuse_quant", knob)
            try:
                got[knob] = bits(nfp.gemm(to_dev(x), up, None, nfp.MODE_FP8))
            finally:
                nfp.tune("small_fuse_quant", -1)
        assert np.array_equal(got[0], got[-1])
