"""GPU parity: activations quantised inside the streaming kernel against the launch of its own, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2506_02024_amd import workloads
from helpers import bits, quantises_itself, to_dev

pytestmark = pytest.mark.gpu


def _activations(M, K, seed):
    X = workloads.act_host(M, K, seed=seed)
    X[:, ::7] *= np.float16(-1.0)
    X[0, :: max(1, K // 5)] = np.float16(-0.0)
    if M > 1:
        X[1, :] = 0                                       # scale 1
        X[1, K // 2] = np.float16(-0.0)
    if M > 2:
        X[2, :] = (X[2, :].astype(np.float32) * 2.0 ** -22).astype(np.float16)      # subnormals and zeros
    if M > 3:
        X[3, K - 1] = np.float16(65504.0)                 # one value decides the scale
    return X


@pytest.mark.parametrize("M,N,K", [(1, 17, 16), (2, 40, 48), (7, 250, 112), (8, 33, 1024), (8, 640, 3072), (5, 2064, 2048 + 16),
                                   (9, 100, 1040), (16, 300, 1280), (16, 70, 512 + 80), (4, 6144, 4096), (8, 5136, 5120)])
@pytest.mark.parametrize("packed", [False, True], ids=["rowmajor", "packed"])
def test_fused_quantisation_gives_the_same_bits(M, N, K, packed):
    from paper_2506_02024_amd import binding as nfp

    up, _ = nfp.decompose(to_dev(workloads.weight_host(N, K, seed=M)), packed=packed)
    X = _activations(M, K, N)
    cases = [X, X.copy()]
    cases[1][M - 1, K // 3] = np.float16(np.inf)          # rows that need the clamp
    cases[1][M // 2, 0] = np.float16(np.nan)
    sc = torch.tensor([0.0123], dtype=torch.float32, device="cuda:0")
    for i, x in enumerate(cases):
        xd = torch.zeros((M, K + 24), dtype=torch.float16, device="cuda:0")[:, 8:8 + K]      # strided rows
        xd.copy_(to_dev(x))
        for scale in (None, sc):
            got = {}
            for knob in (0, 1, -1):
                nfp.tune("small_fuse_quant", knob)
                try:
                    assert quantises_itself(nfp, M, N, K) == (knob != 0)          # (by default too at these sizes)
                    got[knob] = bits(nfp.gemm(xd, up, None, nfp.MODE_FP8, act_scale=scale))
                finally:
                    nfp.tune("small_fuse_quant", -1)
            assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[-1]), (i, scale is None)
            if i == 0:
                q, s = nfp.quantize_act(xd, static_scale=scale)
                assert np.array_equal(got[0], bits(nfp.gemm_fp8_prequantized(q, s, up)))
