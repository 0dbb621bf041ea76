"""GPU: quantised activations whose rows start on 128-byte lines (a workspace of the size that the query names) and dense ones (a
workspace without that room, as programs that kept an older size have it) give the same bits."""
import numpy as np
import pytest

from paper_2506_02024_amd import workloads
from helpers import bits, to_dev

pytestmark = pytest.mark.gpu


def round256(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("M,N,K", [(12, 300, 2064), (33, 1040, 1040), (64, 520, 4112), (100, 257, 2176 + 16), (300, 600, 48), (577, 390, 1136), (1030, 256, 1152)])
@pytest.mark.parametrize("packed", [False, True], ids=["rowmajor", "packed"])
def test_padded_and_dense_rows_of_codes(M, N, K, packed):
    from paper_2506_02024_amd import binding as nfp

    up, _ = nfp.decompose(to_dev(workloads.weight_host(N, K, seed=M)), packed=packed)
    X = to_dev(workloads.act_host(M, K, seed=N))
    full = nfp.gemm_workspace_size(M, N, K, nfp.MODE_FP8)
    dense = full - round256(M * ((K + 127) // 128 * 128)) + round256(M * K)
    assert (dense < full) == (K % 128 != 0)
    got = []
    for size in (full, dense):
        ws = nfp.new_workspace(size, "cuda:0")
        ws.fill_(0x7f)                                     # NaN codes in the rows' ends
        ws[:16384].zero_()
        got.append(bits(nfp.gemm(X, up, None, nfp.MODE_FP8, workspace=ws)))
    assert np.array_equal(got[0], got[1]) and not (got[0] == 0).all(axis=1).any()
    q, s = nfp.quantize_act(X)
    assert np.array_equal(got[0], bits(nfp.gemm_fp8_prequantized(q, s, up)))
    if not packed:
        out = nfp.gemm(X, up, None, nfp.MODE_FP8)
        nfp.gemm_static(X, up, None, nfp.MODE_FP8, out)
        assert np.array_equal(got[0], bits(out))
