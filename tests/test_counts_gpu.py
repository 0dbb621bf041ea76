"""Counts of out-of-range weights that calls wait for: several threads and streams at once, counters left at zero."""
import threading

import numpy as np
import pytest
import torch

from paper_2506_02024_amd import workloads
from helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [1, 8])
def test_waited_counts_of_several_threads(threads):
    from paper_2506_02024_amd import binding as nfp

    W = workloads.weight_host(48, 1040, seed=1)
    errors = []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(12):
                    n = (5 * t + 7 * i) % 23                 # none at all among them
                    Wb = W.copy()
                    Wb.reshape(-1)[np.arange(n) * 131] = np.float16(2.0 + t)
                    Wd = to_dev(Wb)
                    layer = nfp.Layer(Wd, packed=i % 2 == 1)
                    assert layer.out_of_range == n and layer.is_exception == (n > 0)
                    assert nfp.range_check(Wd) == n
                    assert nfp.decompose_count(Wd)[2] == n
        except BaseException as e:                       # noqa: BLE001 (shown by the assertion below)
            errors.append(e)

    pool = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert not errors, errors


def test_device_word_holds_the_count_with_and_without_a_wait():
    import ctypes

    from paper_2506_02024_amd import binding as nfp

    W = workloads.weight_host(33, 256, seed=2)
    W[7, ::50] = np.float16(3.0)
    Wd = to_dev(W)
    up, lo = nfp._new_planes(33, 256, Wd.device, False)
    host = ctypes.c_uint64(99)
    for wait in (True, False, True):
        cnt = torch.full((1,), -1, dtype=torch.int64, device="cuda:0")
        st = nfp.lib().nestedfp_decompose(Wd.data_ptr(), 33, 256, 256, up.data_ptr(), lo.data_ptr(), cnt.data_ptr(),
                                          ctypes.byref(host) if wait else None, nfp._stream())
        assert st == (nfp.ERR_RANGE if wait else nfp.OK)
        assert cnt.item() == 6 and (not wait or host.value == 6)
    # an empty layer clears the word
    assert nfp.lib().nestedfp_decompose(None, 0, 256, 256, None, None, cnt.data_ptr(), ctypes.byref(host), nfp._stream()) == nfp.OK
    assert cnt.item() == 0 and host.value == 0


def test_library_memory_on_side_streams_and_in_a_graph():
    # the library asks a stream for its device: streams of their own, and one that a graph is captured on
    from paper_2506_02024_amd import binding as nfp

    M, N, K = 40, 520, 14336
    Wd, X = to_dev(workloads.weight_host(N, K, seed=3)), to_dev(workloads.act_host(M, K, seed=4))
    up, lo = nfp.decompose(Wd)
    for mode in (nfp.MODE_FP16, nfp.MODE_FP8):
        ref = nfp.gemm(X, up, lo, mode)
        out = torch.zeros_like(ref)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            assert nfp.range_check(Wd) == 0
            nfp.gemm_static(X, up, lo, mode, out)
        side.synchronize()
        assert torch.equal(out, ref)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            nfp.gemm_static(X, up, lo, mode, out)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
