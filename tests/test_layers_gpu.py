"""GPU parity: exception layers (Sec. 4.1 "Handling Exception Layers") keep their FP16 weights
and run the FP16 GEMM in both modes; applicable layers follow the requested mode."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_02024_amd import workloads
from helpers import assert_gemm_close, bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfp():
    from paper_2506_02024_amd import binding

    return binding


@pytest.mark.parametrize("packed", [False, True], ids=["rowmajor", "packed"])
@pytest.mark.parametrize("M", [8, 200])
def test_planted_outlier_makes_an_exception_layer(nfp, M, packed):
    N, K = 272, 1040
    W = workloads.weight_host(N, K, seed=5)
    W_bad = W.copy()
    W_bad[137, 555] = np.float16(2.5)                  # one weight past the 1.75 bound
    W_bad[3, 0] = np.float16(-1.8125)
    X = workloads.act_host(M, K, seed=6)
    Xd = to_dev(X)
    good, bad = nfp.Layer(to_dev(W), packed=packed), nfp.Layer(to_dev(W_bad), packed=packed)
    assert not good.is_exception and good.out_of_range == 0
    assert bad.is_exception and bad.out_of_range == 2 and bad.upper is None

    ref_bad = oracle.gemm_fp16(X, W_bad)
    plain = bits(nfp.plain_gemm_fp16(Xd, to_dev(W_bad)))
    for mode in (nfp.MODE_FP16, nfp.MODE_FP8):
        y = nfp.linear(Xd, bad, mode)
        assert_gemm_close(y.cpu().numpy(), ref_bad, "exception layer, mode %d" % mode)
        assert np.array_equal(bits(y), plain)          # the FP16 kernel, whatever the mode

    # the applicable layer follows the mode: identical to nestedfp_gemm on its planes
    for mode in (nfp.MODE_FP16, nfp.MODE_FP8):
        y = nfp.linear(Xd, good, mode)
        z = nfp.gemm(Xd, good.upper, None if mode == nfp.MODE_FP8 else good.lower, mode)
        assert np.array_equal(bits(y), bits(z))
    up, _, _ = oracle.decompose(W)
    Xq, sc = oracle.quantize_act(X)
    assert_gemm_close(nfp.linear(Xd, good, nfp.MODE_FP8).cpu().numpy(), oracle.gemm_fp8(Xq, sc, up), "FP8 mode")


def test_mixed_stack_switches_only_the_applicable_layers(nfp):
    # a small "model": four linears, one of them an exception; per-step mode switching
    K = 512
    Ws = [workloads.weight_host(256, K, seed=20 + i) for i in range(4)]
    Ws[2][10, 10] = np.float16(3.0)
    layers = [nfp.Layer(to_dev(w), packed=(i % 2 == 1)) for i, w in enumerate(Ws)]
    assert [l.is_exception for l in layers] == [False, False, True, False]
    X = workloads.act_host(16, K, seed=9)
    Xd = to_dev(X)
    out16 = [bits(nfp.linear(Xd, l, nfp.MODE_FP16)) for l in layers]
    out8 = [bits(nfp.linear(Xd, l, nfp.MODE_FP8)) for l in layers]
    assert np.array_equal(out16[2], out8[2])           # exception layer: same result in both modes
    for i in (0, 1, 3):
        assert not np.array_equal(out16[i], out8[i])   # the others really change precision
        assert_gemm_close(out16[i].view(np.float16), oracle.gemm_fp16(X, Ws[i]), "layer %d" % i)


@pytest.mark.parametrize("mode", ["global", "thread_local"])
def test_loader_thread_beside_a_capture(nfp, mode):
    # a thread that has prepared layers ends while another one captures a graph; where the capture leaves other
    # threads alone ("thread_local"; a "global" one forbids them to wait for a stream), it starts
    # and prepares its layers during the capture as well.  Neither side may break the other.
    import threading
    import time

    N, K, M = 272, 1040, 16
    W = workloads.weight_host(N, K, seed=50)
    W_bad = W.copy()
    W_bad[7, 9] = np.float16(2.0)
    Xd, Wd, Wd_bad = to_dev(workloads.act_host(M, K, seed=51)), to_dev(W), to_dev(W_bad)
    layer = nfp.Layer(Wd)
    out = torch.zeros((M, N), dtype=torch.float16, device="cuda:0")
    ws = nfp.new_workspace(nfp.gemm_workspace_size(M, N, K, nfp.MODE_FP16), "cuda:0")
    nfp.linear(Xd, layer, nfp.MODE_FP16, out=out, workspace=ws)
    torch.cuda.synchronize()
    want = bits(out)
    got, errors = [], []
    side = torch.cuda.Stream()
    loaded, end = threading.Event(), threading.Event()

    def load():
        try:
            with torch.cuda.stream(side):
                got.extend([nfp.Layer(Wd), nfp.Layer(Wd_bad), nfp.Layer(Wd, packed=True)])
        except Exception as e:                             # reported by the main thread
            errors.append(e)
        loaded.set()
        end.wait(60)

    t = threading.Thread(target=load)
    if mode == "global":
        t.start()
        assert loaded.wait(60)
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        nfp.linear(Xd, layer, nfp.MODE_FP16, out=out, workspace=ws)
        if mode != "global":
            t.start()
            assert loaded.wait(60)
        end.set()
        t.join()
        time.sleep(0.2)                                    # the native thread is gone too
        nfp.linear(Xd, layer, nfp.MODE_FP16, out=out, workspace=ws)
    assert not errors, errors
    assert [l.out_of_range for l in got] == [0, 1, 0]
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits(out), want)
    assert np.array_equal(bits(nfp.linear(Xd, got[0], nfp.MODE_FP16)), want)


def test_counts_of_many_threads_at_once(nfp):
    # out-of-range counts are handed over through a fixed number of host words: more threads than words,
    # each with a count of its own
    from concurrent.futures import ThreadPoolExecutor

    N, K = 64, 256
    mats = []
    for i in range(8):
        W = workloads.weight_host(N, K, seed=60 + i)
        W.reshape(-1)[:3 * i] = np.float16(-1.875)
        mats.append(to_dev(W))
    torch.cuda.synchronize()
    with ThreadPoolExecutor(max_workers=80) as pool:
        counts = list(pool.map(lambda j: nfp.range_check(mats[j % 8]), range(800)))
    assert counts == [3 * (j % 8) for j in range(800)]


def test_a_replaced_description_is_the_one_that_counts():
    # Layer.c, the struct that the library reads, may be exchanged: shape and linear() follow it
    from paper_2506_02024_amd import binding as nfp

    a, b = (nfp.Layer(to_dev(workloads.weight_host(N, K, seed=N))) for N, K in ((48, 128), (80, 256)))
    X = to_dev(workloads.act_host(3, 256, seed=1))
    want = nfp.linear(X, b, nfp.MODE_FP16)
    a.c = b.c
    assert a.shape == (80, 256) and torch.equal(nfp.linear(X, a, nfp.MODE_FP16), want)
    bare = nfp.Layer.__new__(nfp.Layer)
    bare.c = b.c
    assert bare.shape == (80, 256) and torch.equal(nfp.linear(X, bare, nfp.MODE_FP16), want)
    with pytest.raises(AttributeError):
        a.shape = (1, 2)
