"""Times the launch shapes of the streaming kernel over many layers and fits the constants that the
library compiles in: kSmallCost (csrc/gemm_small.hip) and the lines between the streaming kernel and the
64-token tiles at 17 ... 64 tokens (kLine in csrc/nestedfp_api.hip).

    python -m paper_2506_02024_amd.fit_costs time candidates.jsonl routes.jsonl     # on the GPU, about 7 minutes
    python -m paper_2506_02024_amd.fit_costs fit candidates.jsonl routes.jsonl      # prints the constants

`time` writes one line per timing: [N, K, tokens, storage, [K-steps per wave, K split, tiles per workgroup],
us] and [N, K, tokens, storage, us of the tiled kernel, us of the streaming kernel].  Weights are cold (copies
taken in turn) and the calls are replayed as one graph.  storage: 16p / 16r the planes in FP16 mode, packed and
row-major, 8p / 8r the upper plane in FP8 mode on quantised activations, pr plain row-major FP16.
`fit` mirrors price_small() and choose_tile64() of the library.  The constants minimise the time lost to the
fastest candidate by a soft choice of the cheapest one, plus the error of the prices; the lines are searched on
a grid for the time lost to the faster kernel, prices as the library has them compiled in.
"""
import argparse
import ctypes
import json
import time

import numpy as np

from .tune_tiles import MODEL_SHAPES

# layers of other sizes: small ones, odd row counts, rows that start inside a line, wide and narrow ones
OTHER_SHAPES = [
    (256, 16384), (512, 512), (1024, 1024), (1024, 8192), (1040, 1040), (1040, 2768), (1280, 1280), (1280, 3840),
    (1280, 4224), (1408, 1408), (1536, 1024), (1536, 4352), (1560, 1040), (2048, 2048), (2304, 1152), (2304, 2304),
    (2432, 7104), (2944, 7360), (3072, 3072), (3072, 8192), (3200, 8448), (3328, 11520), (3424, 3424), (3760, 12208),
    (4039, 1344), (4096, 11008), (4480, 4480), (4608, 12928), (4688, 13312), (5312, 17344), (5504, 18944),
    (5544, 1040), (5632, 5632), (5696, 5696), (5840, 5840), (6112, 3056), (6400, 22784), (7680, 7680), (8480, 1440),
    (11520, 3840), (12288, 4096), (14208, 2656), (14336, 4096), (16128, 5376), (17616, 5872), (22016, 4096),
    (23424, 7808), (28128, 5424), (37376, 5632), (43038, 5984), (54667, 8000), (128256, 4096)]
STORAGES = ("16p", "16r", "8p", "8r", "pr")
SPLITS = (1, 2, 3, 4, 6, 8)
TILES = (1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16)
CANDIDATE_TOKENS = (1, 8, 16, 24, 32, 64)
ROUTE_TOKENS = (17, 20, 24, 28, 32, 33, 40, 48, 56, 64)


def geometry(N, K, M, storage, spw, split, per):
    """What price_small() derives from a launch shape; None if the library would not launch it so."""
    kstep = 128 if storage[0] == "8" else 64
    mt = 1 if M <= 16 else (2 if M <= 32 else 4)
    steps = -(-K // kstep)
    slices = -(-steps // spw)
    max_waves = 8 if (mt == 4 or spw == 8) else 16
    passes = -(-(-(-slices // max_waves)) // split)
    waves = -(-slices // (split * passes))
    if split > slices or per > max(1, min((128 // (waves * mt)) & ~1, 16)) or (mt > 1 and spw != 2):
        return None
    lds = ((per + 1) & ~1) * waves * mt * 1024 + waves * 2048
    by_registers = {1: {2: 28, 4: 16, 8: 8}, 2: {2: 20}, 4: {2: 16}}[mt][spw]
    return dict(N=N, K=K, M=M, mt=mt, per=per, split=split, passes=passes, bytes=1 if storage[0] == "8" else 2,
                wgs=-(-(-(-N // 16)) // per) * split, columns=waves * passes * spw * kstep,
                slots=max(1, min(160 * 1024 // lds, by_registers // waves)))


# ---- on the GPU -------------------------------------------------------------------------------------

def time_all(candidates_path, routes_path, shapes):
    import torch

    from . import binding as nfp, workloads

    dev = torch.device("cuda:0")

    def graph_of(call, reps):
        call(0)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for r in range(reps):
                call(r)
        g.replay()
        return g

    def microseconds(g, reps):
        a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        e.record()
        e.synchronize()
        return a.elapsed_time(e) * 1e3 / reps

    t0 = time.time()
    with open(candidates_path, "w") as cand, open(routes_path, "w") as routes:
        for N, K in shapes:
            for storage in STORAGES:
                copies = max(2, min(16, int(600e6 / (N * K * (1 if storage[0] == "8" else 2))) + 1))
                layers = []
                for i in range(copies):
                    W = workloads.weight_device(N, K, 0.02, seed=i)
                    layers.append(W if storage == "pr" else nfp.decompose(W, check=False, packed=storage[-1] == "p"))
                    del W
                reps = max(copies, 8)
                for M in sorted(set(CANDIDATE_TOKENS) | set(ROUTE_TOKENS)):
                    X = workloads.act_device(M, K, seed=2)
                    Xq, sc = nfp.quantize_act(X)
                    Y = torch.empty((M, N), dtype=torch.float16, device=dev)
                    ws = nfp.new_workspace(8 * M * (N + 4) * 4 + M * K + 4 * M + (1 << 20), dev)

                    def call(i):
                        layer = layers[i % copies]
                        if storage == "pr":
                            nfp.plain_gemm_fp16(X, layer, out=Y, workspace=ws)
                        elif storage[0] == "8":
                            nfp.gemm_fp8_prequantized(Xq, sc, layer[0], out=Y, workspace=ws)
                        else:
                            nfp.gemm(X, layer[0], layer[1], nfp.MODE_FP16, out=Y, workspace=ws)

                    if M in ROUTE_TOKENS:
                        graphs = []
                        for limit in (0, 64):              # all to the tiled kernel, all to the streaming kernel
                            nfp.tune("small_max_m", limit)
                            try:
                                graphs.append(graph_of(call, reps))
                            finally:
                                nfp.tune("small_max_m", -1)
                        us = [[microseconds(g, reps) for g in graphs] for _ in range(6)]
                        us = [float(np.median(v)) for v in zip(*us)]
                        routes.write(json.dumps([N, K, M, storage, round(us[0], 2), round(us[1], 2)]) + "\n")
                    if M not in CANDIDATE_TOKENS:
                        continue
                    for spw in (2, 4):
                        for split in SPLITS:
                            for per in TILES:
                                g = geometry(N, K, M, storage, spw, split, per)
                                if g is None or g["wgs"] > 2400 or (g["wgs"] < 64 and per > 1):
                                    continue
                                pins = {"small_max_m": 64, "small_spw": spw, "small_split": split, "small_tiles": per}
                                for k, v in pins.items():
                                    nfp.tune(k, v)
                                try:
                                    graph = graph_of(call, reps)
                                finally:
                                    for k in pins:
                                        nfp.tune(k, -1)
                                us = float(np.median([microseconds(graph, reps) for _ in range(5)]))
                                cand.write(json.dumps([N, K, M, storage, [spw, split, per], round(us, 2)]) + "\n")
                del layers
                torch.cuda.empty_cache()
            print("N=%d K=%d  %.0f s" % (N, K, time.time() - t0), flush=True)


# ---- the fit ----------------------------------------------------------------------------------------

PARAMS = ("base", "chip_rate", "cu_rate", "single", "four", "split", "slice", "x_rate", "round", "part_rate", "pass")
START = (2.9, 8.0, 40.0, 1.5, 1.3, 0.5, 0.7, 120.0, 2.0, 1.0, 1.2)       # us; rates: 1e6, 1e3, -, -, -, -, 1e3, -, 1e6 bytes per us


def price(p, f):
    base, chip, cu, single, four, split, slice_, x, round_, part, pass_ = p
    wg_cu = np.ceil(f["wgs"] / 256)
    a = f["N"] * f["K"] * f["bytes"] / (chip * 1e6)
    b = wg_cu * f["per"] * 16 * np.minimum(f["columns"], f["K"]) * f["bytes"] / (cu * 1e3)
    b = b * np.where(f["per"] == 1, single, 1.0) * np.where(f["mt"] == 4, four, 1.0)
    t = base + (a ** 4 + b ** 4) ** 0.25 + wg_cu * np.minimum(f["M"], 16 * f["mt"]) * f["columns"] * f["bytes"] / (x * 1e3)
    t = t + round_ * (np.ceil(f["wgs"] / (256 * f["slots"])) - 1) + pass_ * (f["passes"] - 1)
    return t + np.where(f["split"] > 1, split + slice_ * f["split"] + f["split"] * f["M"] * f["N"] * 4 / (part * 1e6), 0.0)


def fit_small(path, storages):
    from scipy.optimize import minimize

    geo, us, group, groups = [], [], [], {}
    for line in open(path):
        N, K, M, storage, shape, t = json.loads(line)
        if storage not in storages or isinstance(shape, str):
            continue
        g = geometry(N, K, M, storage, *shape)
        if g is None or shape[0] == 8:
            continue
        geo.append(g)
        us.append(t)
        group.append(groups.setdefault((N, K, M, storage), len(groups)))
    f = {k: np.array([g[k] for g in geo], float) for k in geo[0]}
    us, group = np.array(us), np.array(group)
    best = np.full(len(groups), 1e30)
    np.minimum.at(best, group, us)
    lost = np.log(us / best[group])
    weight = np.exp(-2 * lost)
    weight /= weight.sum()

    def objective(logp):
        lp = np.log(price(np.exp(logp), f))
        low = np.full(len(groups), 1e30)
        np.minimum.at(low, group, lp)
        e = np.exp(-(lp - low[group]) / 0.025)
        soft = np.bincount(group, e * (lost + 2 * np.maximum(lost - 0.05, 0))) / np.bincount(group, e)
        return soft.mean() + np.sqrt((weight * (lp - np.log(us)) ** 2).sum())

    p = np.exp(minimize(objective, np.log(START), method="L-BFGS-B", options=dict(maxiter=300)).x)
    priced = price(p, f)
    order = np.lexsort((priced, group))
    first = order[np.unique(group[order], return_index=True)[1]]
    regret = us[first] / best[group[first]]
    print("// %d timings; chosen against fastest: %.1f %% behind on average, 95th percentile %.1f %%, at most %.1f %%"
          % (len(us), 100 * (np.exp(np.log(regret).mean()) - 1), 100 * (np.percentile(regret, 95) - 1), 100 * (regret.max() - 1)))
    scale = dict(chip_rate="e6", cu_rate="e3", x_rate="e3", part_rate="e6")
    print("{%s}," % ", ".join("%.3g%s" % (v, scale.get(n, "")) for n, v in zip(PARAMS, p)))


class _Tile64Plan(ctypes.Structure):
    _fields_ = [("cost", ctypes.c_double), ("split", ctypes.c_int)]


def fit_lines(path):
    from . import binding

    L = binding.lib()
    args = [ctypes.c_int] + 3 * [ctypes.c_int64]
    stream, tiles = L._ZN3nfp15small_gemm_costEilll, L._ZN3nfp11tile64_planEilll      # nfp::small_gemm_cost, nfp::tile64_plan
    stream.restype, stream.argtypes, tiles.restype, tiles.argtypes = ctypes.c_double, args, _Tile64Plan, args
    rows = {}
    for line in open(path):
        N, K, M, storage, t_tile, t_stream = json.loads(line)
        fp8 = storage[0] == "8"
        if storage == "pr" or (M > 32 and N * K >= 100 << 20):
            continue                                       # follows FP16 mode; always tiled
        plan = tiles(2 if fp8 else 1, M, N, K)
        rows.setdefault(("E4M3" if fp8 else "FP16", "17 ... 32" if M <= 32 else "33 ... 64"), []).append(
            (t_tile, t_stream, stream(2 if fp8 else 1, M, N, K), plan.cost, plan.split > 1))
    for key in sorted(rows):
        t, s, c, tc, sp = np.array(rows[key], float).T
        best, found = np.minimum(t, s), []
        for a in np.arange(1.0, 1.61, 0.05):
            for unsplit in np.arange(0.0, 15.1, 0.5):
                for split in (np.arange(unsplit, 15.1, 0.5) if key == ("FP16", "17 ... 32") else (unsplit,)):
                    x = np.log(np.where(c * a <= tc + np.where(sp > 0, split, unsplit), s, t) / best)
                    found.append((x.mean() + np.maximum(0, x - 0.04).mean(), a, unsplit, split, x.mean(), x.max()))
        _, a, unsplit, split, mean, most = min(found)
        print("// %s, %s tokens: {%.2f, %.1f, %.1f}, %.2f %% behind the faster kernel on average, at most %.0f %%; always tiled %.0f %%, always streaming %.1f %%"
              % (key + (a, unsplit, split, 100 * mean, 100 * most, 100 * np.log(t / best).mean(), 100 * np.log(s / best).mean())))


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("do", choices=("time", "fit"))
    ap.add_argument("candidates")
    ap.add_argument("routes")
    ap.add_argument("--shapes", nargs="*", default=None, help="N,K pairs instead of the built-in layer shapes")
    args = ap.parse_args()
    if args.do == "time":
        shapes = [tuple(int(v) for v in s.split(",")) for s in args.shapes] if args.shapes else \
            sorted({s for v in MODEL_SHAPES.values() for s in v} | set(OTHER_SHAPES))
        time_all(args.candidates, args.routes, shapes)
        return
    print("// kSmallCost: " + ", ".join(PARAMS))
    for storages in (("16p", "16r", "pr"), ("8p", "8r")):
        fit_small(args.candidates, storages)
    fit_lines(args.routes)


if __name__ == "__main__":
    main()
