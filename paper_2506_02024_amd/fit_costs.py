"""Times the launch shapes of the kernels over many layers and fits the constants that the library compiles in:
kSmallCost (csrc/gemm_small.hip), the lines between the streaming kernel and the 64-token tiles at 17 ... 64 tokens
(kLine in csrc/nestedfp_api.hip), kShortCost (65 ... 256 tokens, csrc/gemm_large.hip), kTallCost (more than 256 tokens, there
too); and says how far the choices that the library makes are behind the fastest launch, rows_through_lds among them.

    python -m paper_2506_02024_amd.fit_costs time candidates.jsonl routes.jsonl     # on the GPU, about 7 minutes
    python -m paper_2506_02024_amd.fit_costs fit candidates.jsonl routes.jsonl      # prints the constants
    python -m paper_2506_02024_amd.fit_costs time-tiles tiles.jsonl [--tokens ...]  # on the GPU, about 10 minutes
    python -m paper_2506_02024_amd.fit_costs fit-tiles tiles.jsonl
    python -m paper_2506_02024_amd.fit_costs time-tall tall.jsonl [--tokens ...]    # on the GPU, about 10 s a layer
    python -m paper_2506_02024_amd.fit_costs fit-tall tall.jsonl

`time` writes one line per timing: [N, K, tokens, storage, [K-steps per wave, K split, tiles per workgroup],
us] and [N, K, tokens, storage, us of the tiled kernel, us of the streaming kernel].  Weights are cold (copies
taken in turn) and the calls are replayed as one graph.  storage: 16p / 16r the planes in FP16 mode, packed and
row-major, 8p / 8r the upper plane in FP8 mode on quantised activations, pr plain row-major FP16.  `time-tiles`: [N, K,
tokens, storage, launch, us], launch = null for the built-in choice or [tile tokens, tile weight rows, K split, deeper
pipeline, way of row-major planes]; above 256 tokens, where it serves to check the ways of row-major planes, tiles of 256
are timed at their full height.  The layers taken in turn hold 700 MB: what the 256 MB memory-side cache keeps
from one pass to the next makes non-temporal loads look slow and the others fast.  `time-tall`: launch = null or [tile tokens, tile
weight rows, K split, deeper pipeline, height of the token tiles], those priced at less than 1.6 times the cheapest; FP8 mode with its
quantisation, whose own time is taken off, so that rows of codes start on lines as they do in a call.
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

def graph_of(call, reps):
    import torch

    call(0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for r in range(reps):
            call(r)
    g.replay()
    return g


def microseconds(g, reps):
    import torch

    a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    g.replay()
    e.record()
    e.synchronize()
    return a.elapsed_time(e) * 1e3 / reps


def time_all(candidates_path, routes_path, shapes):
    import torch

    from . import binding as nfp, workloads

    dev = torch.device("cuda:0")
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


TILE_TOKENS = (65, 80, 96, 112, 128, 144, 160, 176, 192, 208, 224, 256)
TILE_SHAPES = ((256, 256), (256, 128), (128, 256), (128, 128), (64, 128))        # tokens x weight rows


def tile_launches(N, K, M, storage):
    """Every launch shape of the tiled kernels that is worth a timing: tile, K split, deeper pipeline (E4M3), way of the
    row-major planes (FP16 mode: straight into registers, through LDS; -1: there is one way)."""
    kt = -(-K // (128 if storage[0] == "8" else 64))
    for tm, tn in TILE_SHAPES:
        for split in SPLITS:
            wgs = -(-M // tm) * -(-N // tn) * split
            if split > 1 and (split > kt // 4 or wgs > 1280):
                break
            for deep in ((0, 1) if storage[0] == "8" and tm * tn < 256 * 256 and tm > 64 else (0,)):
                for way in ((0, 1) if storage == "16r" and tm > 64 else (-1,)):
                    yield tm, tn, split, deep, way


def time_tiles(path, shapes, tokens):
    import torch

    from . import binding as nfp, workloads

    dev = torch.device("cuda:0")
    t0 = time.time()
    with open(path, "w") as out:
        for N, K in shapes:
            for storage in STORAGES[:4]:
                fp8 = storage[0] == "8"
                copies = max(2, min(64, int(700e6 / (N * K * (1 if fp8 else 2))) + 1))
                layers = [nfp.decompose(workloads.weight_device(N, K, 0.02, seed=i), check=False, packed=storage[-1] == "p")
                          for i in range(copies)]
                for M in tokens:
                    X = workloads.act_device(M, K, seed=2)
                    Xq, sc = nfp.quantize_act(X)
                    Y = torch.empty((M, N), dtype=torch.float16, device=dev)
                    ws = nfp.new_workspace(8 * M * (N + 4) * 4 + M * K + 4 * M + (1 << 20), dev)

                    def call(i):
                        up, lo = layers[i % copies]
                        if fp8:
                            nfp.gemm_fp8_prequantized(Xq, sc, up, out=Y, workspace=ws)
                        else:
                            nfp.gemm(X, up, lo, nfp.MODE_FP16, out=Y, workspace=ws)

                    def timed(launch):
                        pins = {} if launch is None else dict(zip(("large_bm", "large_bn", "large_split", "large_deep", "large_rows"), launch))
                        if not fp8:
                            pins.pop("large_deep", None)
                        if pins and M > 256:
                            pins["large_height"] = 256     # (up to 256 tokens it follows the batch)
                        for k, v in pins.items():
                            nfp.tune(k, v)
                        try:
                            graph = graph_of(call, copies)
                        finally:
                            for k in pins:
                                nfp.tune(k, -1)
                        us = float(np.median([microseconds(graph, copies) for _ in range(5)]))
                        out.write(json.dumps([N, K, M, storage, launch, round(us, 2)]) + "\n")

                    timed(None)                                # the built-in choice
                    for launch in tile_launches(N, K, M, storage):
                        timed(launch)
                del layers
                torch.cuda.empty_cache()
            print("N=%d K=%d  %.0f s" % (N, K, time.time() - t0), flush=True)


TALL_TOKENS = (272, 300, 384, 449, 512, 600, 777, 1000, 1200, 1536, 1790, 2048, 2700, 3200, 4096, 5000, 8192)
# kTallCost by weight class (1 FP16 operands through registers, 2 E4M3, 3 plain row-major FP16).  Shapes: tile tokens x weight rows, deeper
# pipeline, microseconds per K-tile and per workgroup at the full height and at 160 tokens, per K-tile squared
TALL = {
    1: dict(shapes=((256, 256, 0, 1.11, 8.54, 0.773, 6.36, 0), (256, 128, 0, 0.573, 6.03, 0.351, 5.53, 0.309e-3), (128, 256, 0, 0.634, 6.39, 0, 0, 0.103e-3),
                    (128, 128, 0, 0.285, 4.28, 0, 0, 0.466e-3)), pair=1.0, l2_rate=28.3, split=2.98, split_rate=6.93, odd=1.05, lone=1.07, lone256=1.0),
    2: dict(shapes=((256, 256, 0, 0.951, 9.83, 0.653, 7.57, 0), (256, 128, 1, 0.445, 7.46, 0, 0, 0.502e-3), (128, 256, 1, 0.598, 5.27, 0, 0, 0.026e-3),
                    (128, 128, 0, 0.515, 4.75, 0, 0, 1.88e-3), (128, 128, 1, 0.247, 5.41, 0, 0, 1.19e-3)), pair=1.83, l2_rate=50.5, split=2.14, split_rate=5.55, odd=1.0, lone=1.09, lone256=1.0),
    3: dict(shapes=((256, 256, 0, 1.04, 7.72, 0.716, 5.68, 0), (256, 128, 1, 0.466, 7.05, 0, 0, 0.286e-3), (128, 256, 1, 0.578, 4.71, 0, 0, 0.168e-3),
                    (128, 128, 0, 0.432, 4.88, 0, 0, 1.34e-3), (128, 128, 1, 0.223, 4.69, 0, 0, 1.00e-3)), pair=1.70, l2_rate=34.3, split=2.61, split_rate=6.13, odd=1.0, lone=1.12, lone256=1.05),
}


def tall_class(storage):
    return 3 if storage == "pr" else (2 if storage[0] == "8" else 1)


def heights_of(cls, tm, tn):
    return (160, 192, 224, 256) if tm == 256 and (cls == 1 or tn == 256) else (tm,)


def tall_launches(cls, N, K, M):
    """Every launch that choose_tall() prices, with what the price is made of."""
    kt = -(-K // (128 if cls == 2 else 64))
    for shape, (tm, tn, deep) in enumerate(e[:3] for e in TALL[cls]["shapes"]):
        for height in heights_of(cls, tm, tn):
            for split in SPLITS:
                if split > 1 and split > kt // 4:
                    break
                per = -(-kt // split)
                slices = -(-kt // per)
                yield (tm, tn, split, deep, height), dict(
                    N=N, K=K, M=M, shape=shape, tn=tn, height=height, per=per, slices=slices, wgs=-(-M // height) * -(-N // tn) * slices,
                    cut=len(heights_of(cls, tm, tn)) > 1)


def columns(launches):
    return {k: np.array([g[k] for g in launches], float) for k in launches[0]}


def price_tall(cls, f, p=None):
    """What choose_tall() prices launches at; p: constants in the order of tall_start()."""
    c = TALL[cls] if p is None else tall_constants(cls, p)
    shape = f["shape"].astype(int)
    tk, tfix, tk160, tfix160, tk2 = np.array([e[3:] for e in c["shapes"]]).T[:, shape]
    at = np.where(f["cut"] > 0, (f["height"] - 160) / 96, 1.0)
    tk, tfix = tk160 + at * (tk - tk160), tfix160 + at * (tfix - tfix160)
    paired = np.array([e[:3] == (128, 128, 0) for e in c["shapes"]])[shape]
    rounds = np.ceil(f["wgs"] / 256)
    t = rounds * (tfix + f["per"] * tk) / np.where((rounds > 1) & paired, c["pair"], 1.0) + rounds * f["per"] ** 2 * tk2
    t = t + f["wgs"] * f["per"] * (f["height"] + f["tn"]) * 128 / (c["l2_rate"] * 1e6)
    split = f["slices"] > 1
    t = t + np.where(split, c["split"] + 8 * f["M"] * f["N"] * f["slices"] / (c["split_rate"] * 1e6), 0.0)
    t = t * np.where(split & (f["per"] % 2 == 1) & (f["K"] % 128 == 0), c["odd"], 1.0)
    lone = ~split & (f["height"] == 128) & (f["wgs"] <= 256) & (5 * ((f["M"] - 1) % 128 + 1) > 2 * 128)
    return t * np.where(lone, np.where(f["tn"] == 128, c["lone"], c["lone256"]), 1.0)


def tall_start(cls):
    c = TALL[cls]
    return np.array([v for e in c["shapes"] for v in e[3:] if v] + [c[k] for k in ("pair", "l2_rate", "split", "split_rate", "odd", "lone", "lone256")])


def tall_constants(cls, p):
    it = iter(p)
    shapes = tuple(e[:3] + tuple(next(it) if v else 0 for v in e[3:]) for e in TALL[cls]["shapes"])
    return dict(shapes=shapes, **dict(zip(("pair", "l2_rate", "split", "split_rate", "odd", "lone", "lone256"), it)))


def time_tall(path, shapes, tokens):
    import torch

    from . import binding as nfp, workloads

    dev = torch.device("cuda:0")
    t0 = time.time()
    with open(path, "w") as out:
        for N, K in shapes:
            for storage in STORAGES:
                cls = tall_class(storage)
                copies = max(2, min(64, int(700e6 / (N * K * (1 if cls == 2 else 2))) + 1))
                layers = []
                for i in range(copies):
                    W = workloads.weight_device(N, K, 0.02, seed=i)
                    layers.append(W if cls == 3 else nfp.decompose(W, check=False, packed=storage[-1] == "p"))
                    del W
                for M in tokens:
                    X = workloads.act_device(M, K, seed=2)
                    Y = torch.empty((M, N), dtype=torch.float16, device=dev)
                    ws = nfp.new_workspace(8 * M * (N + 4) * 4 + M * (K + 128) + 4 * M + (1 << 20), dev)
                    reps = copies if copies * M * N * K < 4e13 else max(2, int(4e13 / (M * N * K)))

                    def call(i):
                        layer = layers[i % copies]
                        if cls == 3:
                            nfp.plain_gemm_fp16(X, layer, out=Y, workspace=ws)
                        else:
                            nfp.gemm(X, layer[0], layer[1], nfp.MODE_FP8 if cls == 2 else nfp.MODE_FP16, out=Y, workspace=ws)

                    def timed(pins, call=call):
                        for k, v in pins.items():
                            nfp.tune(k, v)
                        try:
                            graph = graph_of(call, reps)
                        finally:
                            for k in pins:
                                nfp.tune(k, -1)
                        return float(np.median([microseconds(graph, reps) for _ in range(5)]))

                    timed({})                                  # (the first launches of a batch size run at another clock: 1.5 % slower)
                    off = timed({}, lambda i: nfp.quantize_act(X)) if cls == 2 else 0.0
                    out.write(json.dumps([N, K, M, storage, None, round(timed({}) - off, 2)]) + "\n")
                    launches, geo = zip(*tall_launches(cls, N, K, M))
                    priced = price_tall(cls, columns(geo))
                    for launch, t in zip(launches, priced):
                        if t > 1.6 * priced.min():
                            continue
                        pins = dict(zip(("large_bm", "large_bn", "large_split", "large_deep", "large_height"), launch))
                        if cls == 1:
                            del pins["large_deep"]
                        out.write(json.dumps([N, K, M, storage, launch, round(timed(pins) - off, 2)]) + "\n")
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


def behind(v):
    v = np.array(v)
    return "%.1f %% behind on average, 95th percentile %.0f %%, at most %.0f %%" % (
        100 * (np.exp(np.log(v).mean()) - 1), 100 * (np.percentile(v, 95) - 1), 100 * (v.max() - 1))


def fit_prices(price, start, us, group):
    """Constants that lose the least time to the fastest launch of a problem (group) by a soft choice of the cheapest, and price launches
    near the fastest well; with what the choice loses by the constants at the start and by the new ones."""
    from scipy.optimize import minimize

    best = np.full(group.max() + 1, 1e30)
    np.minimum.at(best, group, us)
    lost = np.log(us / best[group])
    weight = np.exp(-4 * lost)
    weight /= weight.sum()

    def objective(logp):
        lp = np.log(price(np.exp(logp)))
        low = np.full(len(best), 1e30)
        np.minimum.at(low, group, lp)
        e = np.exp(-(lp - low[group]) / 0.02)
        soft = np.bincount(group, e * (lost + 3 * np.maximum(lost - 0.04, 0))) / np.bincount(group, e)
        return soft.mean() + 0.3 * np.sqrt((weight * (lp - np.log(us)) ** 2).sum())

    def regret(p):
        order = np.lexsort((price(p), group))
        first = order[np.unique(group[order], return_index=True)[1]]
        return behind(us[first] / best[group[first]])

    p = np.exp(minimize(objective, np.log(start), method="L-BFGS-B", options=dict(maxiter=150)).x)
    return p, regret(np.array(start)), regret(p)


# kShortCost: per tile shape microseconds per K-tile and per workgroup (tiles of 256 tokens: also at a height of 160), then the rest
SHORT_PARAMS = ("pair128", "pair64", "base", "w_rate", "l2_rate", "cu_rate", "split", "split_rate")
SHORT_START = {False: (0.725, 6.05, 0.556, 3.47, 0.421, 2.63, 0.314, 1.28, 0.5, 2.61, 0.2785, 0.83, 0.271, 0.51, 1.045, 1.045, 3.0, 15.2, 219, 167, 3.45, 5.28),
               True: (0.6255, 3.16, 0.378, 3.16, 0.319, 2.41, 0.319, 2.41, 0.334, 2.71, 0.2136, 1.73, 0.183, 1.54, 1.0, 1.10, 2.0, 10.4, 1e9, 144, 3.28, 4.68)}


def price_short(p, f, fp8):
    """What choose_short() prices a launch at; rates in 1e6 (cu_rate: 1e3) bytes per microsecond."""
    pair128, pair64, base, w, l2, cu, split, split_rate = p[14:]
    at = (f["height"] - 160) / 96
    shape = [f["shape"] == i for i in range(5)]
    tk = np.select(shape, [p[2] + at * (p[0] - p[2]), p[6] + at * (p[4] - p[6]), p[8], p[10], p[12]])
    tfix = np.select(shape, [p[3] + at * (p[1] - p[3]), p[7] + at * (p[5] - p[7]), p[9], p[11], p[13]])
    rounds = np.ceil(f["wgs"] / 256)
    t = rounds * (tfix + f["per"] * tk)
    t = t / np.where(rounds > 1, np.select([shape[3], shape[4]], [pair128, pair64], 1.0), 1.0)
    t = t + base + f["N"] * f["K"] * f["bytes"] / (w * 1e6) + f["wgs"] * f["per"] * (f["height"] + f["tn"]) * 128 / (l2 * 1e6)
    t = t + rounds * f["per"] * (np.minimum(f["height"], f["M"]) + f["tn"]) * 128 / (cu * 1e3)
    t = t + np.where(f["slices"] > 1, split + 8 * f["M"] * f["N"] * f["slices"] / (split_rate * 1e6), 0.0)
    tail = (f["shape"] == 4) & (f["M"] > 128) & (np.ceil(f["N"] / 128) % 8 != 0) & (f["N"] * f["K"] >= 24 << 20)
    return t * np.where(tail & fp8, 1.1, 1.0)


def fit_tiles(path):
    from . import binding

    through = binding.lib()._ZN3nfp16rows_through_ldsEiillli                      # nfp::rows_through_lds
    through.restype, through.argtypes = ctypes.c_bool, [ctypes.c_int] * 2 + [ctypes.c_int64] * 3 + [ctypes.c_int]
    problems = {}
    for line in open(path):
        N, K, M, storage, launch, us = json.loads(line)
        problems.setdefault((N, K, M, storage), {})[None if launch is None else tuple(launch)] = us

    for storage in STORAGES[:4]:
        v = [d[None] / min(us for launch, us in d.items() if launch) for key, d in problems.items() if key[3] == storage]
        if v:
            print("// %s: built-in choice against the fastest of its %d launches on %d problems: %s" % (
                storage, sum(len(d) - 1 for key, d in problems.items() if key[3] == storage), len(v), behind(v)))
    rule, regs = [], []
    for (N, K, M, storage), d in problems.items():
        for launch, us in d.items():
            if storage == "16r" and launch and launch[4] == 1 and launch[:4] + (0,) in d:
                both = (d[launch[:4] + (0,)], us)
                rule.append(both[through(launch[0], launch[1], M, K, K, launch[2])] / min(both))
                regs.append(both[0] / min(both))
    if rule:
        print("// row-major planes, %d launches both ways: the rule %s; all into registers %s" % (len(rule), behind(rule), behind(regs)))
    for fp8 in (False, True):
        geo, us, group, groups = [], [], [], {}
        for (N, K, M, storage), d in problems.items():
            if M > 256 or (storage[0] == "8") != fp8:
                continue
            kt = -(-K // (128 if fp8 else 64))
            for launch, t in d.items():
                if launch is None:
                    continue
                tm, tn, split, deep, way = launch
                if fp8 and tm > 64 and tm * tn < 256 * 256 and not deep:
                    continue                               # (the deeper pipeline where there is one)
                if way >= 0 and way != through(tm, tn, M, K, K, split):
                    continue
                per = -(-kt // split)
                slices = -(-kt // per)
                height = max(160, -(-M // 32) * 32) if tm == 256 and (tn == 256 or not fp8) else tm
                geo.append(dict(N=N, K=K, M=M, shape=TILE_SHAPES.index((tm, tn)), tn=tn, height=height, per=per, slices=slices,
                                wgs=-(-M // tm) * -(-N // tn) * slices, bytes=1 if fp8 else 2))
                us.append(t)
                group.append(groups.setdefault((N, K, M, storage), len(groups)))
        if not geo:
            continue
        f = {k: np.array([g[k] for g in geo], float) for k in geo[0]}
        us, group = np.array(us), np.array(group)
        p, before, after = fit_prices(lambda p: price_short(p, f, fp8), SHORT_START[fp8], us, group)
        print("// %s: %d timings; constants as they are: %s; fitted: %s" % ("E4M3" if fp8 else "FP16", len(us), before, after))
        print("tiles {%s}, %s" % (", ".join("%.3g" % v for v in p[:14]), ", ".join("%s %.4g" % v for v in zip(SHORT_PARAMS, p[14:]))))


def fit_tall(path):
    problems = {}
    for line in open(path):
        N, K, M, storage, launch, us = json.loads(line)
        problems.setdefault((N, K, M, storage), {})[None if launch is None else tuple(launch)] = us
    for cls, name in ((1, "FP16 operands through registers"), (2, "E4M3"), (3, "plain FP16")):
        geo, us, group, built_in, n = [], [], [], [], 0
        for (N, K, M, storage), d in problems.items():
            if tall_class(storage) != cls or len(d) < 2:
                continue
            built_in.append(d[None] / min(t for launch, t in d.items() if launch))
            for launch, g in tall_launches(cls, N, K, M):
                if launch in d:
                    geo.append(g)
                    us.append(d[launch])
                    group.append(n)
            n += 1
        if not geo:
            continue
        f = columns(geo)
        p, before, after = fit_prices(lambda p: price_tall(cls, f, p), tall_start(cls), np.array(us), np.array(group))
        print("// %s: %d timings of %d problems; the library's choice %s; prices as they are %s; fitted %s" % (name, len(us), n, behind(built_in), before, after))
        c = tall_constants(cls, p)
        print("{%d, {%s}, %.3g, %.3ge6, %.3g, %.3ge6, %.3g, %.3g, %.3g, 0, 0, false}" % (
            len(c["shapes"]), ", ".join("{%d, %d, %d, %s}" % (e[:3] + (", ".join("%.3g" % v for v in e[3:]),)) for e in c["shapes"]),
            c["pair"], c["l2_rate"], c["split"], c["split_rate"], c["odd"], c["lone"], c["lone256"]))


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("do", choices=("time", "fit", "time-tiles", "fit-tiles", "time-tall", "fit-tall"))
    ap.add_argument("files", nargs="+", help="candidates.jsonl routes.jsonl, tiles.jsonl or tall.jsonl")
    ap.add_argument("--shapes", nargs="*", default=None, help="N,K pairs instead of the built-in layer shapes")
    ap.add_argument("--tokens", nargs="*", type=int, default=None, help="batch sizes of time-tiles and time-tall")
    args = ap.parse_args()
    shapes = [tuple(int(v) for v in s.split(",")) for s in args.shapes] if args.shapes else \
        sorted({s for v in MODEL_SHAPES.values() for s in v} | set(OTHER_SHAPES))
    one = args.do not in ("time", "fit")
    if len(args.files) != (1 if one else 2):
        ap.error("%s takes %s" % (args.do, "one file" if one else "two files"))
    if args.do == "time-tall" and min(args.tokens or TALL_TOKENS) <= 256:
        ap.error("time-tall is for more than 256 tokens")
    if args.do == "time":
        time_all(args.files[0], args.files[1], shapes)
        return
    if args.do == "time-tiles":
        time_tiles(args.files[0], shapes, args.tokens or TILE_TOKENS)
        return
    if args.do == "time-tall":
        time_tall(args.files[0], shapes, args.tokens or TALL_TOKENS)
        return
    if args.do == "fit-tall":
        fit_tall(args.files[0])
        return
    if args.do == "fit-tiles":
        fit_tiles(args.files[0])
        return
    print("// kSmallCost: " + ", ".join(PARAMS))
    for storages in (("16p", "16r", "pr"), ("8p", "8r")):
        fit_small(args.files[0], storages)
    fit_lines(args.files[1])


if __name__ == "__main__":
    main()
