"""The work that a serving program has this library do, as cases that can be timed and checked.

One case is what happens to one decoder layer of a language model: its four linears (qkv, o,
gate/up, down) over the two byte planes of their weights, for a batch of tokens, in FP16 mode or
FP8 mode, from row-major planes (the default storage) or packed ones; or the conversion of its
FP16 weights into planes when a checkpoint is loaded, and back when one is written.

`listed()` holds the cases, `draw(rng)` makes more of the same ranges, `prepare` makes what a
program has in hand (inputs, planes, workspace, output buffers, a captured graph of the decode
step), `run` is one pass through the entry points of `paper_2506_02024_amd.binding`, and `exact`
the same values in 64 bits from plain torch.
"""
import torch

from paper_2506_02024_amd import binding as nfp

WEIGHT_SIGMA = 0.02       # Gaussian stand-in for trained weights, far inside the format's |w| <= 1.75
DEVICE = "cuda:0"

# (hidden, rows of qkv, rows of the fused gate/up projection, columns of the down projection, columns of o)
LLAMA_8B = dict(hidden=4096, qkv=6144, gate_up=28672, ffn=14336, o_in=4096)
NEMO_12B = dict(hidden=5120, qkv=6144, gate_up=28672, ffn=14336, o_in=4096)
PHI_14B = dict(hidden=5120, qkv=7680, gate_up=35840, ffn=17920, o_in=5120)
SMALL_1B = dict(hidden=1040, qkv=1560, gate_up=5544, ffn=2768, o_in=1040)


def _case(name, kind, dims, tokens, mode, layout, exception=False):
    return dict(dims, name=name, kind=kind, tokens=tokens, mode=mode, layout=layout, exception=exception)


def listed():
    return [
        # a single user of a small model with ragged sizes, called from Python without a graph:
        # launch and call overhead count as much as bytes
        _case("small_m1_fp16_rowmajor", "eager", SMALL_1B, 1, "fp16", "rowmajor"),
        # a single user: one token, the weight stream alone
        _case("decode_m1_fp16_rowmajor", "graph", LLAMA_8B, 1, "fp16", "rowmajor"),
        # the usual decode batch of a serving loop that packed its planes at load time
        _case("decode_m16_fp16_packed", "graph", LLAMA_8B, 16, "fp16", "packed"),
        # the same batch when the load-aware policy has switched to FP8 mode, planes as the format defines them
        _case("decode_m16_fp8_rowmajor", "graph", LLAMA_8B, 16, "fp8", "rowmajor"),
        # a partly filled decode batch of a larger model in FP8 mode
        _case("decode_m11_fp8_packed", "graph", PHI_14B, 11, "fp8", "packed"),
        # a large decode batch, with one layer (down) that has a weight out of the format's range and
        # therefore keeps its FP16 weights
        _case("decode_m48_fp16_rowmajor", "graph", NEMO_12B, 48, "fp16", "rowmajor", True),
        # a step that mixes a prompt chunk with decoding requests: any token count
        _case("mixed_m200_fp16_rowmajor", "eager", LLAMA_8B, 200, "fp16", "rowmajor"),
        # a chunked prefill of odd length in FP8 mode
        _case("prefill_m777_fp8_rowmajor", "eager", LLAMA_8B, 777, "fp8", "rowmajor"),
        # a prefill in FP16 mode
        _case("prefill_m2048_fp16_rowmajor", "eager", LLAMA_8B, 2048, "fp16", "rowmajor"),
        # the largest prefill batch, in FP8 mode as the policy asks for
        _case("prefill_m8192_fp8_packed", "eager", LLAMA_8B, 8192, "fp8", "packed"),
        # several linears that share one input (separate gate and up): quantised once
        _case("shared_m1000_fp8_packed", "shared", LLAMA_8B, 1000, "fp8", "packed"),
        # loading a checkpoint: FP16 weights of the layer into planes, with the range check
        _case("load_rowmajor", "load", LLAMA_8B, 1, "fp16", "rowmajor"),
    ]


def draw(rng):
    def log_int(lo, hi, mult=1):
        v = lo * (hi / lo) ** rng.random()
        return max(mult, int(round(v / mult)) * mult)

    kind = rng.choice(["graph"] * 4 + ["eager"] * 5 + ["shared", "load", "export"])
    mult = rng.choice([16, 64, 128, 128, 256])
    hidden = log_int(1024, 8192, mult)
    ffn = max(mult, int(round(hidden * rng.uniform(2.5, 3.6) / mult)) * mult)
    # odd row counts occur where a layer is cut over GPUs or padded by hand
    odd = rng.choice([0, 0, 0, rng.randrange(1, 64)])
    dims = dict(hidden=hidden, qkv=int(hidden * rng.choice([1.25, 1.5, 2.0, 3.0])) + odd, gate_up=2 * ffn + odd,
                ffn=ffn, o_in=hidden)
    weights = sum(n * k for n, k in _shapes(dims))
    if kind == "graph":
        tokens = log_int(1, 64)
    elif kind == "shared":
        tokens = log_int(16, 4096)
    elif kind == "eager":
        tokens = log_int(1, 8192)
    else:
        tokens = 1
    largest = 8192 * sum(n * k for n, k in _shapes(LLAMA_8B))
    tokens = max(1, min(tokens, largest // weights))
    return dict(dims, kind=kind, tokens=tokens, mode=rng.choice(["fp16", "fp8"]) if kind != "shared" else "fp8",
                layout=rng.choice(["rowmajor", "packed"]), exception=kind in ("graph", "eager") and rng.random() < 0.15)


def _shapes(case):
    """(N, K) of the linears of a case."""
    h = case["hidden"]
    if case.get("kind") == "shared":
        return [(case["gate_up"] // 2, h), (case["gate_up"] // 2, h)]
    return [(case["qkv"], h), (h, case["o_in"]), (case["gate_up"], h), (h, case["ffn"])]


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _weights(case, g):
    out = []
    for i, (n, k) in enumerate(_shapes(case)):
        w = torch.empty((n, k), dtype=torch.float16, device=DEVICE)
        w.normal_(0.0, WEIGHT_SIGMA, generator=g)
        if case["exception"] and i == 3:
            w[n // 2, k // 3] = 2.5                   # one weight the format cannot hold
        out.append(w)
    return out


def _activations(case, g):
    """One input per linear (a single one for linears that share it), tokens of different magnitude."""
    out = []
    for i, (_, k) in enumerate(_shapes(case)):
        if case["kind"] == "shared" and i > 0:
            out.append(out[0])
            continue
        x = torch.empty((case["tokens"], k), dtype=torch.float32, device=DEVICE)
        x.normal_(0.0, 1.0, generator=g)
        size = torch.empty((case["tokens"], 1), dtype=torch.float32, device=DEVICE)
        size.uniform_(0.25, 2.0, generator=g)
        out.append((x * size).to(torch.float16))
    return out


def _mode(case):
    return nfp.MODE_FP8 if case["mode"] == "fp8" else nfp.MODE_FP16


def _linears(state):
    for x, layer, y in zip(state["x"], state["layers"], state["y"]):
        nfp.linear(x, layer, state["mode"], out=y, workspace=state["workspace"])
    return state["y"]


def prepare(case, seed):
    g = _generator(seed)
    weights = _weights(case, g)
    packed = case["layout"] == "packed"
    state = dict(kind=case["kind"], packed=packed, mode=_mode(case))
    if case["kind"] == "load":
        state["weights"] = weights
        return state
    if case["kind"] == "export":
        state["planes"] = [nfp.decompose(w, packed=packed) for w in weights]
        state["out"] = [torch.empty_like(w) for w in weights]
        return state
    state["x"] = _activations(case, g)
    state["layers"] = [nfp.Layer(w, packed=packed) for w in weights]
    m = case["tokens"]
    state["y"] = [torch.empty((m, n), dtype=torch.float16, device=DEVICE) for n, _ in _shapes(case)]
    need = max(nfp.gemm_workspace_size(m, n, k, mode) for n, k in _shapes(case) for mode in (nfp.MODE_FP16, nfp.MODE_FP8))
    state["workspace"] = nfp.new_workspace(need, DEVICE)
    if case["kind"] == "graph":                       # a serving loop captures its decode step once
        _linears(state)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _linears(state)
    return state


def run(state):
    kind = state["kind"]
    if kind == "graph":
        state["graph"].replay()
        return state["y"]
    if kind == "eager":
        return _linears(state)
    if kind == "shared":
        xq, scales = nfp.quantize_act(state["x"][0])
        for layer, y in zip(state["layers"], state["y"]):
            nfp.gemm_fp8_prequantized(xq, scales, layer.upper, out=y, workspace=state["workspace"])
        return {"y": state["y"], "xq": xq, "scales": scales}
    if kind == "load":
        layers = [nfp.Layer(w, packed=state["packed"]) for w in state["weights"]]
        planes = [(l.upper.data, l.lower.data) if state["packed"] else (l.upper, l.lower) for l in layers]
        return {"planes": planes, "out_of_range": [l.out_of_range for l in layers]}
    return [nfp.reconstruct(u, l, out=o) for (u, l), o in zip(state["planes"], state["out"])]


def work(case):
    """Each weight byte, input and output once; two flops per multiply-add."""
    m = case["tokens"]
    total_bytes = total_flops = 0
    for i, (n, k) in enumerate(_shapes(case)):
        if case["kind"] in ("load", "export"):
            total_bytes += 4 * n * k
            continue
        fp16 = case["mode"] == "fp16" or (case["exception"] and i == 3)
        total_bytes += (2 if fp16 else 1) * n * k + 2 * m * n
        if case["kind"] != "shared":
            total_bytes += 2 * m * k
        elif i == 0:
            total_bytes += 3 * m * k + 4 * m
        total_flops += 2 * m * n * k
    return {"bytes": total_bytes, "flops": total_flops}


def tolerance(case):
    if case["kind"] in ("load", "export"):
        return "exact"
    # FP16 outputs of FP32 sums: the rounding of the output is 2.1e-4 of the result in the 2-norm and
    # at most one unit in the last place (9.8e-4) for a value; a sum in another order moves few of them.
    # The E4M3 codes and their scales are whole values that every implementation makes alike.
    return {"rel": 8e-4, "max": 4e-3, "differ": 0.0}


def _quantized(x):
    """Per-token E4M3: codes as 64-bit values, and scales, from the definition (amax / 448 in binary32)."""
    # quotients in 64 bits, rounded to 32: the correctly rounded binary32 quotients
    amax = x.abs().amax(dim=1, keepdim=True).double()
    scale = torch.where(amax == 0, torch.ones_like(amax), amax / 448.0).float()
    q = (x.double() / scale.double()).float().clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q, scale


def exact(case, seed):
    if case["kind"] in ("load", "export"):
        return None                                   # whole values; the tolerance is "exact"
    g = _generator(seed)
    weights = _weights(case, g)
    xs = _activations(case, g)
    ys = []
    for i, (w, x) in enumerate(zip(weights, xs)):
        if case["mode"] == "fp16" or (case["exception"] and i == 3):
            ys.append(x.double() @ w.double().t().contiguous())
        else:
            q, scale = _quantized(x)
            upper = (w.float() * 256.0).to(torch.float8_e4m3fn)      # the upper plane read as E4M3
            ys.append((q.float().double() @ upper.float().double().t().contiguous()) * (scale.double() / 256.0))
    if case["kind"] == "shared":
        q, scale = _quantized(xs[0])
        return {"y": ys, "xq": None, "scales": scale.reshape(-1).double()}
    return ys
