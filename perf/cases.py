"""The workloads whose speed this library is judged by, each one pass of a
user's program through the public entry points of the binding.

Kinds of case:
  gemv       one decode projection, called eagerly (a program that schedules
             single projections itself).
  step       a whole decode step: every projection of every layer in order,
             q/k/v and gate/up batched, o and down alone, captured once in a
             graph as a decode loop keeps it, one replay per token.
  prefill    the projections of some layers over a chunk of M prompt tokens,
             the ones that read the same input stacked (q/k/v, gate/up), with
             the workspace that the library asks for.
  product    one matrix product of any size without a workspace, for each of
             the three weight operands.
  convert    float32 weights quantized into blocks and dequantized again: the
             offline conversion and its check.
  attention  FlowKV decode attention of one token over the caches of every
             layer (five sliding-window layers per global layer), captured in
             a graph like the step.

Model shapes come from workloads/.  Inputs are synthetic: uniform codes,
scales |N(0, 0.02)|, offsets of -scale times a zero point, normal activations
and caches.
"""
import math

import torch

import paper_2602_06063_amd as q4
from workloads import ATTENTION, GLOBAL_EVERY, MODELS, SWA_WINDOW

FP4 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0, -0.0, -0.5, -1.0, -1.5, -2.0, -3.0, -4.0, -6.0)
BLOCK = {"q4nx": 5120, "mx": 4352}            # bytes of a 32 x 256 block
PER_WEIGHT = {"q4nx": 0.625, "mx": 0.53125, "bf16": 2.0}
OUT = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest call: one query projection of the smallest model, for one token.
        {"name": "gemv 1b q", "kind": "gemv", "N": 1024, "K": 1152, "fmt": "q4nx", "out": "f32"},
        # One token of each model.  The smallest is a chain of launches of a few microseconds, the
        # largest streams 16 GB of weights; the 4b step ends in the vocabulary head.
        {"name": "step 1b", "kind": "step", "model": "1b", "fmt": "q4nx", "out": "bf16"},
        {"name": "step 4b", "kind": "step", "model": "4b", "fmt": "q4nx", "out": "f32"},
        {"name": "step 27b", "kind": "step", "model": "27b", "fmt": "q4nx", "out": "f32"},
        # A very short prompt, or sixteen decoding users in one batch.
        {"name": "prefill 1b m16", "kind": "prefill", "model": "1b", "M": 16, "layers": 8, "fmt": "q4nx", "out": "bf16"},
        # A question of a sentence or two (a ragged number of tokens).
        {"name": "prefill 4b m77", "kind": "prefill", "model": "4b", "M": 77, "layers": 4, "fmt": "q4nx", "out": "bf16"},
        # A page of text.
        {"name": "prefill 4b m512", "kind": "prefill", "model": "4b", "M": 512, "layers": 2, "fmt": "q4nx", "out": "f32"},
        # The chunk lengths that long prompts are cut into, of the benchmark.
        {"name": "prefill 4b m2048", "kind": "prefill", "model": "4b", "M": 2048, "layers": 1, "fmt": "q4nx", "out": "f32"},
        {"name": "prefill 27b m4096", "kind": "prefill", "model": "27b", "M": 4096, "layers": 1, "fmt": "q4nx", "out": "f32"},
        # A paragraph, or the ragged last chunk of a long prompt, on the MXFP4 variant.
        {"name": "prefill 27b mx m300", "kind": "prefill", "model": "27b", "M": 300, "layers": 1, "fmt": "mx", "out": "bf16"},
        # A large matrix converted from its float32 checkpoint, and back for a check.
        {"name": "convert 27b gate", "kind": "convert", "N": 21504, "K": 5376, "fmt": "q4nx", "out": "bf16"},
        # One token's attention with a long context.
        {"name": "attention 4b 32k", "kind": "attention", "model": "4b", "n": 32768, "static": False, "out": "f32"},
    ]


def _spread(rng, lo, hi):
    """A whole number of lo..hi, even over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["gemv", "step"] + ["prefill"] * 4 + ["product", "convert", "attention"])
    fmt = rng.choice(["q4nx", "q4nx", "mx"])
    out = rng.choice(["f32", "bf16"])
    if kind == "gemv":
        return {"kind": kind, "N": _spread(rng, 32, 43008), "K": 32 * _spread(rng, 8, 672), "fmt": fmt, "out": out}
    if kind == "step":  # the first layers of a model, so that no two are alike
        model = rng.choice(["1b", "4b", "27b"])
        return {"kind": kind, "model": model, "layers": rng.randint(4, MODELS[model]["layers"]), "fmt": fmt, "out": out}
    if kind == "prefill":
        model, M = rng.choice(["1b", "4b", "27b"]), _spread(rng, 2, 4096)
        layers = {"1b": 8, "4b": 4, "27b": 1}[model] if M <= 256 else 1
        return {"kind": kind, "model": model, "M": M, "layers": layers, "fmt": fmt, "out": out}
    if kind == "product":
        return {"kind": kind, "M": _spread(rng, 1, 2048), "N": _spread(rng, 32, 16384), "K": 32 * _spread(rng, 2, 336),
                "fmt": rng.choice(["q4nx", "mx", "bf16"]), "out": out}
    if kind == "convert":
        return {"kind": kind, "N": _spread(rng, 256, 21504), "K": 32 * _spread(rng, 16, 336), "fmt": fmt, "out": out}
    return {"kind": kind, "model": rng.choice(["1b", "4b", "27b"]), "n": _spread(rng, 16, 32768),
            "static": rng.random() < 0.5, "out": out}


# ------------------------------------------------------------------ shapes
def _jobs(case):
    """(M, N, K) of every product of a pass, launch by launch: a list of lists."""
    if case["kind"] == "gemv":
        return [[(1, case["N"], case["K"])]]
    if case["kind"] == "product":
        return [[(case["M"], case["N"], case["K"])]]
    model = MODELS[case["model"]]
    p = {name: (N, K) for name, N, K in model["proj"]}
    if case["kind"] == "step":
        layer = [[(1, *p["q"]), (1, *p["k"]), (1, *p["v"])], [(1, *p["o"])], [(1, *p["gate"]), (1, *p["up"])],
                 [(1, *p["down"])]]
        head = [[(1, *model["lm_head"][1:])]] if model["lm_head"] and "layers" not in case else []
        return layer * case.get("layers", model["layers"]) + head
    M, D = case["M"], p["q"][1]
    layer = [[(M, p["q"][0] + p["k"][0] + p["v"][0], D)], [(M, *p["o"])], [(M, 2 * p["gate"][0], D)], [(M, *p["down"])]]
    return layer * case["layers"]


def _layers(case):
    """(cache positions attended, window) of each attention layer for the token at position n - 1."""
    return [(case["n"], 0) if (i + 1) % GLOBAL_EVERY == 0 else (min(case["n"], SWA_WINDOW), SWA_WINDOW)
            for i in range(MODELS[case["model"]]["layers"])]


def work(case):
    esize = 4 if case["out"] == "f32" else 2
    if case["kind"] == "convert":
        return {"bytes": case["N"] * case["K"] * (4 + 2 * PER_WEIGHT[case["fmt"]] + esize), "flops": 4 * case["N"] * case["K"]}
    if case["kind"] == "attention":
        a = ATTENTION[case["model"]]
        H, G, d = a["H"], a["G"], a["d"]
        n = sum(k for k, _ in _layers(case))
        return {"bytes": 4 * G * n * d + len(_layers(case)) * H * d * (2 + esize), "flops": 4 * H * n * d}
    each = [j for launch in _jobs(case) for j in launch]
    return {"bytes": sum(N * K * PER_WEIGHT[case["fmt"]] + 2 * M * K + esize * M * N for M, N, K in each),
            "flops": sum(2 * M * N * K for M, N, K in each)}


def tolerance(case):
    if case["kind"] == "convert":
        return "exact"  # codes, scales and the dequantized weights are defined bit by bit
    if case["out"] == "bf16":  # one rounding to 8 bits: 1.7e-3 over many values, half a unit at most
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 4e-6, "max": 4e-5}


# ------------------------------------------------------------------ inputs
def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _weights(g, N, K, fmt):
    """A packed matrix of random weights (blocks of 32 x 256, strip by strip, padding as the
    packer writes it), or a bf16 one."""
    if fmt == "bf16":
        return _normal(g, N, K) * 0.02
    NS, KB = -(-N // 32), -(-K // 256)
    n = NS * KB
    codes = torch.randint(-(1 << 31), 1 << 31, (n * 1024,), generator=g, device="cuda", dtype=torch.int32)
    codes = codes.view(torch.uint8).view(NS, KB, 32, 128)
    if fmt == "mx":
        scales = torch.randint(119, 123, (NS, KB, 32, 8), generator=g, device="cuda", dtype=torch.uint8)
        tables, pads = [scales], [127]
    else:
        s = (torch.randn((NS, KB, 32, 8), generator=g, device="cuda") * 0.02).abs().clamp_min(2.0 ** -100).bfloat16()
        z = torch.randint(0, 16, (NS, KB, 32, 8), generator=g, device="cuda", dtype=torch.int32)
        tables, pads = [s, (s.float() * -z).bfloat16()], [0, 0]
    rows, cols = N % 32, K % 256
    for t, width, pad in [(codes, 2, 0)] + [(t, 32, p) for t, p in zip(tables, pads)]:
        if rows:
            t[-1, :, rows:] = pad
        if cols:
            t[:, -1, :, cols // width:] = pad
    return torch.cat([codes.view(n, 4096)] + [t.reshape(n, 256).view(torch.uint8).view(n, -1) for t in tables], 1).view(-1)


def _dequantized(blob, N, K, fmt):
    """The weights of a packed matrix in float64, unrounded."""
    if fmt == "bf16":
        return blob.double()
    NS, KB = -(-N // 32), -(-K // 256)
    b = blob.view(NS, KB, BLOCK[fmt])
    c = b[:, :, :4096].reshape(NS, KB, 32, 128)
    q = torch.stack([c & 15, c >> 4], -1).view(NS, KB, 32, 8, 32)
    if fmt == "mx":
        w = torch.tensor(FP4, device="cuda")[q.int()] * torch.exp2(b[:, :, 4096:].reshape(NS, KB, 32, 8, 1).double() - 127)
    else:
        t = b[:, :, 4096:].reshape(NS, KB, 1024).view(torch.bfloat16).view(NS, KB, 2, 32, 8, 1).double()
        w = q * t[:, :, 0] + t[:, :, 1]
    return w.view(NS, KB, 32, 256).transpose(1, 2).reshape(NS * 32, KB * 256)[:N, :K]


def _inputs(case, seed):
    """What a pass reads: (weights, activations) of every product, the float32 matrix, or the
    (query, K cache, V cache) of every layer."""
    g = _rng(seed)
    if case["kind"] == "convert":
        return torch.randn((case["N"], case["K"]), generator=g, device="cuda") * 0.02
    if case["kind"] == "attention":
        a = ATTENTION[case["model"]]
        return [(_normal(g, a["H"], a["d"]), _normal(g, a["G"], case["n"], a["d"]), _normal(g, a["G"], case["n"], a["d"]))
                for _ in _layers(case)]
    out = []
    for launch in _jobs(case):
        x = _normal(g, launch[0][0], launch[0][2])  # the products of a launch read the same activations
        out.append([(_weights(g, N, K, case["fmt"]), x) for _, N, K in launch])
    return out


def _captured(calls):
    """One graph of the calls, as a decode loop keeps it, after one pass to warm up."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    return graph


def prepare(case, seed):
    inputs, dtype, kind = _inputs(case, seed), OUT[case["out"]], case["kind"]
    state = {"case": case, "inputs": inputs}
    if kind == "convert":
        size = q4.q4nx_packed_size if case["fmt"] == "q4nx" else q4.q4nx_mx_packed_size
        state["blob"] = torch.empty(size(case["N"], case["K"]), dtype=torch.uint8, device="cuda")
        state["out"] = torch.empty_like(inputs, dtype=dtype)
        return state
    if kind == "attention":
        a, layers, n = ATTENTION[case["model"]], _layers(case), case["n"]
        H, G, d = a["H"], a["G"], a["d"]
        state["out"] = out = torch.empty((len(layers), H, d), dtype=dtype, device="cuda")
        work = torch.empty(q4.q4nx_flowkv_workspace_size(H, d, n), dtype=torch.uint8, device="cuda")

        def calls():
            for (q, k, v), (_, window), o in zip(inputs, layers, out):
                if case["static"]:
                    q4.q4nx_flowkv_decode_static(q, k, v, H, G, d, n, n - 1, window, d ** -0.5, o)
                else:
                    q4.q4nx_flowkv_decode(q, k, v, H, G, d, n, n - 1, window, d ** -0.5, o, work)

        state["work"], state["graph"] = work, _captured(calls)
        return state
    jobs = _jobs(case)
    if kind in ("gemv", "step"):
        state["out"] = out = torch.empty(sum(N for launch in jobs for _, N, _ in launch), dtype=dtype, device="cuda")
        launches, at = [], 0
        for launch, data in zip(jobs, inputs):
            items = []
            for (_, N, K), (w, x) in zip(launch, data):
                items.append((w, x, out[at:at + N], N, K))
                at += N
            launches.append(items)
        if kind == "gemv":
            state["item"] = launches[0][0]
            return state
        batched = q4.q4nx_gemv_batched if case["fmt"] == "q4nx" else q4.q4nx_mx_gemv_batched

        def calls():
            for items in launches:
                batched(items)

        state["graph"] = _captured(calls)
        return state
    state["out"] = [torch.empty((M, N), dtype=dtype, device="cuda") for ((M, N, _),) in jobs]
    state["products"] = [(M, N, K, x, w, y) for ((M, N, K),), ((w, x),), y in zip(jobs, inputs, state["out"])]
    if kind == "prefill":
        state["format"] = q4.Q4NX_WEIGHTS_Q4NX if case["fmt"] == "q4nx" else q4.Q4NX_WEIGHTS_MXFP4
        need = max(q4.q4nx_gemm_workspace_size(state["format"], M, N, K) for ((M, N, K),) in jobs)
        state["work"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    return state


# ------------------------------------------------------------------ passes
def run(state):
    case, out = state["case"], state["out"]
    kind, fmt = case["kind"], case["fmt"] if "fmt" in case else None
    if kind in ("step", "attention"):
        state["graph"].replay()
    elif kind == "gemv":
        (q4.q4nx_gemv if fmt == "q4nx" else q4.q4nx_mx_gemv)(*state["item"])
    elif kind == "prefill":
        for M, N, K, x, w, y in state["products"]:
            q4.q4nx_gemm_ex(state["format"], M, N, K, x, w, y, work=state["work"])
    elif kind == "product":
        M, N, K, x, w, y = state["products"][0]
        {"q4nx": q4.q4nx_gemm, "mx": q4.q4nx_mx_gemm, "bf16": q4.q4nx_gemm_bf16}[fmt](M, N, K, x, w, y)
    else:
        N, K, blob = case["N"], case["K"], state["blob"]
        if fmt == "q4nx":
            q4.q4nx_quantize(state["inputs"], N, K, blob)
            q4.q4nx_dequant(blob, N, K, out)
        else:
            q4.q4nx_mx_quantize(state["inputs"], N, K, blob)
            q4.q4nx_mx_dequant(blob, N, K, out)
        return {"blob": blob, "weights": out}
    return out


# ------------------------------------------------------------------ 64 bits
def _bf16(x):
    """float64 values rounded to bf16 as the library defines it (by way of float32)."""
    return x.float().bfloat16().double()


def _requantized(W, fmt):
    """float32 weights after quantization, in float64: the value of each weight's code."""
    w = W.view(-1, 32).double()
    if fmt == "mx":
        amax = w.abs().amax(1, keepdim=True)
        x = torch.exp2(torch.floor(torch.log2(amax)) - 2)
        grid = torch.tensor(FP4[:8], device="cuda", dtype=torch.float64)
        a = (w / x).abs()
        mids = (grid[1:] + grid[:-1]) / 2
        code = torch.bucketize(a, mids)  # values below or at a midpoint: the smaller code
        tie = (code < 7) & (code % 2 == 1) & (a == mids[code.clamp(max=6)])
        return (grid[code + tie] * x * torch.sign(w)).view(W.shape)
    lo, hi = W.view(-1, 32).aminmax(dim=1, keepdim=True)
    # (float32 values: the quotient by way of float64, since a division by a number may multiply by its inverse)
    d, m = ((hi - lo).double() / 15).float().bfloat16().double(), lo.bfloat16().double()
    best, value = torch.full_like(w, math.inf), torch.zeros_like(w)
    for q in range(16):
        level = (q * d + m).float().double()
        near = (level - w).abs()
        value = torch.where(near < best, level, value)
        best = torch.minimum(near, best)
    return value.view(W.shape)


def exact(case, seed):
    inputs, kind = _inputs(case, seed), case["kind"]
    if kind == "convert":
        rows = [_requantized(part, case["fmt"]) for part in inputs.split(2048)]
        w = torch.cat([r.float() for r in rows]).to(OUT[case["out"]])
        return {"blob": None, "weights": w.double()}
    if kind == "attention":
        d, out = ATTENTION[case["model"]]["d"], []
        for (q, k, v), (n, _) in zip(inputs, _layers(case)):
            k, v = k[:, -n:].double(), v[:, -n:].double()
            s = q.double().view(k.shape[0], -1, d) @ k.transpose(1, 2).contiguous() * d ** -0.5
            out.append((torch.softmax(s, -1) @ v).reshape(q.shape))
        return torch.stack(out)
    out = []
    for launch, data in zip(_jobs(case), inputs):
        for (M, N, K), (w, x) in zip(launch, data):
            w = _dequantized(w, N, K, case["fmt"])
            if kind in ("gemv", "step"):
                out.append(w @ x.view(-1).double())
            else:  # the matrix product takes its weights in bf16
                out.append(x.double() @ _bf16(w).t())
    return torch.cat(out) if kind in ("gemv", "step") else out
