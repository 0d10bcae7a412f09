"""What this library's speed is measured on.

Every case is one call sequence that a user's program makes through the Python binding
(``paper_2605_08565_amd.mxq``): quantising weights offline, quantising activations while serving,
searching the best scales, reading quantised tensors back, and the diagnostics of a study.  Shapes
and value distributions are those of the benchmark, the model sweep, the numerical study and the
tests of this repository.

The library promises bits, not approximations (codes, scale bytes and the fp32 block SSE follow one
pinned sequence of roundings), so every case is compared exactly.
"""
import math

import torch

from paper_2605_08565_amd import mxq
from paper_2605_08565_amd.workloads import LAYER_SHAPES

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
FORMATS = {"e8m0": mxq.SCALE_E8M0, "e4m3": mxq.SCALE_E4M3, "ue5m3": mxq.SCALE_UE5M3}
RECIPES = {"absmax": mxq.RECIPE_ABSMAX, "absmax_pz": mxq.RECIPE_ABSMAX_PZ, "4over6": mxq.RECIPE_4OVER6,
           "4over6_pz": mxq.RECIPE_4OVER6_PZ, "brute": mxq.RECIPE_BRUTE, "brute_pruned": mxq.RECIPE_BRUTE_PRUNED}
CANDIDATES = {"e8m0": 255, "e4m3": 126, "ue5m3": 254}
BLOCKS = (2, 4, 8, 16, 32, 64, 128)
STUDY_SIGMAS = 151                       # standard deviations of the numerical study, 0.0005 .. 0.05


def listed():
    return [
        # Serving, one decode step of 16 sequences: the hidden state is scaled as a whole and
        # quantised, nobody asks for the error, the program keeps its output buffers.  The smallest
        # call: launches and host work.
        dict(name="decode_hier", op="hier", data="activations", dtype="bf16", rows=16, cols=4096, block=16,
             fmt="e4m3", recipe="absmax", sse=False, keep=True),
        # Serving, a prefill of 8192 tokens: both passes of hierarchical scaling with 4-over-6.
        dict(name="prefill_hier_4over6", op="hier", data="activations", dtype="bf16", rows=8192, cols=4096, block=16,
             fmt="e4m3", recipe="4over6", sse=True, keep=True),
        # A small fp32 matrix, abs-max scales: a few microseconds of work in one launch.
        dict(name="small_f32_absmax", op="quantize", data="normal", dtype="f32", rows=1024, cols=4096, block=16,
             fmt="e4m3", recipe="absmax", sse=True, tscale=False),
        # Offline quantisation of one MLP weight matrix with the plain recipe ...
        dict(name="weights_absmax", op="quantize", data="weights", dtype="bf16", rows=4096, cols=14336, block=16,
             fmt="e4m3", recipe="absmax", sse=True, tscale=False),
        # ... and with 4-over-6 at a small block size, the better recipe of the two.
        dict(name="weights_4over6", op="quantize", data="weights", dtype="bf16", rows=4096, cols=14336, block=8,
             fmt="e4m3", recipe="4over6", sse=True, tscale=False),
        # An odd-sized matrix whose element count is no multiple of 8, smallest blocks, the wide scale
        # format, a per-tensor scale known on the host.
        dict(name="ragged_ue5m3_b2", op="quantize", data="weights", dtype="bf16", rows=2563, cols=4110, block=2,
             fmt="ue5m3", recipe="4over6_pz", sse=True, tscale=True),
        # A decoder layer's seven matrices in one call, as the model sweep does it.
        dict(name="layer_batch", op="batch", data="weights", dtype="bf16", shrink=1, block=32, fmt="e4m3",
             recipe="4over6", sse=True),
        # Offline search of the MSE-optimal scales: every code, and the pruned form with the same
        # result.  The largest work per element.
        dict(name="weights_brute", op="quantize", data="weights", dtype="bf16", rows=4096, cols=14336, block=16,
             fmt="e4m3", recipe="brute", sse=True, tscale=False),
        dict(name="weights_pruned_b4", op="quantize", data="weights", dtype="bf16", rows=4096, cols=14336, block=4,
             fmt="ue5m3", recipe="brute_pruned", sse=True, tscale=False),
        # The numerical study: fp32 blocks of growing standard deviation, one block per row, searched.
        dict(name="study_brute_f32", op="quantize", data="study", dtype="f32", rows=STUDY_SIGMAS * 5000, cols=8,
             block=8, fmt="e4m3", recipe="brute", sse=True, tscale=False),
        # Reading a quantised weight matrix back.
        dict(name="dequant_weights", op="dequant", data="weights", dtype="bf16", rows=4096, cols=14336, block=16,
             fmt="e4m3", recipe="4over6", hier=False),
        # Diagnostics of a quantised tensor: the clipping-only error and both histograms.
        dict(name="diagnostics", op="diag", data="weights", dtype="bf16", rows=4096, cols=4096, block=16,
             fmt="e4m3", recipe="absmax"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("quantize",) * 6 + ("hier",) * 3 + ("search",) * 4 + ("dequant",) * 3 + ("batch", "diag"))
    dtype = rng.choice(("bf16", "bf16", "f32"))
    block = rng.choice(BLOCKS)
    fmt = rng.choice(("e4m3", "e4m3", "ue5m3", "e8m0"))
    recipe = "absmax" if fmt == "e8m0" else rng.choice(("absmax", "absmax_pz", "4over6", "4over6_pz"))
    data = rng.choice(("weights", "weights", "activations", "normal"))
    if op == "batch":
        return dict(op=op, data="weights", dtype=dtype, shrink=_log_int(rng, 2, 32), block=block, fmt=fmt,
                    recipe=recipe, sse=rng.random() < 0.7)
    # sizes over the whole range, odd ones among them
    limit = 4096 * 14336
    if op == "search":
        recipe = "brute" if fmt == "e8m0" else rng.choice(("brute", "brute_pruned", "brute_pruned"))
        if recipe == "brute":
            limit = limit * 126 // CANDIDATES[fmt] // (2 if block >= 64 or block == 2 else 1)
    n = _log_int(rng, 16 * 4096, limit)
    cols = min(_log_int(rng, 256, 14336), n) // block * block
    rows = max(1, n // cols)
    case = dict(op=op, data=data, dtype=dtype, rows=rows, cols=cols, block=block, fmt=fmt, recipe=recipe)
    if op == "hier":
        case.update(sse=rng.random() < 0.5, keep=rng.random() < 0.5)
    elif op in ("quantize", "search"):
        case.update(op="quantize", sse=rng.random() < 0.7, tscale=op == "quantize" and rng.random() < 0.3)
    elif op == "dequant":
        case.update(hier=rng.random() < 0.4)
    return case


def _values(data, dtype, rows, cols, gen):
    """A [rows, cols] tensor with the distribution of the named workload."""
    dev = "cuda"
    z = torch.randn((rows, cols), generator=gen, device=dev, dtype=torch.float32)
    if data == "weights":                                  # 0.02 * Student-t with 4 degrees of freedom
        chi = torch.zeros_like(z)
        for _ in range(4):
            chi += torch.randn(z.shape, generator=gen, device=dev, dtype=torch.float32) ** 2
        z = 0.02 * z / torch.sqrt(chi / 4.0)
    elif data == "activations":                            # 1 % of the channels are 50 times larger
        hot = torch.randperm(cols, generator=gen, device=dev)[: max(1, round(0.01 * cols))]
        z[:, hot] *= 50.0
    elif data == "study":                                  # rows of sigma i, i = 0 .. 150, one after the other
        sigma = torch.linspace(0.0005, 0.05, STUDY_SIGMAS, device=dev)
        z *= sigma.repeat_interleave(rows // STUDY_SIGMAS)[:, None]
    return z.to(DTYPES[dtype]).contiguous()


def _layer_shapes(case):
    """The seven matrices of a decoder layer; draws use smaller layers of the same proportions."""
    k, b = case["shrink"], case["block"]
    return [(max(1, r // k), max(b, c // k // b * b)) for r, c in LAYER_SHAPES.values()]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    state = {"case": case, "fmt": FORMATS[case["fmt"]], "recipe": RECIPES[case["recipe"]], "block": case["block"]}
    if case["op"] == "batch":
        state["xs"] = [_values(case["data"], case["dtype"], r, c, gen) for r, c in _layer_shapes(case)]
        return state
    rows, cols, block = case["rows"], case["cols"], case["block"]
    x = _values(case["data"], case["dtype"], rows, cols, gen)
    state["x"] = x
    if case["op"] == "hier" and case["keep"]:
        state["bufs"] = {"codes_out": torch.empty((rows, cols // 2), dtype=torch.uint8, device=x.device),
                         "scales_out": torch.empty((rows, cols // block), dtype=torch.uint8, device=x.device),
                         "tensor_scale_out": torch.ones(1, dtype=torch.float32, device=x.device)}
        if case["sse"]:
            state["bufs"]["sse_out"] = torch.empty((rows, cols // block), dtype=torch.float32, device=x.device)
        state["word"] = torch.empty(1, dtype=torch.float32, device=x.device)
    elif case["op"] == "quantize":
        state["T"] = 1.0
        if case["tscale"]:
            state["T"] = mxq.tensor_scale_from_absmax(float(mxq.tensor_absmax(x).cpu()[0]), state["fmt"])
    elif case["op"] == "dequant":
        if case["hier"]:
            codes, scales, _, t = mxq.quantize_hier(x, block, state["fmt"], state["recipe"], mxq.tensor_absmax(x))
        else:
            codes, scales, _ = mxq.quantize(x, block, state["fmt"], state["recipe"])
            t = 1.0
        del state["x"]
        state.update(codes=codes, scales=scales, T=t)
    elif case["op"] == "diag":
        state["codes"], state["scales"], _ = mxq.quantize(x, block, state["fmt"], state["recipe"])
    return state


def run(state):
    case, fmt, recipe, block = state["case"], state["fmt"], state["recipe"], state["block"]
    op = case["op"]
    if op == "hier":
        x = state["x"]
        if case["keep"]:
            amax = mxq.tensor_absmax(x, out=state["word"])
            return mxq.quantize_hier(x, block, fmt, recipe, amax, want_sse=case["sse"], **state["bufs"])
        return mxq.quantize_hier(x, block, fmt, recipe, mxq.tensor_absmax(x), want_sse=case["sse"])
    if op == "quantize":
        return mxq.quantize(state["x"], block, fmt, recipe, tensor_scale=state["T"], want_sse=case["sse"])
    if op == "batch":
        return mxq.quantize_batch(state["xs"], block, fmt, recipe, want_sse=case["sse"])
    if op == "dequant":
        return mxq.dequantize(state["codes"], state["scales"], block, fmt, state["T"], DTYPES[case["dtype"]])
    clip = mxq.clip_sse(state["x"], state["scales"], block, fmt)
    return clip, mxq.histogram(state["codes"], state["scales"], block)


def work(case):
    """Bytes: inputs once, outputs once.  Operations per element: 1 for the abs-max, 6 per scale tried
    (scale, round, multiply-subtract, square, add), 3 to read an element back."""
    if case["op"] == "batch":
        n = sum(r * c for r, c in _layer_shapes(case))
    else:
        n = case["rows"] * case["cols"]
    size = 2 if case["dtype"] == "bf16" else 4
    coded = n * (0.5 + 1.0 / case["block"])
    if case["op"] == "dequant":
        return {"bytes": coded + size * n, "flops": 3 * n}
    if case["op"] == "diag":
        # clipping-only error: x and the scales in, one fp32 per block out; histograms: codes and scales
        return {"bytes": (size + 5.0 / case["block"]) * n + coded + 2112, "flops": 6 * n}
    tried = {"absmax": 1, "absmax_pz": 1, "4over6": 2, "4over6_pz": 2, "brute": CANDIDATES[case["fmt"]],
             # the winner and the code on either side of it
             "brute_pruned": 3}[case["recipe"]]
    out = coded + (4.0 * n / case["block"] if case["sse"] else 0.0)
    # (hierarchical scaling needs the maximum before the first quotient, but its input only once if it
    # stays on the chip)
    return {"bytes": size * n + out, "flops": (1 + 6 * tried) * n}


def tolerance(case):
    return "exact"
