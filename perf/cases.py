"""What is timed of this framework: its entry points over the sizes, element types and head sizes it is used at.

Five of the listed cases are the configurations that the benchmark reports (one small fp32 head, the dedicated row
softmax, three sizes of the fused weights); the others are the shapes off them that the benchmark's own shape list
holds: an odd class-token length, fp32 weights, the unfused three-kernel pipeline on rows off the 16-byte
boundaries, and the attention output on many heads, on one head, on a wide head and in fp32.
"""
import math

import torch

import paper_2407_13885_amd as attnw

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
_CODE = {"bf16": attnw.ATTNW_BF16, "f32": attnw.ATTNW_F32}
_SIZE = {"bf16": 2, "f32": 4}


def _qk(call, dtype, batch, heads, tokens, head_size, sharp=False):
    return {"call": call, "dtype": dtype, "batch": batch, "heads": heads, "tokens": tokens, "head_size": head_size,
            "sharp": sharp}


def _rows(in_dtype, out_dtype, rows, cols):
    return {"call": "softmax", "dtype": in_dtype, "out_dtype": out_dtype, "rows": rows, "cols": cols}


def listed():
    cases = [
        # one short head in fp32: the smallest call, a launch and its latency
        ("weights-f32-one-head", _qk("weights", "f32", 1, 1, 128, 64)),
        # weights of a class-token length (14 x 14 patches and one): no row of P but the first is 16-byte aligned
        ("weights-bf16-n197", _qk("weights", "bf16", 64, 16, 197, 64)),
        # an encoder layer of 1024 tokens, a batch of four
        ("weights-bf16-n1024", _qk("weights", "bf16", 4, 12, 1024, 64)),
        # the paper's head size and its longest fused sequence
        ("weights-bf16-n4096", _qk("weights", "bf16", 1, 16, 4096, 128)),
        # long context, rows of every sharpness: 4 GiB of weights, the largest output
        ("weights-bf16-n16384", _qk("weights", "bf16", 1, 8, 16384, 64, sharp=True)),
        # full precision weights, as for analysing a model
        ("weights-f32-n2048", _qk("weights", "f32", 1, 16, 2048, 64)),
        # the dedicated row softmax over scores made elsewhere, some of them peaked
        ("softmax-bf16-2048", _rows("bf16", "bf16", 24576, 2048)),
        # multiply, scaling and softmax as three kernels, over an odd length
        ("unfused-bf16-n1025", _qk("unfused", "bf16", 8, 16, 1025, 64)),
        # attention output: many heads, ...
        ("attention-bf16-n4096", _qk("attention", "bf16", 1, 16, 4096, 128)),
        # ... a single head, which has to be spread over the chip, ...
        ("attention-bf16-one-head", _qk("attention", "bf16", 1, 1, 4096, 128)),
        # ... the widest heads, ...
        ("attention-bf16-d256", _qk("attention", "bf16", 1, 16, 4096, 256)),
        # ... and full precision
        ("attention-f32-n4096", _qk("attention", "f32", 1, 16, 4096, 128)),
    ]
    return [dict(case, name=name) for name, case in cases]


def _spread(rng, low, high):
    """A whole number between low and high, even over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    call = rng.choice(["weights", "weights", "weights", "softmax", "unfused", "attention", "attention", "attention"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if call == "softmax":
        out = rng.choice([dtype, dtype, "bf16"])
        cols = _spread(rng, 8, 131072)
        if rng.random() < 0.5:
            cols = (cols + 7) // 8 * 8
        elements = _spread(rng, 1 << 18, 1 << 27)
        return _rows(dtype, out, max(1, elements // cols), cols)
    step = 4 if dtype == "f32" else 16
    head_size = rng.choice([32, 64, 64, 128, 128, 256, rng.randrange(step, 257, step)])
    tokens = _spread(rng, 32, 8192 if dtype == "bf16" else 4096)
    if rng.random() < 0.5:
        tokens = (tokens + 31) // 32 * 32
    # heads: from one to as many as the largest listed case of the kind affords
    if call == "attention":
        flops = 2.2e11 if dtype == "bf16" else 1.0e11
        most = flops / (4.0 * tokens * tokens * head_size)
    else:
        elements = (1 << 28) if dtype == "bf16" else (1 << 26)
        most = elements / (tokens * max(tokens, head_size))
    all_heads = _spread(rng, 1, max(1.0, min(most, 8192.0)))
    heads = min(all_heads, rng.choice([1, 4, 8, 12, 16]))
    sharp = call != "unfused" and rng.random() < 0.25
    return _qk(call, dtype, max(1, all_heads // heads), heads, tokens, head_size, sharp=sharp)


def _normal(generator, shape, dtype, sharp=False):
    x = torch.randn(shape, generator=generator, device="cuda", dtype=torch.float32)
    if sharp:   # every row times a factor of its own: flat and peaked rows side by side
        x *= 0.5 + 2.5 * torch.rand(shape[:-1] + (1,), generator=generator, device="cuda")
    return x.to(_TORCH[dtype])


def prepare(case, seed):
    generator = torch.Generator(device="cuda").manual_seed(seed)
    state = dict(case)
    dtype = case["dtype"]
    if case["call"] == "softmax":
        shape = (case["rows"], case["cols"])
        scores = 2.0 * torch.randn(shape, generator=generator, device="cuda", dtype=torch.float32)
        peaked = torch.rand(shape, generator=generator, device="cuda") < 0.01
        state["S"] = scores.masked_fill_(peaked, 8.0).to(_TORCH[dtype])
        state["P"] = torch.empty(shape, device="cuda", dtype=_TORCH[case["out_dtype"]])
        return state
    lead = (case["batch"], case["heads"], case["tokens"])
    state["Q"] = _normal(generator, lead + (case["head_size"],), dtype, case["sharp"])
    state["K"] = _normal(generator, lead + (case["head_size"],), dtype, case["sharp"])
    if case["call"] == "attention":
        state["V"] = _normal(generator, lead + (case["head_size"],), dtype)
        state["O"] = torch.empty_like(state["Q"])
    else:
        state["P"] = torch.empty(lead + (case["tokens"],), device="cuda", dtype=_TORCH[dtype])
        if case["call"] == "unfused":
            state["S"] = torch.empty_like(state["P"])
    return state


def run(state):
    stream = torch.cuda.current_stream()
    code = _CODE[state["dtype"]]
    if state["call"] == "softmax":
        if state["out_dtype"] == state["dtype"]:
            attnw.attnw_softmax(state["S"], state["P"], state["rows"], state["cols"], code, stream)
        else:
            attnw.attnw_softmax_cast(state["S"], state["P"], state["rows"], state["cols"], code,
                                     _CODE[state["out_dtype"]], stream)
        return state["P"]
    B, H, N, d = state["batch"], state["heads"], state["tokens"], state["head_size"]
    scale = d ** -0.5
    if state["call"] == "weights":
        attnw.attnw_fused(state["Q"], state["K"], state["P"], B, H, N, d, scale, code, stream)
        return state["P"]
    if state["call"] == "attention":
        attnw.attnw_attention(state["Q"], state["K"], state["V"], state["O"], B, H, N, d, scale, code, stream)
        return state["O"]
    attnw.attnw_gemm_scores(state["Q"], state["K"], state["S"], B, H, N, d, 1.0, code, stream)
    attnw.attnw_scale(state["S"], state["S"], B * H * N * N, scale, code, stream)
    attnw.attnw_softmax(state["S"], state["P"], B * H * N, N, code, stream)
    return state["S"], state["P"]


def work(case):
    size = _SIZE[case["dtype"]]
    if case["call"] == "softmax":
        elements = case["rows"] * case["cols"]
        return {"bytes": elements * (size + _SIZE[case["out_dtype"]]), "flops": 4 * elements}
    heads, N, d = case["batch"] * case["heads"], case["tokens"], case["head_size"]
    if case["call"] == "attention":
        return {"bytes": 4 * size * heads * N * d, "flops": 4 * heads * N * N * d}
    outputs = 2 if case["call"] == "unfused" else 1
    return {"bytes": size * heads * N * (2 * d + outputs * N), "flops": 2 * heads * N * N * d}


def tolerance(case):
    # about four times the largest error of each kind of case against the same computed in 64 bits: weights and softmax
    # rows are rounded once at the store (bf16: 1.7e-3 and 3.9e-3), the attention output also rounds its weights (bf16:
    # 2.3e-3 and 1.1e-2), the unfused pipeline its scores, twice (bf16: 5.4e-3 and 2.2e-2); fp32 with sharp rows and wide
    # heads 2.1e-6 and 5.3e-5
    if case.get("out_dtype", case["dtype"]) == "bf16":
        return {"weights": {"rel": 7e-3, "max": 1.6e-2}, "softmax": {"rel": 7e-3, "max": 1.6e-2},
                "attention": {"rel": 1e-2, "max": 4e-2}, "unfused": {"rel": 2e-2, "max": 9e-2}}[case["call"]]
    if case["call"] == "softmax":
        return {"rel": 3e-7, "max": 1.2e-6}
    return {"rel": 8e-6, "max": 2e-4}
