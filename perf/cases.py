"""The work whose speed counts: passes of a user's program through the public entry points, from one appended token
to the prefill of a 70B-shaped decoder layer.

A case is one of five kinds:

* "layer": the four linears of a decoder layer of a shard (QKV, output projection, gate/up, down), each on an
  activation of its own (attention, normalisation and the gate stand between them in a model), the weights
  pre-quantized once.  The output projection and the down projection are added onto the residual stream.  Options:
  the layer that stands at the shard's border takes the hidden state coded and hands it on coded ("boundary"), or it
  carries low-rank adapters on all four linears ("rank").  Activations are Gaussian with a few large feature
  dimensions (prefill) or heavy-tailed (Student-t with 3 degrees of freedom: decode).
* "vit": the four linears of a vision transformer block, with bias, GELU behind the first MLP linear, residuals.
* "encode", "decode": the blockwise codec on a hidden state.
* "append": new tokens' keys and values coded into a cache, one block per token and head.

Inputs are drawn on the GPU from the seed alone and follow the recipes of paper_2407_19775_amd/workloads.py.
"""
import math

import torch

from paper_2407_19775_amd import binding, workloads

TAU = workloads.TAU


# ------------------------------------------------------------------------------------------------- the cases
def _layer(name, tokens, hidden, qkv, ffn, x, critical=0.0, boundary=0, rank=0):
    return dict(name=name, kind="layer", tokens=tokens, hidden=hidden, qkv=qkv, ffn=ffn, x=x, critical=critical,
                boundary=boundary, rank=rank)


def listed():
    return [
        # The smallest call of a serving loop: one token's keys and values go into the coded cache.
        dict(name="append_1_token", kind="append", tokens=1, heads=32, head_dim=128),
        # The hidden state at a shard's border, both directions; large tensors, one power-of-two block size each.
        dict(name="encode_8192x8192", kind="encode", elements=8192 * 8192, cols=8192, block=256, half_scales=False),
        dict(name="decode_8192x8192", kind="decode", elements=8192 * 8192, cols=8192, block=1024, half_scales=False),
        # Token generation, Llama-7B-shaped: one user, a small batch, a full batch.
        _layer("generate_1", 1, 4096, 12288, 11008, "student_t"),
        _layer("generate_8", 8, 4096, 12288, 11008, "student_t"),
        _layer("generate_32", 32, 4096, 12288, 11008, "student_t"),
        _layer("generate_64", 64, 4096, 12288, 11008, "student_t"),
        # A short prompt of a ragged length, the layer carrying a fine-tuned adapter.
        _layer("prompt_333_adapter", 333, 4096, 12288, 11008, "gaussian", 0.001, rank=16),
        # A prompt whose activations are heavy-tailed: nearly every feature dimension is critical.
        _layer("prompt_256_heavy", 256, 4096, 12288, 11008, "student_t"),
        # Eight images through a ViT-L block.
        dict(name="vit_l_8_images", kind="vit", tokens=1576, width=1024),
        # Prefill inside a Llama-7B-shaped shard, and of a 70B-shaped layer between two borders.
        _layer("prefill_7b_2048", 2048, 4096, 12288, 11008, "gaussian", 0.001),
        _layer("prefill_70b_4096", 4096, 8192, 10240, 28672, "gaussian", 0.001, boundary=256),
    ]


def _log_uniform(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _draw_layer(rng, lo, hi, hidden_lo, hidden_hi, x):
    """Sizes are cut down until the layer costs no more than the 70B-shaped one at 4096 tokens."""
    while True:
        hidden = _log_uniform(rng, hidden_lo, hidden_hi, 16)
        qkv = int(hidden * rng.choice((1.25, 1.5, 3.0))) // 8 * 8
        ffn = int(hidden * rng.uniform(2.5, 4.0)) // 16 * 16
        case = _layer("", _log_uniform(rng, lo, hi), hidden, qkv, ffn, x, rng.uniform(0.0, 0.01) if x == "gaussian" else 0.0)
        del case["name"]
        if work(case)["flops"] <= 7.0e12:
            return case


def draw(rng):
    kind = rng.choice(("encode", "decode", "append", "generate", "generate", "prefill", "prefill", "adapter", "heavy", "vit"))
    if kind in ("encode", "decode"):
        n = _log_uniform(rng, 1 << 16, 1 << 26)        # ragged: the last block is short more often than not
        return dict(kind=kind, elements=n, cols=rng.choice((1024, 4096, 5120, 8192)),
                    block=rng.choice((64, 128, 256, 512, 576, 1024, 2048, 4096)), half_scales=rng.random() < 0.3)
    if kind == "append":
        return dict(kind=kind, tokens=_log_uniform(rng, 1, 2048), heads=rng.choice((8, 12, 32, 40, 64)),
                    head_dim=rng.choice((64, 128, 256)))
    if kind == "vit":
        return dict(kind=kind, tokens=197 * _log_uniform(rng, 1, 32), width=64 * rng.randint(12, 22))
    if kind == "generate":
        return _draw_layer(rng, 1, 128, 1024, 8192, "student_t")
    if kind == "heavy":
        return _draw_layer(rng, 129, 512, 1024, 4096, "student_t")
    case = _draw_layer(rng, 129 if kind == "prefill" else 1, 4096, 1024, 8192, "gaussian")
    if kind == "adapter":
        case["rank"] = 8 * rng.randint(1, 8)
    elif rng.random() < 0.5:
        case["boundary"] = rng.choice((64, 128, 256, 1024))
    return case


# ------------------------------------------------------------------------------------------------- the inputs
def _normal(gen, shape, std=1.0):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std)


def _half(t):
    return t.clamp_(-workloads.FP16_MAX, workloads.FP16_MAX).to(torch.float16)


def _student_t(gen, shape):
    """Student-t with 3 degrees of freedom: a normal over the root of a mean of three squared normals."""
    d = _normal(gen, shape).square_()
    d += _normal(gen, shape).square_()
    d += _normal(gen, shape).square_()
    return _normal(gen, shape).div_(d.div_(3.0).sqrt_().clamp_(min=1e-6))


def _scale_dimensions(gen, x, count, lo, hi):
    dims = torch.randperm(x.shape[1], generator=gen, device="cuda")[:count]
    x[:, dims] *= torch.rand(count, generator=gen, device="cuda").mul_(hi - lo).add_(lo)
    return x


def _activation(gen, M, K, x, critical):
    if x == "student_t":
        return _half(_student_t(gen, (M, K)))
    return _half(_scale_dimensions(gen, _normal(gen, (M, K)), int(round(critical * K)), 8.0, 60.0))


def _linears(case):
    """(name, K, N) in the order in which a block runs them."""
    if case["kind"] == "vit":
        d = case["width"]
        return [("qkv", d, 3 * d), ("proj", d, d), ("fc1", d, 4 * d), ("fc2", 4 * d, d)]
    d, f = case["hidden"], case["ffn"]
    return [("qkv", d, case["qkv"]), ("o", d, d), ("gate_up", d, 2 * f), ("down", f, d)]


def _prepare_linears(case, gen):
    dev = torch.device("cuda")
    M = case["tokens"]
    vit = case["kind"] == "vit"
    boundary, rank = case.get("boundary", 0), case.get("rank", 0)
    std = 0.015 if case.get("hidden", 0) >= 8192 else 0.02
    need, calls = [], []
    hidden = _linears(case)[0][1]
    state = {"case": dict(case), "residual": _activation(gen, M, hidden, case.get("x", "gaussian"), case.get("critical", 0.001))}
    for i, (name, K, N) in enumerate(_linears(case)):
        W = _half(_normal(gen, (K, N), std))
        call = {"w": binding.prequantize_weight(W), "x": _activation(gen, M, K, case.get("x", "gaussian"), case.get("critical", 0.001)),
                "bias": _half(_normal(gen, (N,), 0.1)) if vit else None,
                "lora": (_half(_normal(gen, (rank, K), 0.02)), _half(_normal(gen, (N, rank), 0.02))) if rank else None,
                "add": N == hidden and i in (1, 3), "gelu": vit and name == "fc1",
                "out": torch.empty((M, N), dtype=torch.float16, device=dev)}
        del W
        need.append((K, N))
        calls.append(call)
    if boundary:
        # the hidden state as the shard before this one has sent it; the first call decodes it into its own buffer
        calls[0]["coded"] = binding.quantize_blockwise(calls[0]["x"], boundary) + (boundary,)
        calls[0]["x"] = torch.empty((M, hidden), dtype=torch.float16, device=dev)
        state["codes_out"] = torch.empty(M * hidden, dtype=torch.uint8, device=dev)
        state["absmax_out"] = torch.empty(-(-M * hidden // boundary), dtype=torch.float32, device=dev)
    spaces = [binding.linear_workspace(M, K, N, dev, rank) for K, N in need]
    if boundary:
        spaces.append(binding.linear_workspace(M, need[3][0], need[3][1], dev, exit_block=boundary))
    state["workspace"] = max(spaces, key=torch.Tensor.numel)      # one workspace serves the whole layer
    state["calls"] = calls
    return state


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    if kind in ("layer", "vit"):
        return _prepare_linears(case, gen)
    if kind == "append":
        rows, B = case["tokens"] * case["heads"], case["head_dim"]
        kv = [_half(_normal(gen, (rows, B))) for _ in range(2)]
        return {"case": dict(case), "kv": kv,
                "codes": [torch.empty(rows * B, dtype=torch.uint8, device="cuda") for _ in kv],
                "absmax": [torch.empty(rows, dtype=torch.float32, device="cuda") for _ in kv]}
    n, B, cols = case["elements"], case["block"], case["cols"]
    rows = -(-n // cols)
    x = _half(_scale_dimensions(gen, _student_t(gen, (rows, cols)), max(1, int(round(0.0005 * cols))), 50.0, 50.0)).view(-1)[:n]
    scale = torch.float16 if case["half_scales"] else torch.float32
    state = {"case": dict(case), "x": x.clone(), "codes": torch.empty(n, dtype=torch.uint8, device="cuda"),
             "absmax": torch.empty(-(-n // B), dtype=scale, device="cuda")}
    if kind == "decode":
        binding.quantize_blockwise(state["x"], B, codes=state["codes"], absmax=state["absmax"], fp16_scales=case["half_scales"])
    return state


# ------------------------------------------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "append":
        for x, codes, absmax in zip(state["kv"], state["codes"], state["absmax"]):
            binding.quantize_blockwise(x, case["head_dim"], codes=codes, absmax=absmax)
        return {"codes": state["codes"], "absmax": state["absmax"]}
    if kind == "encode":
        codes, absmax = binding.quantize_blockwise(state["x"], case["block"], codes=state["codes"], absmax=state["absmax"],
                                                   fp16_scales=case["half_scales"])
        return {"codes": codes, "absmax": absmax}
    if kind == "decode":
        return binding.dequantize_blockwise(state["codes"], state["absmax"], case["block"], out=state["x"])
    calls, ws = state["calls"], state["workspace"]
    boundary, rank = case.get("boundary", 0), case.get("rank", 0)
    outs = []
    for i, c in enumerate(calls):
        if boundary and i == 3:
            codes, absmax = binding.mixed_int8_linear_to_codes(c["x"], c["w"], TAU, boundary, residual=state["residual"],
                                                               codes=state["codes_out"], absmax=state["absmax_out"], H=c["out"], workspace=ws)
            outs += [c["out"], codes, absmax]
        elif rank:
            outs.append(binding.mixed_int8_linear(c["x"], c["w"], TAU, out=c["out"], workspace=ws, lora=c["lora"]))
        elif boundary and i == 0:
            binding.mixed_int8_linear(c["x"], c["w"], TAU, out=c["out"], workspace=ws, coded=c["coded"])
            outs += [c["x"], c["out"]]
        else:
            outs.append(binding.mixed_int8_linear(c["x"], c["w"], TAU, bias=c["bias"], out=c["out"], workspace=ws, gelu=c["gelu"],
                                                  residual=state["residual"] if c["add"] else None))
    return outs


# ------------------------------------------------------------------------------------------------- what it takes
def work(case):
    """Bytes: activations, residuals and outputs in fp16, weights as codes; each read or written once.  Operations: two
    per weight and row, whichever of the two products the row's element goes through."""
    kind = case["kind"]
    if kind == "append":
        n, B, width, copies = case["tokens"] * case["heads"] * case["head_dim"], case["head_dim"], 4, 2
    elif kind in ("encode", "decode"):
        n, B, width, copies = case["elements"], case["block"], 2 if case["half_scales"] else 4, 1
    if kind in ("append", "encode", "decode"):
        # a lookup, a comparison and a product per element
        return {"bytes": copies * (3 * n + width * -(-n // B)), "flops": copies * 3 * n}
    M, rank, boundary = case["tokens"], case.get("rank", 0), case.get("boundary", 0)
    nbytes, ops = 0, 0
    for i, (_, K, N) in enumerate(_linears(case)):
        nbytes += K * N + 4 * N + 2 * M * K + 2 * M * N + (2 * N if kind == "vit" else 0)
        ops += 2 * M * K * N + 2 * M * rank * (K + N)
        nbytes += 2 * rank * (K + N)
        if i in (1, 3) and not rank:
            nbytes += 2 * M * N                        # the residual stream
        if boundary and i == 0:
            nbytes += M * K + 4 * -(-M * K // boundary)
        if boundary and i == 3:
            nbytes += M * N + 4 * -(-M * N // boundary)
    return {"bytes": nbytes, "flops": ops}


def tolerance(case):
    """The codec is defined bit for bit.  The layer's outputs are rounded to fp16 once (twice with GELU or a residual)
    behind an exact integer product and an fp32 sum.  Against the same sums in 64 bits: rel 3e-4 where the 16-bit
    weights of critical dimensions are rounded once less than the definition says (5e-6 where they are not), max 4e-3
    (one fp16 step before the residual is added); an fp16 step in the output moves a code of the boundary now and then."""
    if case["kind"] in ("append", "encode", "decode"):
        return "exact"
    return {"rel": 1.2e-3, "max": 1.5e-2, "differ": 2e-3 if case.get("boundary") else 0.0}
