"""The calls whose time counts: what a program built on this library has it do, from one token of a
draft model to the prompt of a request, with the sizes of the 7B- and 70B-shaped stacks of `synth.py`.

A case is a dict of plain values with a "kind":

- "linear"  y = x W^T on MXFP4 weights, with any of bias, gate (interleaved rows) and residual behind it,
            on the row-major weights or on their tile-major copy;
- "step"    the linears of one decoder layer (and the LM head with its pick) at one token, one grouped call;
- "head"    the LM head of a verification pass: product, greedy pick, comparison with the draft's tokens;
- "draft"   the product on one of the other element formats;
- "target"  the product on unquantised BF16 weights;
- "cast"    BF16 weights to MXFP4.

Weights are heavy-tailed and activations have a few large channels, as in `synth.py`.
"""
import math

import torch

from paper_2503_13565_amd import binding, synth

DEV = "cuda"

# Formats: (largest exponent of an element, bits per weight of a block's elements, magnitudes by code).


def _grid(exp_bits, man_bits, bias, largest):
    got = []
    for e in range(1 << exp_bits):
        for m in range(1 << man_bits):
            f = m / (1 << man_bits)
            got.append(f * 2.0 ** (1 - bias) if e == 0 else (1 + f) * 2.0 ** (e - bias))
    return [v for v in got if v <= largest]


FORMATS = {
    "mxfp4": (2, 4, _grid(2, 1, 1, 6.0)),
    "e4m3": (8, 8, _grid(4, 3, 7, 448.0)),
    "e2m3": (2, 6, _grid(2, 3, 1, 7.5)),
    "e5m2": (15, 8, _grid(5, 2, 15, 57344.0)),
    "e3m2": (4, 6, _grid(3, 2, 3, 28.0)),
    "t2": (0, 2, [0.0, 1.0]),
}
FMT_IDS = {"e5m2": binding.FMT_E5M2, "e3m2": binding.FMT_E3M2, "t2": binding.FMT_T2}


def listed():
    return [
        # drafting: one linear for one token, the smallest call (bounded by latency and launch)
        {"name": "decode_linear", "kind": "linear", "m": 1, "n": 4096, "k": 4096, "act": 0, "bias": False,
         "residual": False, "tiled": False},
        # drafting: the linears of a 7B layer and the LM head's pick for one token, as one grouped call
        {"name": "decode_step_7b", "kind": "step", "hidden": 4096, "mlp": 11008, "kv": 4096, "vocab": 32000},
        # drafting with a 70B-shaped model: one layer for one token
        {"name": "decode_layer_70b", "kind": "step", "hidden": 8192, "mlp": 28672, "kv": 1024, "vocab": 0},
        # verifying four draft tokens: gate and up projections with the gate applied
        {"name": "verify_gate", "kind": "linear", "m": 5, "n": 22016, "k": 4096, "act": 1, "bias": False,
         "residual": False, "tiled": False},
        # verifying eight draft tokens: the LM head with pick and acceptance
        {"name": "verify_head", "kind": "head", "fmt": "mxfp4", "m": 9, "n": 32000, "k": 4096},
        # verifying seven draft tokens: the down projection on the tile-major copy
        {"name": "verify_down_tiled", "kind": "linear", "m": 8, "n": 4096, "k": 11008, "act": 0, "bias": False,
         "residual": False, "tiled": True},
        # several sequences verified together: the largest row count of the verification sweep
        {"name": "batch_qkv", "kind": "linear", "m": 32, "n": 12288, "k": 4096, "act": 0, "bias": True,
         "residual": False, "tiled": False},
        # the prompt of a request goes through the quantised model before it can draft
        {"name": "prefill_gate", "kind": "linear", "m": 509, "n": 22016, "k": 4096, "act": 1, "bias": False,
         "residual": False, "tiled": False},
        # an 8-bit draft model: one token
        {"name": "draft_e4m3", "kind": "draft", "fmt": "e4m3", "m": 1, "n": 22016, "k": 4096},
        # the unquantised target verifying four draft tokens
        {"name": "target_qkv", "kind": "target", "m": 5, "n": 12288, "k": 4096},
        # an eighth of the down projection's inputs (11008 / 8 is no multiple of 128): ragged K
        {"name": "verify_ragged", "kind": "linear", "m": 7, "n": 4096, "k": 1376, "act": 0, "bias": False,
         "residual": True, "tiled": False},
        # loading a model: one weight tensor is cast
        {"name": "cast_gate", "kind": "cast", "n": 22016, "k": 4096},
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "linear", "step", "head", "draft", "target", "cast"])
    n = _log(rng, 256, 32000)
    k = 128 * _log(rng, 4, 96) if rng.random() < 0.75 else 32 * _log(rng, 16, 384)
    if kind == "step":                                  # one layer of a model of any width, with or without a head
        hidden, mlp = 128 * rng.randint(6, 64), 128 * rng.randint(16, 200)
        return {"kind": kind, "hidden": hidden, "mlp": mlp, "kv": hidden // rng.choice([1, 4, 8]),
                "vocab": rng.choice([0, rng.randint(8000, 33000)])}
    if kind == "head":
        return {"kind": kind, "fmt": rng.choice(["mxfp4", "mxfp4", "bf16"]), "m": _log(rng, 2, 32),
                "n": rng.randint(8000, 33000), "k": 128 * rng.randint(6, 40)}
    if kind == "draft":
        return {"kind": kind, "fmt": rng.choice(["e4m3", "e2m3", "e5m2", "e3m2", "t2"]), "m": _log(rng, 1, 64),
                "n": n, "k": 128 * max(1, k // 128)}
    if kind == "target":
        return {"kind": kind, "m": _log(rng, 1, 64), "n": n, "k": k}
    if kind == "cast":
        return {"kind": kind, "n": n, "k": k}
    m, act, tiled = _log(rng, 1, 512), rng.choice([0, 0, 1]), rng.random() < 0.25
    bias, residual = rng.random() < 0.3, rng.random() < 0.4
    if tiled:                                           # verification passes; fused, K is not split there
        m, k, bias, residual = min(m, 4 if act else 32), 128 * max(1, k // 128), False, False
    while m * n * k > 509 * 22016 * 4096:               # no more work than the listed prompt
        n = max(256, n // 2)
    return {"kind": kind, "m": m, "n": n + n % 2 if act else n, "k": k, "act": act, "bias": bias,
            "residual": residual, "tiled": tiled}


# ---- inputs -----------------------------------------------------------------------------------


def _weights(n, k, seed):
    return synth.weights_student_t(n, k, seed=seed, device=DEV)


def _rows(m, k, seed):
    return synth.activations_outlier_channels(m, k, seed=seed, device=DEV)


def _vector(shape, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device=DEV) * 0.3).to(torch.bfloat16)


def _links(case):
    """(n, k, act, residual) of the linears of a "step"."""
    h, mlp = case["hidden"], case["mlp"]
    return [(h + 2 * case["kv"], h, 0, False), (h, h, 0, True), (2 * mlp, h, 1, False), (h, mlp, 0, True)]


def _inputs(case, seed):
    """Every tensor of a case before any of it is cast, from the seed alone."""
    at = seed * 64
    if case["kind"] == "step":
        d = {"w": [], "x": [], "res": []}
        for i, (n, k, _, res) in enumerate(_links(case)):
            d["w"].append(_weights(n, k, at + 4 * i))
            d["x"].append(_rows(1, k, at + 4 * i + 1))   # (the down projection reads the gate's output instead)
            d["res"].append(_vector((1, n), at + 4 * i + 2) if res else None)
        if case["vocab"]:
            d["w"].append(_weights(case["vocab"], case["hidden"], at + 32))
            d["x"].append(_rows(1, case["hidden"], at + 33))
        return d
    n, k = case["n"], case["k"]
    d = {"w": _weights(n, k, at)}
    if case["kind"] != "cast":
        d["x"] = _rows(case["m"], k, at + 1)
    if case["kind"] == "linear":
        c = n // 2 if case["act"] else n
        d["bias"] = _vector((n,), at + 2) if case["bias"] else None
        d["res"] = _vector((case["m"], c), at + 3) if case["residual"] else None
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "cast":
        return {"case": case, "w": d["w"]}
    if kind == "step":
        pairs = [binding.mxfp4_direct_cast(w) for w in d["w"]]
        items = []
        for i, (_, _, act, _) in enumerate(_links(case)):
            items.append({"x": d["x"][i], "q": pairs[i][0], "s": pairs[i][1], "act": act, "residual": d["res"][i]})
        # the down projection reads what gate and up wrote
        items[2]["y"] = items[3]["x"] = torch.empty((1, case["mlp"]), dtype=torch.bfloat16, device=DEV)
        if case["vocab"]:
            items.append({"x": d["x"][4], "q": pairs[4][0], "s": pairs[4][1], "argmax": True})
        return {"case": case, "group": binding.GemmGroup(items)}
    m, n, k = case["m"], case["n"], case["k"]
    state = {"case": case, "x": d["x"]}
    if kind == "target":
        state["w"] = d["w"]
    elif kind == "draft":
        cast = {"e4m3": binding.mxfp4_e4m3_direct_cast, "e2m3": binding.mxfp4_e2m3_direct_cast}.get(case["fmt"])
        state["q"], state["s"] = cast(d["w"]) if cast else binding.mxfp4_fmt_direct_cast(FMT_IDS[case["fmt"]], d["w"])
    elif kind == "head":
        # the draft's tokens: the picks of the same weights at another precision, so that some are accepted
        if case["fmt"] == "bf16":
            state["w"] = d["w"]
            need = binding.mxfp4_bf16_gemm_argmax_workspace_bytes(m, n, k)
            other = _product(d["x"], d["w"], "mxfp4")
        else:
            state["q"], state["s"] = binding.mxfp4_direct_cast(d["w"])
            need = binding.mxfp4_woq_gemm_argmax_workspace_bytes(m, n, k)
            other = _product(d["x"], d["w"], None)
        state["draft"] = other.argmax(dim=1).to(torch.int32)[: m - 1].contiguous()
        state["ws"] = torch.empty((need,), dtype=torch.uint8, device=DEV)
    else:
        state["q"], state["s"] = binding.mxfp4_direct_cast(d["w"])
        state["bias"], state["res"] = d["bias"], d["res"]
        if case["tiled"]:
            state["tiles"] = binding.mxfp4_tile_repack(state.pop("q"), state.pop("s"))
        need = binding.mxfp4_woq_gemm_workspace_bytes(m, n, k)
        state["ws"] = torch.empty((need,), dtype=torch.uint8, device=DEV) if need else None
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "cast":
        return binding.mxfp4_direct_cast(state["w"])
    if kind == "step":
        state["group"].run()
        return state["group"].ys
    if kind == "target":
        return binding.mxfp4_bf16_gemm(state["x"], state["w"])
    if kind == "draft":
        if case["fmt"] == "e4m3":
            return binding.mxfp4_e4m3_woq_gemm(state["x"], state["q"], state["s"])
        if case["fmt"] == "e2m3":
            return binding.mxfp4_e2m3_woq_gemm(state["x"], state["q"], state["s"])
        return binding.mxfp4_fmt_woq_gemm(FMT_IDS[case["fmt"]], state["x"], state["q"], state["s"])
    if kind == "head":
        if case["fmt"] == "bf16":
            return binding.mxfp4_bf16_gemm_verify(state["x"], state["w"], state["draft"], workspace=state["ws"])
        return binding.mxfp4_woq_gemm_verify(state["x"], state["q"], state["s"], state["draft"], workspace=state["ws"])
    if case["tiled"]:
        if case["act"]:
            return binding.mxfp4_woq_gemm_tiled_fused(state["x"], state["tiles"], act=case["act"])
        return binding.mxfp4_woq_gemm_tiled(state["x"], state["tiles"], workspace=state["ws"])
    if case["act"] or case["bias"] or case["residual"]:
        return binding.mxfp4_woq_gemm_fused(state["x"], state["q"], state["s"], bias=state["bias"], act=case["act"],
                                            residual=state["res"], workspace=state["ws"])
    return binding.mxfp4_woq_gemm(state["x"], state["q"], state["s"], workspace=state["ws"])


# ---- what a pass cannot do without, and what it should give -------------------------------------


def _packed(n, k, fmt):
    return n * k * FORMATS[fmt][1] // 8 + n * k // 32


def work(case):
    kind = case["kind"]
    if kind == "cast":
        return {"bytes": 2 * case["n"] * case["k"] + _packed(case["n"], case["k"], "mxfp4"), "flops": 0}
    if kind == "step":
        data = flops = 0
        for n, k, act, res in _links(case):
            c = n // 2 if act else n
            data += _packed(n, k, "mxfp4") + 2 * k + 2 * c * (2 if res else 1)
            flops += 2 * n * k
        if case["vocab"]:
            data += _packed(case["vocab"], case["hidden"], "mxfp4") + 2 * case["hidden"] + 8
            flops += 2 * case["vocab"] * case["hidden"]
        return {"bytes": data, "flops": flops}
    m, n, k = case["m"], case["n"], case["k"]
    plain = kind == "target" or case.get("fmt") == "bf16"
    data = (2 * n * k if plain else _packed(n, k, case.get("fmt", "mxfp4"))) + 2 * m * k
    if kind == "head":
        data += 12 * m
    else:
        c = n // 2 if case.get("act") else n
        data += 2 * m * c * (2 if case.get("residual") else 1) + (2 * n if case.get("bias") else 0)
    return {"bytes": data, "flops": 2 * m * n * k}


def tolerance(case):
    if case["kind"] == "cast":
        return "exact"
    if case["kind"] == "head":                          # picks and float32 sums
        return {"rel": 1e-5, "max": 1e-4}
    # BF16 results: 1.7e-3 is what their rounding alone leaves against 64 bits; two units in the last place at most
    return {"rel": 7e-3, "max": 2.0 ** -6}


def _hat(w, fmt):
    """The values that BF16 weights take in a format, in 64 bits: blocks of 32 along the row, scale a power
    of two from the block's largest magnitude, elements rounded to nearest, ties to the even code."""
    emax, _, grid = FORMATS[fmt]
    n, k = w.shape
    v = w.double().reshape(n, k // 32, 32)
    _, e = torch.frexp(v.abs().amax(dim=2, keepdim=True))
    # the exponent field written out: a power function on the device need not give exact powers of two
    scale = (((e.long() - 1 - emax).clamp(min=-127) + 1023) << 52).view(torch.float64)
    values = torch.tensor(grid, dtype=torch.float64, device=w.device)
    middles = (values[1:] + values[:-1]) / 2
    r = v.abs() / scale
    low, high = torch.bucketize(r, middles), torch.bucketize(r, middles, right=True)
    code = torch.where(low % 2 == 0, low, high)
    return (values[code] * scale * torch.sign(v)).reshape(n, k)


def _product(x, w, fmt):
    """x times the weights (as they are, or in a format), in 64 bits."""
    x64, out = x.double(), []
    for r in range(0, w.shape[0], 2048):
        part = w[r:r + 2048]
        out.append(x64 @ (part.double() if fmt is None else _hat(part, fmt)).t())
    return torch.cat(out, dim=1)


def _gated(z, act):
    return z[:, 0::2] / (1 + torch.exp(-z[:, 0::2])) * z[:, 1::2] if act else z


def _plus(t, res):
    return t if res is None else t + res.double()


def exact(case, seed):
    kind = case["kind"]
    if kind == "cast":                                  # whole numbers, compared as they are
        return None
    d = _inputs(case, seed)
    if kind == "step":
        out = []
        for i, (_, _, act, _) in enumerate(_links(case)):
            x = out[2] if i == 3 else d["x"][i]
            out.append(_plus(_gated(_product(x, d["w"][i], "mxfp4"), act), d["res"][i]))
        if case["vocab"]:
            value, index = _product(d["x"][4], d["w"][4], "mxfp4").max(dim=1)
            out.append((index.to(torch.int32), value))
        return out
    if kind == "target":
        return _product(d["x"], d["w"], None)
    if kind == "draft":
        return _product(d["x"], d["w"], case["fmt"])
    if kind == "head":
        value, index = _product(d["x"], d["w"], None if case["fmt"] == "bf16" else "mxfp4").max(dim=1)
        return None, index.to(torch.int32), value
    z = _product(d["x"], d["w"], "mxfp4")
    if d["bias"] is not None:
        z = z + d["bias"].double()
    return _plus(_gated(z, case["act"]), d["res"])
