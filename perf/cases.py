"""The work that users of this framework have it do, as a list of cases to measure.

A case is one pass through the public entry points (`binding.Context`): a layer group or a layer stack over a
hybrid batch of decode and prefill tokens, or the four step calls one after the other.  Shapes are those of
`inputs.WORKLOADS` (the five baseline workloads and the second model family) and, in `draw`, sizes of the same
ranges: hidden sizes of 256 to 4096, 8 to 128 experts, batches from one token to a whole 8192-token prompt.
"""
import math

import torch

from paper_2510_08055_amd import binding, inputs

DEV = "cuda:0"

# What a case may leave out.  call: "group" (moe_group_forward), "stack" (moe_stack_forward), "steps" (the four step
# calls).  schedule / chunk / groups / granule: as the entry points take them.  zipf: the per-expert router bias is
# -zipf * ln(rank), which makes some experts popular.
DEFAULTS = {"call": "group", "schedule": "layered", "chunk": 0, "groups": 0, "granule": 512, "layers": 1, "D": 0, "P": 0,
            "dtype": "bf16", "weights": "", "residual": True, "y_perm_f32": False, "act_split": False, "zipf": 0.0}

QWEN3 = {"H": 2048, "E": 128, "K": 8, "I": 768}
GPTOSS = {"H": 2880, "E": 32, "K": 4, "I": 2880}
MIXTRAL = {"H": 4096, "E": 8, "K": 2, "I": 14336}
LARGE = {"H": 2880, "E": 128, "K": 4, "I": 2880}
TINY = {"H": 256, "E": 8, "K": 2, "I": 512}


def listed():
    return [
        # one user's decode step: 8 of 128 experts, a few layers in a row; launches and latency are what it costs
        {"name": "decode_one", **QWEN3, "layers": 4, "D": 1},
        # the usual decode batch of a stable server (up to 32 in the arXiv trace): nearly every expert, one or two rows each
        {"name": "decode_batch", **QWEN3, "layers": 2, "D": 32},
        # chunked prefill at the paper's chunk of 512 beside 128 decode rows: every chunk streams the weights again
        {"name": "chunked_prefill", **QWEN3, "layers": 2, "D": 128, "P": 1536, "schedule": "chunked", "chunk": 512},
        # one layer over a hybrid batch with a 2048-token chunk (the `qwen3_layer` workload)
        {"name": "hybrid_layer", **QWEN3, "D": 64, "P": 2048, "residual": False},
        # layered prefill of a whole 8192-token prompt through a layer group (the `qwen3_group8` workload, half its layers)
        {"name": "layered_prefill", **QWEN3, "layers": 4, "D": 128, "P": 8192},
        # the whole-stack driver with the group-count rule: 3 groups of 2 layers, a ragged prompt, 32 decode rows
        {"name": "stack", **QWEN3, "call": "stack", "layers": 6, "D": 32, "P": 1357},
        # few wide experts under skewed routing, the intermediate held as a pair (the `mixtral_zipf` workload)
        {"name": "skewed_wide", **MIXTRAL, "D": 32, "P": 4096, "residual": False, "y_perm_f32": True, "act_split": True,
         "zipf": 1.2},
        # decode over large experts, bound by streaming the weights (the `decode_large` workload, one of its layers)
        {"name": "decode_large", **LARGE, "D": 256, "y_perm_f32": True},
        # the same with 4-bit expert weights (the `decode_large_w4` workload, two of its layers)
        {"name": "decode_large_w4", **LARGE, "layers": 2, "D": 256, "y_perm_f32": True, "weights": "mxfp4"},
        # the second model family as it ships: 4-bit experts under a hybrid batch (the `gptoss_layer_w4` workload)
        {"name": "hybrid_w4", **GPTOSS, "D": 64, "P": 2048, "residual": False, "weights": "mxfp4"},
        # a caller with a schedule of its own: router, permutation, grouped FFN and combine one by one, a ragged batch
        {"name": "steps", **GPTOSS, "call": "steps", "D": 1029},
        # the fp32 path (the `tiny_f32` workload)
        {"name": "tiny_f32", **TINY, "P": 64, "dtype": "f32", "residual": False},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above; it costs no more than the largest listed one."""
    kind = rng.choice(["decode", "decode", "chunked", "layered", "layered", "stack", "skewed", "large", "w4_decode",
                       "w4_hybrid", "steps", "odd", "f32"])
    if kind == "decode":
        return {**QWEN3, "layers": rng.randint(1, 4), "D": _log_int(rng, 1, 256)}
    if kind == "chunked":
        chunk = rng.choice([256, 512, 768, 1024])
        return {**QWEN3, "layers": rng.randint(1, 2), "D": _log_int(rng, 1, 128), "P": rng.randint(chunk + 1, 3 * chunk),
                "schedule": "chunked", "chunk": chunk}
    if kind == "layered":
        shape, longest = rng.choice([(QWEN3, 8192), (QWEN3, 8192), (GPTOSS, 4096)])
        return {**shape, "layers": rng.randint(1, 2), "D": _log_int(rng, 1, 128), "P": _log_int(rng, 128, longest),
                "residual": rng.random() < 0.7}
    if kind == "stack":
        layers = rng.randint(2, 4)
        return {**QWEN3, "call": "stack", "layers": layers, "D": _log_int(rng, 1, 64), "P": rng.randint(100, 2000),
                "groups": rng.choice([0, 0, 1, layers])}
    if kind == "skewed":
        split = rng.random() < 0.5
        return {**MIXTRAL, "D": rng.randint(1, 64), "P": _log_int(rng, 64, 3500), "residual": False, "y_perm_f32": True,
                "act_split": split, "zipf": rng.choice([0.0, 0.6, 1.2])}
    if kind == "large":
        return {**LARGE, "D": _log_int(rng, 4, 512), "y_perm_f32": rng.random() < 0.5}
    if kind == "w4_decode":
        return {**rng.choice([LARGE, GPTOSS]), "layers": rng.randint(1, 2), "D": _log_int(rng, 1, 512),
                "y_perm_f32": rng.random() < 0.5, "weights": "mxfp4"}
    if kind == "w4_hybrid":
        return {**GPTOSS, "D": _log_int(rng, 1, 64), "P": _log_int(rng, 256, 4096), "residual": False, "weights": "mxfp4"}
    if kind == "steps":
        return {**rng.choice([QWEN3, GPTOSS]), "call": "steps", "D": _log_int(rng, 16, 4096)}
    if kind == "odd":      # other model shapes, sizes that are multiples of 8 only
        return {"H": 8 * rng.randint(32, 384), "E": rng.randint(4, 96), "K": rng.randint(1, 4), "I": 8 * rng.randint(24, 256),
                "D": _log_int(rng, 1, 64), "P": _log_int(rng, 16, 2048), "layers": rng.randint(1, 2)}
    return {"H": 64 * rng.randint(2, 8), "E": rng.choice([4, 8, 16]), "K": rng.randint(1, 4), "I": 64 * rng.randint(2, 12),
            "P": _log_int(rng, 16, 128), "dtype": "f32", "residual": rng.random() < 0.5}


def _full(case):
    return {**DEFAULTS, **case}


def prepare(case, seed):
    """Weights, context, hidden states and output buffers: what a serving loop holds before it calls a pass."""
    c = _full(case)
    w = inputs.Workload("case", H=c["H"], E=c["E"], K=c["K"], I=c["I"], n_layers=c["layers"], D=c["D"], P=c["P"],
                        dtype=c["dtype"], seed=seed, residual=c["residual"], weight_format=c["weights"])
    dt = inputs.torch_dtype(c["dtype"])
    layers = [inputs.make_layer(w, l, device=DEV) for l in range(c["layers"])]
    if c["zipf"] > 0:
        bias = -c["zipf"] * torch.log(torch.arange(1, c["E"] + 1, dtype=torch.float32, device=DEV))
        for L in layers:
            L["router_bias"] = bias
    xd = inputs.randn((c["D"], c["H"]), 1.0, seed, "x_decode", 0, c["dtype"], DEV)
    xp = inputs.randn((c["P"], c["H"]), 1.0, seed, "x_prefill", 0, c["dtype"], DEV)
    rows = c["D"] + (min(c["P"], c["chunk"]) if c["chunk"] > 0 else c["P"])
    ctx = binding.Context(c["H"], c["E"], c["K"], c["I"], dt, max_tokens=rows, residual=c["residual"], device=DEV,
                          weight_format=c["weights"], y_perm_f32=c["y_perm_f32"], act_split=c["act_split"])
    return {"case": c, "ctx": ctx, "layers": layers, "packed": ctx.pack_layers(layers), "xd": xd, "xp": xp,
            "yd": torch.empty_like(xd), "yp": torch.empty_like(xp)}


def run(state):
    c, ctx, layers = state["case"], state["ctx"], state["layers"]
    xd = state["xd"] if c["D"] else None
    xp = state["xp"] if c["P"] else None
    if c["call"] == "group":
        ctx.moe_group_forward(layers, xd, xp, c["schedule"], c["chunk"], packed=state["packed"], y_decode=state["yd"],
                              y_prefill=state["yp"])
        return [y for y in (state["yd"], state["yp"]) if y.shape[0]]
    if c["call"] == "stack":
        ctx.moe_stack_forward(layers, xd, xp, chunk=c["chunk"], n_groups=c["groups"], granule=c["granule"],
                              packed=state["packed"], y_decode=state["yd"], y_prefill=state["yp"])
        return [y for y in (state["yd"], state["yp"]) if y.shape[0]]
    x, L = xd, layers[0]
    idx, w = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
    counts, offsets, perm, inv, x_perm = ctx.moe_permute(x, idx)
    y_perm = ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"])
    y = ctx.moe_combine(y_perm, inv, w, residual=x, out=state["yd"])
    return {"idx": idx, "w": w, "counts": counts, "offsets": offsets, "perm": perm, "inv": inv, "y_perm": y_perm, "y": y}


def _passes(c):
    """(batch rows of every layer pass, layer passes that carry them): the iterations of the schedule."""
    D, P, n = c["D"], c["P"], c["layers"]
    if c["call"] == "steps" or P == 0:
        return [(D + P, n)]
    if c["call"] == "group":
        if c["schedule"] == "layered":
            return [(D + P, n)]
        step = c["chunk"]
        return [(D + min(step, P - p), n) for p in range(0, P, step)]
    g = c["groups"] or max(1, min(n, -(-P // c["granule"])))
    # over the g iterations every layer sees the prompt once and the decode rows alone g - 1 times
    return [(D + P, n), (D, n * (g - 1))]


def work(case):
    c = _full(case)
    H, E, K, I = c["H"], c["E"], c["K"], c["I"]
    esz = 4 if c["dtype"] == "f32" else 2
    wsz = 17.0 / 32.0 if c["weights"] == "mxfp4" else esz
    nbytes = flops = 0.0
    for rows, passes in _passes(c):
        active = E * (1.0 - (1.0 - K / E) ** rows)        # experts with a row, under even routing
        nbytes += passes * (active * 3 * H * I * wsz + E * H * esz)
        flops += passes * (rows * K * 6.0 * H * I + 2.0 * rows * E * H)
    nbytes += 2.0 * (c["D"] + c["P"]) * H * esz           # the hidden states in and out, once
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what a plain fp32 computation of the same layers, rounded where the framework rounds, differs by."""
    c = _full(case)
    if c["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    if c["layers"] == 1:
        return {"rel": 2e-3, "max": 0.06}
    # a value rounded the other way between two layers sends a token in a hundred to another expert: few outputs, far off
    return {"rel": 0.004 * c["layers"], "max": 0.9}
