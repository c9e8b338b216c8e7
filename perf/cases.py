"""The work that programs have this library do, as cases that can be prepared, run and checked.

A case is one of two kinds:

  layer      one pass over a sharded fully-connected layer: forward, backward w.r.t. the input and
             backward w.r.t. the weight (one, two or all three of them, `ops`), each in its natural
             mode (NN, NT, TN) or, for `entry` "tuned", in the mode a tuner has remembered;
  transpose  re-storage of one operand for another mode.

`entry` of a layer: "ops" (the three entry points with a registered scratch area, what a training
loop calls), "static" (the entry point for callers that cannot allocate) or "tuned" (the dispatch to
the remembered mode with a transposed copy of the weight that the caller holds).
"""
import math

import torch

from paper_2502_08145_amd import binding as B

ALL = "fwd,bwd_data,bwd_weight"


def _layer(tokens, d_in, d_out, ops=ALL, entry="ops", mode=""):
    return {"kind": "layer", "tokens": tokens, "d_in": d_in, "d_out": d_out, "ops": ops, "entry": entry, "mode": mode}


def _transpose(rows, cols):
    return {"kind": "transpose", "rows": rows, "cols": cols}


def _named(name, case):
    return {"name": name, **case}


def listed():
    return [
        # the smallest training configuration: 1024 tokens, hidden 512, first layer of the MLP
        _named("tiny_mlp_fc1", _layer(1024, 512, 2048)),
        # smallest shard of the model table (hidden 5120 split 8 x 8): calls of a few GFLOP
        _named("shard_640", _layer(2048, 640, 640)),
        # an unsharded layer of the benchmark model: attention output, 128 large tiles
        _named("attn_out_4096", _layer(2048, 4096, 4096)),
        # and its first MLP layer, the bulk of a training step (the largest case)
        _named("mlp_fc1_16384", _layer(2048, 4096, 16384)),
        # a shard whose reduction is long and whose output is small, called from code that may not allocate
        _named("skinny_fc2_static", _layer(2048, 8192, 2048, entry="static")),
        # the forward and data products of a step whose weight is held transposed for the tuned mode
        _named("tuned_held_weight", _layer(1024, 3072, 3072, ops="fwd,bwd_data", entry="tuned", mode="other")),
        # one token more than whole tiles: a packed batch that is not padded
        _named("tokens_2049", _layer(2049, 2048, 8192)),
        # tokens and widths that are multiples of 8 and of nothing larger
        _named("ragged_by_8", _layer(1064, 1608, 4168)),
        # sizes without any alignment: rows that start at odd addresses
        _named("odd_everything", _layer(391, 777, 1003)),
        # the last, short batch of an epoch, or evaluation on a handful of tokens: weight-bound
        _named("few_tokens", _layer(24, 2048, 8192)),
        # re-storing a weight of the benchmark model for another mode, once per optimiser step
        _named("restore_weight", _transpose(4096, 12288)),
        # and an activation of a ragged batch
        _named("restore_ragged", _transpose(2049, 4100)),
    ]


_MAX_FLOPS = 6.0 * 2048 * 4096 * 16384


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    """Whole tiles (training shards), multiples of 8, sizes without alignment, few tokens, re-storage."""
    while True:
        family = rng.choice(["whole", "whole", "whole", "by8", "by8", "odd", "few", "transpose"])
        if family == "transpose":
            step = rng.choice([1, 8, 64])
            rows, cols = _log_int(rng, 64, 16384, step), _log_int(rng, 64, 16384, step)
            if rows * cols <= 1 << 27:
                return _transpose(rows, cols)
            continue
        if family == "whole":
            t, i, o = _log_int(rng, 256, 4096, 128), _log_int(rng, 256, 16384, 128), _log_int(rng, 256, 16384, 128)
        elif family == "by8":
            t, i, o = _log_int(rng, 128, 4096), _log_int(rng, 256, 8192, 8), _log_int(rng, 256, 8192, 8)
        elif family == "odd":
            t, i, o = _log_int(rng, 64, 2048), _log_int(rng, 64, 4096), _log_int(rng, 64, 4096)
        else:
            t, i, o = _log_int(rng, 1, 96), _log_int(rng, 512, 16384, 8), _log_int(rng, 512, 16384, 8)
        if 6.0 * t * i * o > _MAX_FLOPS:
            continue
        entry = rng.choice(["ops", "ops", "ops", "tuned"])
        if entry == "tuned":
            return _layer(t, i, o, ops="fwd,bwd_data", entry="tuned", mode="other")
        return _layer(t, i, o)


def _normal(gen, shape, sigma):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * sigma).to(torch.bfloat16)


_scratch_registered = False


def _register_scratch_once():
    # a program registers the split-K scratch area at start-up and keeps it
    global _scratch_registered
    if not _scratch_registered:
        B.axonn_linear_init()
        B.register_workspace()
        _scratch_registered = True


def _inputs(case, seed):
    """Activations and gradients N(0, 1), weights N(0, 0.02^2), as the layers of a GPT meet them."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "transpose":
        return {"src": _normal(gen, (case["rows"], case["cols"]), 0.02)}
    t, i, o = case["tokens"], case["d_in"], case["d_out"]
    return {"X": _normal(gen, (t, i), 1.0), "W": _normal(gen, (i, o), 0.02), "dY": _normal(gen, (t, o), 1.0)}


def prepare(case, seed):
    _register_scratch_once()
    state = {"case": case, **_inputs(case, seed)}

    def out(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda")

    if case["kind"] == "transpose":
        state["dst"] = out(case["cols"], case["rows"])
        return state
    t, i, o = case["tokens"], case["d_in"], case["d_out"]
    state["out"] = {"fwd": out(t, o), "bwd_data": out(t, i), "bwd_weight": out(i, o)}
    if case["entry"] == "tuned":
        # forward in NT and data gradient in NN, both on the weight stored the other way ([out, in]),
        # which the program re-stores once per optimiser step and keeps
        B.axonn_linear_tuned_set("fwd", t, o, i, "NT")
        B.axonn_linear_tuned_set("bwd_data", t, i, o, "NN")
        state["W_t"] = out(o, i)
        B.axonn_transpose_bf16(i, o, state["W"], state["W_t"])
    return state


_OPERANDS = {"fwd": ("X", "W"), "bwd_data": ("dY", "W"), "bwd_weight": ("X", "dY")}
_NATURAL = {"fwd": "NN", "bwd_data": "NT", "bwd_weight": "TN"}


def _sizes(case, op):
    t, i, o = case["tokens"], case["d_in"], case["d_out"]
    return {"fwd": (t, o, i), "bwd_data": (t, i, o), "bwd_weight": (i, o, t)}[op]


def run(state):
    case = state["case"]
    if case["kind"] == "transpose":
        B.axonn_transpose_bf16(case["rows"], case["cols"], state["src"], state["dst"])
        return state["dst"]
    results = []
    for op in case["ops"].split(","):
        m, n, k = _sizes(case, op)
        first, second = (state[x] for x in _OPERANDS[op])
        c = state["out"][op]
        if case["entry"] == "ops":
            B.OPS[op](m, n, k, _NATURAL[op], first, second, c)
        elif case["entry"] == "static":
            B.axonn_linear_gemm_static(m, n, k, _NATURAL[op], first, second, c)
        else:
            B.axonn_linear_tuned_call(op, m, n, k, first, second, c, state["W_t"])
        results.append(c)
    return results


def work(case):
    if case["kind"] == "transpose":
        return {"bytes": 4.0 * case["rows"] * case["cols"], "flops": 0.0}
    nbytes = flops = 0.0
    for op in case["ops"].split(","):
        m, n, k = _sizes(case, op)
        nbytes += 2.0 * (m * k + k * n + m * n)
        flops += 2.0 * m * n * k
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Results are rounded once to bf16: against 64 bits the relative error is 1.7e-3 (2-norm), at most
    # half a unit in the last place of a value (3.9e-3 of it) plus what 32-bit sums leave; two correct
    # implementations differ by a whole unit where the sums fall on either side of a rounding boundary.
    if case["kind"] == "transpose":
        return "exact"
    return {"rel": 6.6e-3, "max": 1.6e-2}


def exact(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "transpose":
        return x["src"].to(torch.float64).t().contiguous()
    results = []
    for op in case["ops"].split(","):
        first, second = (x[name].to(torch.float64) for name in _OPERANDS[op])
        if op == "bwd_data":
            second = second.t().contiguous()
        elif op == "bwd_weight":
            first = first.t().contiguous()
        results.append(first @ second)
    return results
