"""Performance cases: the calls that a user of this library makes, at the sizes they come in.

The library runs one layer of an LLM at a time: the two-layer MLP
``Y = act(X @ W1) @ W2`` through a plan (``binding.Plan``), the same call
without a plan for code that may not allocate (``binding.run_noalloc``), and
chains of GEMMs (``binding.ChainPlan``).  A program holds one plan per batch
shape and layer, runs it with each new activation, and walks through layers,
so consecutive calls have other weights.

Every case is a dict of plain values: ``kind`` ("mlp", "noalloc" or "chain"),
the row count ``M``, the widths (``H`` and ``F``; for a chain ``layers`` equal
widths ``H``), the activation and the mode.
"""
import math

import torch

from paper_2607_07862_amd import binding as B

ACTS = {"identity": B.ACT_IDENTITY, "gelu_tanh": B.ACT_GELU_TANH, "swiglu": B.ACT_SWIGLU}

# The most that one case may cost: the matrix products of 8192 rows through
# two 8192 x 8192 weights, and the weights of one 70B gated MLP.
MOST_FLOPS = 4 * 8192.0**3
MOST_BYTES = 1.42e9


def _mlp(name, M, H, F, act, mode="tile_pipelined", kind="mlp"):
    return {"name": name, "kind": kind, "M": M, "H": H, "F": F, "act": act, "mode": mode}


def _chain(name, M, H, layers, act="gelu_tanh", mode="tile_pipelined"):
    return {"name": name, "kind": "chain", "M": M, "H": H, "layers": layers, "act": act, "mode": mode}


def listed():
    return [
        # the smallest call of the benchmark: launches and latencies
        _mlp("tiny_64x512x2048", 64, 512, 2048, "identity"),
        # one token of one sequence through the gated MLP of an 8B model
        _mlp("token_1x4096x14336_swiglu", 1, 4096, 14336, "swiglu"),
        # a small batch from code that may not allocate (graph capture, a serving loop)
        _mlp("noalloc_24x2048x5632", 24, 2048, 5632, "gelu_tanh", kind="noalloc"),
        # 32 tokens through one of eight tensor-parallel shards of a 70B model
        _mlp("shard_32x8192x3584", 32, 8192, 3584, "gelu_tanh"),
        # a decode batch of 128 sequences, 8B model
        _mlp("decode_128x4096x14336", 128, 4096, 14336, "gelu_tanh"),
        # a decode batch of 256 sequences through the gated MLP of a 70B model
        _mlp("gated_256x8192x28672", 256, 8192, 28672, "swiglu"),
        # a chunk of a prompt through an 8B gated MLP, the two kernels one after the other
        _mlp("chunk_512x4096x14336_swiglu", 512, 4096, 14336, "swiglu", mode="sequential"),
        # a ragged batch through widths that are multiples of 64 only, queue scheduling
        _mlp("ragged_777x2112x5440", 777, 2112, 5440, "gelu_tanh", mode="workqueue"),
        # prefill of 2048 tokens, 8B model, plain and gated
        _mlp("prefill_2048x4096x14336", 2048, 4096, 14336, "gelu_tanh"),
        _mlp("prefill_2048x4096x14336_swiglu", 2048, 4096, 14336, "swiglu"),
        # the method's own shape: 8192 x 8192 weights, no activation, many rows
        _mlp("square_8192x8192x8192", 8192, 8192, 8192, "identity"),
        # four GEMMs in a row with 1024 rows
        _chain("chain_1024x8192_4", 1024, 8192, 4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        mode = rng.choice(["tile_pipelined", "tile_pipelined", "tile_pipelined", "sequential", "workqueue"])
        if rng.random() < 0.2:
            M = _log_int(rng, 1, 4096)
            c = _chain("", M, 128 * _log_int(rng, 8, 64), rng.randint(2, 6), rng.choice(["identity", "gelu_tanh"]),
                       rng.choice(["tile_pipelined", "sequential"]))
        else:
            M = _log_int(rng, 1, 8192)
            H = 64 * _log_int(rng, 8, 128)
            F = 64 * _log_int(rng, 16, 448)
            if rng.random() < 0.5:  # most models' widths are multiples of 256
                H, F = -(-H // 256) * 256, -(-F // 256) * 256
            noalloc = M <= 128 and H <= 4096 and F <= 16384 and rng.random() < 0.25
            c = _mlp("", M, H, F, rng.choice(["identity", "gelu_tanh", "swiglu", "swiglu"]), mode, "noalloc" if noalloc else "mlp")
        del c["name"]
        w = work(c)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return c


def _dims(case):
    return [case["H"]] * (case["layers"] + 1)


def _inputs(case, seed):
    """X ~ N(0, 1) and weights ~ N(0, 1 / fan-in), rounded to bf16 (see ``inputs.py``), made on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(shape, std):
        return torch.randn(shape, generator=gen, dtype=torch.float32, device="cuda").mul_(std).to(torch.bfloat16)

    X = normal((case["M"], case["H"]), 1.0)
    if case["kind"] == "chain":
        d = _dims(case)
        return X, [normal((d[l], d[l + 1]), d[l] ** -0.5) for l in range(case["layers"])]
    H, F = case["H"], case["F"]
    W1 = normal((2, H, F) if case["act"] == "swiglu" else (H, F), H**-0.5)
    return X, [W1, normal((F, H), F**-0.5)]


def prepare(case, seed):
    """Activations and weights on the GPU, an output buffer, and (but for "noalloc") the plan of this shape."""
    X, W = _inputs(case, seed)
    act = ACTS[case["act"]]
    plan = None
    if case["kind"] == "mlp":
        plan = B.Plan(case["M"], case["H"], case["F"], act)
    elif case["kind"] == "chain":
        plan = B.ChainPlan(case["M"], _dims(case), act)
    Y = torch.empty(case["M"], case["H"], dtype=torch.bfloat16, device="cuda")
    return {"kind": case["kind"], "plan": plan, "act": act, "mode": case["mode"], "X": X, "W": W, "Y": Y}


def run(state):
    X, W, Y = state["X"], state["W"], state["Y"]
    if state["kind"] == "chain":
        state["plan"].run(X, W, Y, state["mode"])
    elif state["kind"] == "noalloc":
        B.run_noalloc(X, W[0], W[1], Y, state["act"], state["mode"])
    else:
        state["plan"].run(X, W[0], W[1], Y, state["mode"])
    return Y


def work(case):
    """Every weight read once, X read and Y written once; two operations per multiply-add."""
    M, H = case["M"], case["H"]
    if case["kind"] == "chain":
        weights = case["layers"] * H * H
    else:
        weights = (3 if case["act"] == "swiglu" else 2) * H * case["F"]
    return {"bytes": 2.0 * (weights + 2 * M * H), "flops": 2.0 * M * weights}


def tolerance(case):
    """bf16 results with each intermediate rounded to bf16: against 64 bits each
    rounding adds about 1.7e-3 (measured 2.3e-3 after two of them, 3.4e-3 over a
    chain of four); four times that."""
    if case["kind"] == "chain":
        return {"rel": min(0.03, 0.0067 * math.sqrt(case["layers"]))}
    return {"rel": 0.01}


def _act64(act, t):
    if act == "swiglu":
        return torch.nn.functional.silu(t[0]) * t[1]
    return torch.nn.functional.gelu(t, approximate="tanh") if act == "gelu_tanh" else t


def exact(case, seed):
    """Plain torch in 64 bits, by blocks of rows."""
    X, W = _inputs(case, seed)
    W = [w.double() for w in W]
    out = []
    for rows in X.split(2048):
        t = rows.double()
        for l, w in enumerate(W):
            if l + 1 < len(W):
                t = _act64(case["act"], (t @ w[0], t @ w[1]) if w.dim() == 3 else t @ w)
            else:
                t = t @ w
        out.append(t)
    return torch.cat(out)
