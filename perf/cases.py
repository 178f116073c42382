"""The work that this framework is used for, as cases that can be timed and compared.

A case is a plain dict: an operation of the library, its sizes, element type and options.  `listed()` gives the fixed
ones, `draw(rng)` one more from the ranges they stand for, `prepare` the tensors a program holds before the call,
`run` one call through the public entry points, `work` the bytes and operations the result cannot do without, and
`tolerance` how far two correct implementations at the same precision may differ.

Outputs are allocated once with the inputs, as a program that calls the library in a loop does.
"""
import math

import torch

import paper_2501_08071_amd as P

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # Attention.  A short prompt in a small batch, ragged length, output handed on in half precision: latency counts.
        {"name": "attn_short_ragged_o16", "op": "attn", "B": 2, "H": 4, "S": 333, "D": 128, "dtype": "f16", "causal": True,
         "o16": True, "peaked": False},
        # An encoder layer of moderate length: one round of workgroups.
        {"name": "attn_encoder", "op": "attn", "B": 4, "H": 16, "S": 1024, "D": 64, "dtype": "f16", "causal": False,
         "o16": False, "peaked": False},
        # Prefill of a decoder layer at the usual context: the benchmark's default workload.
        {"name": "attn_prefill_4k", "op": "attn", "B": 2, "H": 32, "S": 4096, "D": 128, "dtype": "bf16", "causal": True,
         "o16": False, "peaked": False},
        # Prefill of a long context: the largest.
        {"name": "attn_prefill_16k", "op": "attn", "B": 1, "H": 32, "S": 16384, "D": 128, "dtype": "bf16", "causal": True,
         "o16": False, "peaked": False},
        # A large batch with sharp attention: the softmax reference keeps moving.
        {"name": "attn_batch_peaked", "op": "attn", "B": 16, "H": 16, "S": 2048, "D": 64, "dtype": "f16", "causal": False,
         "o16": False, "peaked": True},
        # Few heads, small head dimension, long sequence (the paper's own shape): few workgroups, vector work dominates.
        {"name": "attn_few_heads", "op": "attn", "B": 1, "H": 4, "S": 4096, "D": 32, "dtype": "f16", "causal": False,
         "o16": False, "peaked": False},
        # Row softmax at the paper's shape: a small memory-bound launch.
        {"name": "softmax_small", "op": "softmax", "rows": 512, "cols": 4096, "dtype": "f16"},
        # Row softmax over a row length that is not a multiple of anything (class scores, a masked-off column).
        {"name": "softmax_odd_rows", "op": "softmax", "rows": 4096, "cols": 4095, "dtype": "bf16"},
        # RMS norm over head dimensions, sixteen times the paper's rows: streams through HBM.
        {"name": "rmsnorm_stream", "op": "rmsnorm", "rows": 2097152, "cols": 64, "dtype": "f16"},
        # GEMM + LeakyReLU at the paper's shape: a small matrix product with a long K.
        {"name": "gemm_small_long_k", "op": "gemm", "batch": 1, "M": 512, "N": 512, "K": 2048, "dtype": "f16", "slope": 0.01},
        # A batched product with sizes that fit no tile.
        {"name": "gemm_batch_ragged", "op": "gemm", "batch": 2, "M": 777, "N": 1000, "K": 1000, "dtype": "bf16", "slope": 0.01},
        # A large product: bound by the matrix cores.
        {"name": "gemm_large", "op": "gemm", "batch": 1, "M": 4096, "N": 4096, "K": 4096, "dtype": "bf16", "slope": 0.01},
    ]


def _spread(rng, lo, hi):
    """An integer of lo .. hi, even over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    dtype = rng.choice(["f16", "bf16"])
    kind = rng.random()
    if kind < 0.5:
        D = rng.choice([32, 64, 128])
        B, H = _spread(rng, 1, 16), _spread(rng, 1, 32)
        S = _spread(rng, 64, 16384)
        S = min(S, int(math.sqrt(1.5e9 / (B * H))))      # scores
        return {"op": "attn", "B": B, "H": H, "S": S, "D": D, "dtype": dtype, "causal": rng.random() < 0.5,
                "o16": rng.random() < 0.3, "peaked": rng.random() < 0.2}
    if kind < 0.75:
        op = rng.choice(["softmax", "rmsnorm"])
        cols = _spread(rng, 32, 32768)
        if rng.random() < 0.5:
            cols = max(8, cols // 8 * 8)
        rows = max(1, _spread(rng, 1 << 19, 1 << 26) // cols)    # elements
        return {"op": op, "rows": rows, "cols": cols, "dtype": dtype}
    batch = rng.choice([1, 1, 2, 4])
    M, N, K = _spread(rng, 32, 4096), _spread(rng, 32, 4096), _spread(rng, 64, 4096)
    if rng.random() < 0.6:                       # sizes of weight matrices
        N, K = (N + 31) // 32 * 32, (K + 31) // 32 * 32
    else:                                        # ragged ones are small problems
        M = max(1, min(M, int(2.0e9 / (N * K * batch))))
    return {"op": "gemm", "batch": batch, "M": M, "N": N, "K": K, "dtype": dtype, "slope": rng.choice([0.01, 1.0, 0.2])}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = DTYPES[case["dtype"]]

    def normal(shape, mul=1.0):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * mul).to(dt)

    if case["op"] == "attn":
        shape = (case["B"], case["H"], case["S"], case["D"])
        mul = 4.0 if case["peaked"] else 1.0
        q, k = normal(shape, mul), normal(shape, mul)
        if case["peaked"]:
            v = (torch.rand(shape, generator=g, device="cuda", dtype=torch.float32) * 2.0 - 1.0).to(dt)
        else:
            v = normal(shape)
        return {"op": "attn", "q": q, "k": k, "v": v, "causal": case["causal"], "scale": 1.0 / math.sqrt(case["D"]),
                "o16": case["o16"], "o": torch.empty(shape, dtype=dt if case["o16"] else torch.float32, device="cuda"),
                "lse": torch.empty(shape[:3], dtype=torch.float32, device="cuda")}
    if case["op"] == "gemm":
        a = normal((case["batch"], case["M"], case["K"]))
        b = normal((case["batch"], case["K"], case["N"]))
        return {"op": "gemm", "a": a, "b": b, "slope": case["slope"],
                "c": torch.empty((case["batch"], case["M"], case["N"]), dtype=dt, device="cuda")}
    x = normal((case["rows"], case["cols"]), 3.0 if case["op"] == "softmax" else 1.0)
    state = {"op": case["op"], "x": x, "y": torch.empty_like(x)}
    if case["op"] == "rmsnorm":
        state["w"] = normal((case["cols"],))
    return state


def run(state):
    op = state["op"]
    if op == "attn":
        fwd = P.attn_fwd_o16 if state["o16"] else P.attn_fwd
        return fwd(state["q"], state["k"], state["v"], state["causal"], state["scale"], o=state["o"], lse=state["lse"])
    if op == "gemm":
        return P.gemm_leakyrelu_fwd(state["a"], state["b"], state["slope"], c=state["c"])
    if op == "softmax":
        return P.softmax_rows_fwd(state["x"], y=state["y"])
    return P.rmsnorm_fwd(state["x"], state["w"], 1e-6, y=state["y"])


def work(case):
    if case["op"] == "attn":
        rows, S, D = case["B"] * case["H"] * case["S"], case["S"], case["D"]
        scores = rows * (S + 1) / 2 if case["causal"] else rows * S
        return {"bytes": rows * (6 * D + (2 if case["o16"] else 4) * D + 4), "flops": 4.0 * scores * D}
    if case["op"] == "gemm":
        b, M, N, K = case["batch"], case["M"], case["N"], case["K"]
        return {"bytes": 2 * b * (M * K + K * N + M * N), "flops": 2.0 * b * M * N * K}
    n = case["rows"] * case["cols"]
    w = 2 * case["cols"] if case["op"] == "rmsnorm" else 0
    return {"bytes": 4 * n + w, "flops": 4.0 * n}


def tolerance(case):
    # About four times the error measured against the same operation in 64 bits on the same inputs.  Attention: the
    # softmax weights are rounded to the input type before the second product.  The others: one rounding of the result.
    if case["op"] == "attn":
        return {"rel": 9e-3 if case["dtype"] == "bf16" else 1e-3}
    return {"rel": 6.5e-3 if case["dtype"] == "bf16" else 8.5e-4}
