"""Performance cases of the jagged operators: what a recommendation model's program asks of this package.

A case is a plain dict.  `op` says which public entry points it goes through:

    attention  self attention.  train: `autograd.jagged_flash_attention`, forward and backward; otherwise
               `binding.jfa_forward`, as a serving program calls it (out and lse)
    cross      cross attention of a sample's target items to its feature rows, in the same two ways
    features   the feature operators: a softmax along each sample's rows and a product with a matrix per sample,
               and the backward of both
    pad        jagged -> padded dense and back, around a dense operator

The lengths of a case follow one of the package's length recipes (`synthetic.lengths_for`) with the case's own
`lengths_seed`, so that the work of a case is a function of the case alone; `prepare`'s seed deals those lengths to the
samples in another order and draws every value.  `max_len` is the bound a program passes: the longest history that its
model admits, not the longest of the batch at hand.
"""
import math

import numpy as np
import torch

from paper_2409_15373_amd import binding
from paper_2409_15373_amd.autograd import jagged_flash_attention, jagged_flash_cross_attention
from paper_2409_15373_amd.synthetic import lengths_for, offsets_from_lengths


def listed():
    return [
        # The smallest call there is: four samples of at most 64 rows in fp32.  Launches and latency are all of it.
        dict(name="tiny_f32_forward", op="attention", train=False, causal=False, dtype="f32", B=4, H=1, D=32, max_len=64,
             recipe="uniform", sigma=1.0, lengths_seed=0),
        # Training step on short histories (mean 64 rows): a small model's batch, still bound by latency.
        dict(name="geom_d64_train", op="attention", train=True, causal=False, dtype="bf16", B=256, H=2, D=64, max_len=256,
             recipe="trunc_geom", sigma=1.0, lengths_seed=1),
        # Serving on heavy-tailed histories: many short samples and a pile at the longest admitted length.
        dict(name="zipf_d128_forward", op="attention", train=False, causal=False, dtype="bf16", B=1024, H=4, D=128, max_len=1024,
             recipe="zipf", sigma=0.5, lengths_seed=2),
        # The benchmark's step: a tenth of the samples is 2048 to 4096 long, the rest short.  The largest case.
        dict(name="bimodal_d128_train", op="attention", train=True, causal=False, dtype="bf16", B=512, H=8, D=128, max_len=4096,
             recipe="bimodal", sigma=1.0, lengths_seed=3),
        # Training step on evenly spread medium lengths.
        dict(name="uniform_d128_train", op="attention", train=True, causal=False, dtype="bf16", B=1024, H=4, D=128, max_len=1024,
             recipe="uniform", sigma=1.0, lengths_seed=4),
        # The same rows in heads of 64: the usual head size of recommendation models.
        dict(name="uniform_d64_train", op="attention", train=True, causal=False, dtype="bf16", B=1024, H=8, D=64, max_len=1024,
             recipe="uniform", sigma=1.0, lengths_seed=4),
        # A sequential model's training step (row i sees rows 0 .. i) on the bimodal lengths.
        dict(name="bimodal_d128_causal_train", op="attention", train=True, causal=True, dtype="bf16", B=512, H=8, D=128, max_len=4096,
             recipe="bimodal", sigma=1.0, lengths_seed=3),
        # Full-precision training of a small model, and gradient checks.
        dict(name="uniform_f32_d64_train", op="attention", train=True, causal=False, dtype="f32", B=256, H=2, D=64, max_len=512,
             recipe="uniform", sigma=1.0, lengths_seed=5),
        # Target attention, training: at most 32 target items per sample against its whole history.
        dict(name="few_targets_d128_train", op="cross", train=True, dtype="bf16", B=512, H=8, D=128, max_len=4096, recipe="bimodal",
             max_len_q=32, recipe_q="uniform", sigma=1.0, lengths_seed=3),
        # Ranking of some hundred candidates per sample against its history, serving, narrow heads.
        dict(name="targets_d32_forward", op="cross", train=False, dtype="bf16", B=512, H=8, D=32, max_len=1024, recipe="uniform",
             max_len_q=256, recipe_q="uniform", sigma=1.0, lengths_seed=6),
        # The feature operators, forward and backward, on a large batch of feature lists.
        dict(name="features_d64_train", op="features", dtype="bf16", B=16384, D=64, T=64, max_len=512, recipe="uniform",
             lengths_seed=7),
        # Padding for a dense operator and stripping the padding again, one values tensor.
        dict(name="pad_and_strip", op="pad", dtype="bf16", B=1024, H=4, D=128, max_len=1024, recipe="uniform", lengths_seed=4),
    ]


# Cost of a pass relative to bf16 at head size 128, per flop: smaller heads have more softmax work per flop, fp32 runs
# on another unit.  Only used to keep drawn cases below the largest listed one.
_COST = {("bf16", 128): 1.0, ("bf16", 64): 1.6, ("bf16", 32): 3.0, ("f32", 128): 60.0, ("f32", 64): 60.0, ("f32", 32): 80.0}


def _cost(case):
    w = work(case)
    flops = w["flops"] * _COST[case["dtype"], case["D"]] if case["op"] in ("attention", "cross") else 0.0
    return max(flops / 8e14, w["bytes"] / 2e12)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = 0.8 * _cost(next(c for c in listed() if c["name"] == "bimodal_d128_train"))
    while True:
        op = rng.choices(["attention", "cross", "features", "pad"], weights=[6, 2, 1, 1])[0]
        case = dict(op=op, dtype="bf16", B=_log_int(rng, 4, 4096), max_len=_log_int(rng, 32, 4096),
                    recipe=rng.choice(["uniform", "trunc_geom", "zipf", "bimodal"]), lengths_seed=rng.randrange(1 << 30))
        if op == "features":
            case.update(B=_log_int(rng, 64, 20000), max_len=_log_int(rng, 32, 1024), D=rng.choice([32, 64, 128]),
                        T=rng.choice([32, 64, 128]))
        else:
            case.update(H=rng.randint(1, 8), D=rng.choice([32, 64, 64, 128, 128]))
        if op in ("attention", "cross"):
            case.update(train=rng.random() < 0.6, sigma=rng.choice([0.5, 1.0]))
            if rng.random() < 0.15:
                case["dtype"] = "f32"
        if op == "attention":
            case["causal"] = rng.random() < 0.35
        if op == "cross":
            case.update(max_len_q=_log_int(rng, 8, 1024), recipe_q="uniform")
        if op == "pad" and rng.random() < 0.3:
            case["dtype"] = "f32"
        if _cost(case) <= limit and _bytes_held(case) <= 24e9:
            return case


def _bytes_held(case):
    if case["op"] != "pad":
        return 4 * work(case)["bytes"]
    return 3.0 * case["B"] * case["max_len"] * case["H"] * case["D"] * (4 if case["dtype"] == "f32" else 2)


def _lengths(case):
    rng = np.random.Generator(np.random.PCG64(case["lengths_seed"]))
    L = lengths_for(case["recipe"], case["B"], case["max_len"], rng)
    Lq = lengths_for(case["recipe_q"], case["B"], case["max_len_q"], rng) if case["op"] == "cross" else L
    return Lq, L


def work(case):
    Lq, L = (x.astype(np.float64) for x in _lengths(case))
    n, nq = L.sum(), Lq.sum()
    size = 4 if case["dtype"] == "f32" else 2
    if case["op"] == "features":
        D, T, B = case["D"], case["T"], case["B"]
        # in: x, dout, w and its transpose; out: softmax(x), its product with w, dw, dx
        return {"bytes": size * (3 * n * D + 2 * n * T + 3 * B * D * T), "flops": 6 * n * D * T}
    row = case["H"] * case["D"] * size
    if case["op"] == "pad":
        return {"bytes": row * (3 * n + float(case["B"]) * case["max_len"]), "flops": 0.0}
    pairs = (L * (L + 1) / 2).sum() if case.get("causal") else (Lq * L).sum()
    f = case["H"] * case["D"] * pairs
    if case["train"]:   # in: q, k, v, dout; out: out, dq, dk, dv
        return {"bytes": row * 4 * (n + nq), "flops": 14 * f}
    return {"bytes": row * 2 * (n + nq) + 4 * case["H"] * nq, "flops": 4 * f}


def prepare(case, seed):
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    deal = np.random.Generator(np.random.PCG64([seed, case["lengths_seed"]])).permutation(case["B"])
    Lq, L = (x[deal] for x in _lengths(case))
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, sigma=1.0):
        x = torch.randn(*shape, device="cuda", generator=gen)
        return (x.mul_(sigma) if sigma != 1.0 else x).to(dtype)

    s = dict(case, offsets=torch.from_numpy(offsets_from_lengths(L)).cuda())
    n, nq = int(L.sum()), int(Lq.sum())
    if case["op"] == "features":
        s.update(x=normal(n, case["D"]), w=normal(case["B"], case["D"], case["T"]), dout=normal(n, case["T"]))
        s["w_t"] = s["w"].transpose(1, 2).contiguous()   # the operand of the product's gradient, laid out once
        return s
    H, D = case["H"], case["D"]
    if case["op"] == "pad":
        s["values"] = normal(n, H, D)
        return s
    for name, rows in (("q", nq), ("k", n), ("v", n)):
        s[name] = normal(rows, H, D, sigma=case["sigma"]).requires_grad_(case["train"])
    if case["train"]:
        s["dout"] = normal(nq, H, D)
    if case["op"] == "cross":
        s["offsets_q"] = torch.from_numpy(offsets_from_lengths(Lq)).cuda()
    return s


def run(s):
    if s["op"] == "features":
        probs = binding.jfa_jagged_softmax(s["x"], s["offsets"], s["max_len"])
        out = binding.jfa_jagged_dense_bmm(probs, s["w"], s["offsets"], s["max_len"])
        dw = binding.jfa_jagged_jagged_bmm(probs, s["dout"], s["offsets"], s["max_len"])
        dprobs = binding.jfa_jagged_dense_bmm(s["dout"], s["w_t"], s["offsets"], s["max_len"])
        dx = binding.jfa_jagged_softmax_backward(probs, dprobs, s["offsets"], s["max_len"])
        return probs, out, dw, dx
    if s["op"] == "pad":
        dense = binding.jfa_jagged_to_dense(s["values"], s["offsets"], s["max_len"])
        return dense, binding.jfa_dense_to_jagged(dense, s["offsets"], torch.empty_like(s["values"]))
    q, k, v = s["q"], s["k"], s["v"]
    if s["op"] == "cross":
        lens = (s["offsets_q"], s["offsets"], s["max_len_q"], s["max_len"])
        if not s["train"]:
            return binding.jfa_forward_cross(q, k, v, *lens)
        out = jagged_flash_cross_attention(q, k, v, *lens)
    else:
        if not s["train"]:
            return binding.jfa_forward(q, k, v, s["offsets"], s["max_len"], causal=s["causal"])
        out = jagged_flash_attention(q, k, v, s["offsets"], s["max_len"], causal=s["causal"])
    return (out.detach(),) + torch.autograd.grad(out, (q, k, v), s["dout"])


def tolerance(case):
    if case["op"] == "pad":
        return "exact"
    # Four times the distance from the same operation in 64 bits, measured on 48 samples of each listed case and on
    # drawn ones: up to 3.0e-3 in bf16 (the gradients of k), up to 5.5e-7 in fp32.
    return {"rel": 2.2e-6 if case["dtype"] == "f32" else 1.2e-2}
