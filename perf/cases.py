"""The workloads whose speed this repository is held to: what each stands for, its inputs, one pass and the work in it.

A case is a dict of plain values.  `op` names the path it takes through the public entry points:

  score      maxsim_forward: a uniform corpus resident on the GPU, with or without the winning token of every query token
  rerank     maxsim_forward_ragged: documents of different lengths packed back to back
  score_i8   the query quantised by maxsim_quantize_rows_i8, then maxsim_forward_i8 against an int8 corpus
  rerank_i8  the same against a packed int8 corpus
  step       a contrastive training step over the C boundary: forward with argmax, cross-entropy gradient, backward
  autograd   the same step as a torch program writes it: the differentiable scores, torch's cross-entropy, torch.autograd.grad
  quantize   maxsim_quantize_rows_i8 over rows of a corpus at index time
"""
import math

import torch
import torch.nn.functional as F

from paper_2605_29517_amd import autograd as A
from paper_2605_29517_amd import binding as M
from paper_2605_29517_amd import workloads as W

TAU = 0.02
_SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def _rerank(name, n_q, docs, op="rerank"):
    return {"name": name, "op": op, "n_q": n_q, "l_q": 32, "docs": docs, "lo": 64, "hi": 300, "d": 128, "dtype": "f16"}


def listed():
    return [
        # One short fp32 query against a thousand short documents, winning tokens wanted (to show the match): the call
        # that a latency-bound program makes.
        {"name": "tiny_argmax", "op": "score", "n_q": 1, "l_q": 32, "docs": 1000, "l_d": 128, "d": 128, "dtype": "f32", "argmax": True},
        # Second stage of retrieval: one query, the thousand candidates of the first stage, texts of 64 to 300 tokens.
        _rerank("rerank_1k", 1, 1000),
        # The same texts, a hundred thousand of them: one query at a time (served as it comes), a small batch, a full one.
        _rerank("rerank_100k_1q", 1, 100_000),
        _rerank("rerank_100k_8q", 8, 100_000),
        _rerank("rerank_100k_64q", 64, 100_000),
        # Pages as queries against pages (1024 patch embeddings each): the matrix-bound end of scoring.
        {"name": "pages_bf16", "op": "score", "n_q": 4, "l_q": 1024, "docs": 10_000, "l_d": 1024, "d": 128, "dtype": "bf16", "argmax": False},
        # Pages at the width of a model's hidden state instead of a projected one.
        {"name": "pages_wide", "op": "score", "n_q": 4, "l_q": 1024, "docs": 500, "l_d": 1024, "d": 1024, "dtype": "bf16", "argmax": False},
        # In-batch negatives, 256 short queries x 256 long documents: a training step over the C boundary.
        {"name": "step_text", "op": "step", "n": 256, "l_q": 32, "l_d": 1024, "ragged": False, "d": 128, "dtype": "f16"},
        # The same with pages on both sides, through torch.autograd.
        {"name": "autograd_pages", "op": "autograd", "n": 32, "l_q": 1024, "l_d": 1024, "d": 128, "dtype": "bf16"},
        # A page against a corpus of pages stored as int8.
        {"name": "pages_i8", "op": "score_i8", "n_q": 1, "l_q": 1024, "docs": 40_000, "l_d": 1024, "d": 128},
        # Reranking over texts stored as int8.
        _rerank("rerank_100k_i8", 1, 100_000, "rerank_i8"),
        # Index time: a piece of a corpus is quantised.
        {"name": "quantize_pages", "op": "quantize", "rows": 2_048_000, "d": 128, "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tokens(case):
    """Document tokens of a case (their expectation where lengths are drawn)."""
    if "hi" in case:
        return case["docs"] * (case["lo"] + case["hi"]) / 2
    return case.get("docs", case.get("n")) * case["l_d"]


def _cost(case):
    """Rough seconds of one pass, to keep drawn cases below the largest listed one."""
    w = work(case)
    rate = 2.2e15 if case["op"].endswith("i8") else (8e13 if case.get("dtype") == "f32" else (1.0e15 if case["d"] > 128 else 1.3e15))
    return w["bytes"] / 5e12 + w["flops"] / rate


def _one(rng):
    kind = rng.choice(["tiny", "rerank", "rerank", "pages", "wide", "step", "autograd", "pages_i8", "rerank_i8", "quantize"])
    two = rng.choice(["f16", "bf16"])
    if kind == "tiny":
        return {"op": "score", "n_q": 1, "l_q": rng.randint(8, 64), "docs": _log(rng, 100, 5000), "l_d": _log(rng, 16, 300), "d": 128, "dtype": "f32",
                "argmax": rng.random() < 0.7}
    if kind == "rerank":
        return {"op": "rerank", "n_q": _log(rng, 1, 64), "l_q": rng.choice([32, 32, rng.randint(8, 64)]), "docs": _log(rng, 1000, 100_000),
                "lo": rng.randint(8, 120), "hi": rng.randint(180, 512), "d": 128, "dtype": two}
    if kind == "pages":
        return {"op": "score", "n_q": rng.randint(1, 8), "l_q": _log(rng, 128, 1024), "docs": _log(rng, 500, 10_000), "l_d": rng.randint(256, 1030), "d": 128,
                "dtype": two, "argmax": False}
    if kind == "wide":
        return {"op": "score", "n_q": rng.randint(1, 4), "l_q": _log(rng, 32, 1024), "docs": _log(rng, 64, 4000), "l_d": rng.randint(128, 1030),
                "d": rng.choice([256, 512, 768, 1024, 2048, 32 * rng.randint(5, 64)]), "dtype": two, "argmax": False}
    if kind == "step":
        return {"op": "step", "n": _log(rng, 16, 256), "l_q": rng.choice([32, rng.randint(8, 64)]), "l_d": rng.randint(64, 1024), "ragged": rng.random() < 0.4,
                "d": 128, "dtype": two}
    if kind == "autograd":
        return {"op": "autograd", "n": _log(rng, 8, 64), "l_q": rng.randint(256, 1030), "l_d": rng.randint(256, 1030), "d": 128, "dtype": two}
    if kind == "pages_i8":
        return {"op": "score_i8", "n_q": rng.randint(1, 4), "l_q": _log(rng, 128, 1024), "docs": _log(rng, 500, 40_000), "l_d": rng.randint(256, 1030), "d": 128}
    if kind == "rerank_i8":
        return {"op": "rerank_i8", "n_q": rng.randint(1, 8), "l_q": rng.choice([32, rng.randint(8, 64)]), "docs": _log(rng, 1000, 100_000),
                "lo": rng.randint(8, 120), "hi": rng.randint(180, 512), "d": 128, "dtype": "f16"}
    return {"op": "quantize", "rows": _log(rng, 1000, 2_048_000), "d": 128, "dtype": rng.choice(["f32", "f16", "bf16"])}


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        case = _one(rng)
        if _cost(case) <= most:
            return case


def _quantized(tokens, d, seed, dev):
    """int8 codes and scales of unit-norm fp32 rows, a piece at a time."""
    codes = torch.empty(tokens, d, dtype=torch.int8, device=dev)
    scale = torch.empty(tokens, dtype=torch.float32, device=dev)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    for t in range(0, tokens, 1 << 22):
        n = min(1 << 22, tokens - t)
        M.maxsim_quantize_rows_i8(W.unit_rows((n, d), "f32", 0, dev, generator=g), codes[t:t + n], scale[t:t + n])
    return codes, scale


def prepare(case, seed):
    dev = "cuda"
    op = case["op"]
    d = case["d"]
    s = {"case": case}
    if op == "quantize":
        s["X"] = W.unit_rows((case["rows"], d), case["dtype"], seed, dev)
    elif op in ("step", "autograd"):
        n, l_d = case["n"], case["l_d"]
        if op == "autograd":
            Q = W.colpali_pages(n, case["l_q"], d, case["dtype"], 2 * seed, dev)
            D = W.colpali_pages(n, l_d, d, case["dtype"], 2 * seed + 1, dev)
            s["Q"], s["D"] = Q.requires_grad_(), D.requires_grad_()
            s["label"] = torch.arange(n, device=dev)
        elif case["ragged"]:
            # the order of the lengths is the seed's; their sum is the case's, so that gradients keep their shape
            lengths, s["offsets"] = W.ragged_lengths(n, max(1, l_d // 4), l_d, 9, dev)
            g = torch.Generator(device=dev)
            g.manual_seed(seed)
            s["offsets"][1:] = torch.cumsum(lengths[torch.randperm(n, generator=g, device=dev)], 0)
            s["Q"] = W.unit_rows((n, case["l_q"], d), case["dtype"], 2 * seed, dev)
            s["D"] = W.unit_rows((int(s["offsets"][-1]), d), case["dtype"], 2 * seed + 1, dev)
        else:
            s["Q"], s["D"] = W.contrastive_batch(n, case["l_q"], l_d, d, case["dtype"], seed, dev)
    elif op == "rerank":
        s["Q"], s["D"], s["offsets"], _ = W.colbert_rerank(case["n_q"], case["l_q"], case["docs"], case["lo"], case["hi"], d, case["dtype"], seed, dev)
    elif op == "score":
        if case["dtype"] == "f32" or case["l_q"] < 128:
            s["Q"] = W.unit_rows((case["n_q"], case["l_q"], d), case["dtype"], 2 * seed, dev)
            s["D"] = W.unit_rows((case["docs"], case["l_d"], d), case["dtype"], 2 * seed + 1, dev)
        else:
            s["Q"] = W.colpali_pages(case["n_q"], case["l_q"], d, case["dtype"], 2 * seed, dev)
            s["D"] = W.colpali_pages(case["docs"], case["l_d"], d, case["dtype"], 2 * seed + 1, dev)
    else:
        s["Q"] = W.unit_rows((case["n_q"], case["l_q"], d), "f16", 2 * seed, dev)
        if op == "rerank_i8":
            _, s["offsets"] = W.ragged_lengths(case["docs"], case["lo"], case["hi"], seed, dev)
            s["D8"], s["scale"] = _quantized(int(s["offsets"][-1]), d, 2 * seed + 1, dev)
        else:
            codes, scale = _quantized(case["docs"] * case["l_d"], d, 2 * seed + 1, dev)
            s["D8"], s["scale"] = codes.view(case["docs"], case["l_d"], d), scale.view(case["docs"], case["l_d"])
    return s


def run(s):
    op = s["case"]["op"]
    if op == "score":
        return M.maxsim_forward(s["Q"], s["D"], want_argmax=s["case"]["argmax"])
    if op == "rerank":
        return M.maxsim_forward_ragged(s["Q"], s["D"], s["offsets"])
    if op == "score_i8":
        q8, qs = M.maxsim_quantize_rows_i8(s["Q"])
        return M.maxsim_forward_i8(q8, qs, s["D8"], s["scale"])
    if op == "rerank_i8":
        q8, qs = M.maxsim_quantize_rows_i8(s["Q"])
        return M.maxsim_forward_i8_ragged(q8, qs, s["D8"], s["scale"], s["offsets"])
    if op == "quantize":
        return M.maxsim_quantize_rows_i8(s["X"])
    if op == "autograd":
        scores = A.maxsim(s["Q"], s["D"])
        loss = F.cross_entropy(scores / TAU, s["label"])
        dQ, dD = torch.autograd.grad(loss, (s["Q"], s["D"]))
        return loss.detach(), scores.detach(), dQ, dD
    if s["case"]["ragged"]:
        scores, argmax = M.maxsim_forward_ragged(s["Q"], s["D"], s["offsets"], want_argmax=True)
        g, loss = M.maxsim_ce_grad(scores, TAU)
        dQ, dD = M.maxsim_backward_ragged(s["Q"], s["D"], s["offsets"], argmax, g)
    else:
        scores, argmax = M.maxsim_forward(s["Q"], s["D"], want_argmax=True)
        g, loss = M.maxsim_ce_grad(scores, TAU)
        dQ, dD = M.maxsim_backward(s["Q"], s["D"], argmax, g)
    return loss, scores, argmax, dQ, dD


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: two for every multiply-add of the similarities, and of the
    gradients' sums."""
    op, d = case["op"], case["d"]
    if op == "quantize":
        return {"bytes": case["rows"] * (d * (_SIZE[case["dtype"]] + 1) + 4), "flops": 0}
    n_q = case.get("n_q", case.get("n"))
    docs = case.get("docs", case.get("n"))
    q_rows = n_q * case["l_q"]
    t = _tokens(case) * (0.625 if case.get("ragged") else 1)
    flops = 2.0 * q_rows * t * d
    offsets = 4 * (docs + 1) if "hi" in case or case.get("ragged") else 0
    if op.endswith("i8"):
        return {"bytes": int(t * (d + 4) + q_rows * d * 2 + 4 * n_q * docs + offsets), "flops": flops}
    size = _SIZE[case["dtype"]]
    rows = q_rows + t
    out = 4 * n_q * docs
    if op in ("score", "rerank"):
        return {"bytes": int(rows * d * size + out + offsets + (out * case["l_q"] if case.get("argmax") else 0)), "flops": flops}
    grads = rows * d * (size if op == "autograd" else 4)
    argmax = out * case["l_q"] if op == "step" else 0  # the autograd step returns no argmax: it need not reach memory
    return {"bytes": int(rows * d * size + out + offsets + grads + argmax), "flops": flops + 4.0 * q_rows * docs * d}


def tolerance(case):
    """Four times what the outputs differ by from the same pass in 64 bits (twelve seeds of each kind).  The packed fold of the winning
    token takes similarities within 2^-19 of each other as tied, so a few of a million winners may be others; the gradient row of such
    a query token then moves to another document row, which is what bounds the training steps (without one: 1e-5 in the 2-norm for
    fp32 gradients, 1.7e-3 after bf16 rounding, 2.1e-4 after fp16 rounding; with one: up to 1.1e-2, and single values by more than
    their root mean square)."""
    op = case["op"]
    if op.endswith("i8") or op == "quantize":
        return "exact"
    if op in ("step", "autograd"):
        return {"rel": 1.2e-2, "max": 0.99, "differ": 2.5e-5}
    return {"rel": 4e-7, "max": 1e-6, "differ": 1e-5}
