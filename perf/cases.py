"""Performance cases of the document-masked attention library: what a training or evaluation
program asks of it, through the C-ABI entry points of `paper_2605_06374_amd.binding`.

A case names a mode (which calls make one pass), a head layout, and a rule with its own seed for
the document lengths of the packed microbatch (the work follows the lengths, so they belong to
the case; the tensors' values come from the seed given to `prepare`).

Modes
  step            forward that plans, then backward on that plan: one layer of a training step
  layer           forward and backward on a plan made beforehand: the further layers of the same
                  microbatch (a program keeps the plan in the workspace)
  forward         forward that plans: evaluation, prefill, the forward of a recomputed layer
  forward_static  forward without a caller's workspace
  backward        backward alone on a kept plan: a pipeline schedule runs the backward of a
                  microbatch long after its forward
"""
import math

import numpy as np
import torch

from paper_2605_06374_amd import binding
from paper_2605_06374_amd import workloads as W

MODES = ("step", "layer", "forward", "forward_static", "backward")


def _case(name, mode, tokens, lengths, doc_seed, q_heads, kv_heads, head_dim, a=0.0, b=0.0, lo=16, std=1.0,
          no_split=False):
    return {"name": name, "mode": mode, "tokens": tokens, "lengths": lengths, "a": a, "b": b, "lo": lo,
            "doc_seed": doc_seed, "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": head_dim, "std": std,
            "no_split": no_split}


def listed():
    return [
        # the smallest call: a short evaluation pack, forward only, by a caller that cannot allocate
        _case("forward_static_777", "forward_static", 777, "lognormal", 11, 4, 4, 128, a=128.0, b=0.8),
        # the tiny configuration: four documents, two heads of 64
        _case("step_tiny_2k", "step", 2048, "cuts", 1001, 2, 2, 64, a=4, lo=64),
        # one microbatch of the length-skew sweep at its short end: many short documents
        _case("step_short_docs_4k", "step", 4096, "lognormal", 5001, 4, 4, 128, a=64.0, b=0.8),
        # the headline configuration: one tensor-parallel shard of a 7B-style model, 8K tokens
        _case("step_8k", "step", 8192, "lognormal", 1002, 4, 4, 128, a=512.0, b=1.2),
        # a further layer of such a microbatch, at a ragged size
        _case("layer_ragged_7k", "layer", 7001, "lognormal", 23, 4, 4, 128, a=700.0, b=1.0),
        # forward only over a ragged 12K pack, grouped queries
        _case("forward_ragged_12k_gqa", "forward", 12345, "lognormal", 29, 8, 2, 128, a=900.0, b=1.2),
        # backward only, heads of 64, grouped queries (a full small model without tensor parallelism)
        _case("backward_6k_heads64_gqa", "backward", 6144, "lognormal", 31, 16, 4, 64, a=600.0, b=1.0),
        # chains never cut: results that do not depend on what else is in the pack
        _case("step_no_split_10k", "step", 9999, "lognormal", 37, 8, 8, 128, a=800.0, b=0.9, no_split=True),
        # the 70B-style shard: 8 q heads on one kv head, 16K tokens
        _case("step_16k_gqa", "step", 16384, "lognormal", 1004, 8, 1, 128, a=1024.0, b=1.3, lo=32, std=0.5),
        # the microbatches of an iteration handed over as one pack of documents of ordinary length
        _case("step_32k_pack", "step", 32768, "lognormal", 41, 4, 4, 128, a=512.0, b=1.2),
        # the long-tail configuration: documents of up to the whole 32K pack
        _case("step_32k_longtail", "step", 32768, "mixture", 1003, 4, 4, 128, a=300.0, b=1.0),
        # one document of 131072 tokens: long-context training
        _case("step_131k_one_document", "step", 131072, "one", 5, 2, 1, 128),
    ]


def _lengths(case):
    n, rng = case["tokens"], np.random.default_rng(case["doc_seed"])
    kind, lo = case["lengths"], case["lo"]
    if kind == "one":
        return [n]
    if kind == "cuts":
        return W.uniform_cuts(rng, n, int(case["a"]), lo)
    if kind == "equal":
        each = int(case["a"])
        return [each] * (n // each) + ([n % each] if n % each else [])
    if kind == "lognormal":
        return W.pack(rng, n, W.lognormal_draw(case["a"], case["b"]), lo)
    return W.pack(rng, n, W.mixture_draw(0.9, case["a"], case["b"], max(lo, n // 8), n), lo)


def _pairs(case):
    return sum(l * (l + 1) // 2 for l in _lengths(case))


def _params(case):
    flags = binding.FLAG_NO_SPLIT if case["no_split"] else 0
    return binding.make_params(case["tokens"], len(_lengths(case)), case["q_heads"], case["kv_heads"],
                               case["head_dim"], 1.0 / math.sqrt(case["head_dim"]), flags)


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    most = work(listed()[-1])["flops"]
    while True:
        mode = rng.choices(MODES, (9, 3, 3, 1, 4))[0]
        q_heads, kv_heads = rng.choice([(1, 1), (2, 1), (2, 2), (4, 4), (4, 4), (4, 2), (8, 8), (8, 2), (8, 1), (6, 3),
                                        (16, 4), (32, 8)])
        tokens = int(_log_uniform(rng, 256, 4096 if mode == "forward_static" else 40000))
        kind = rng.choices(("lognormal", "mixture", "cuts", "equal", "one"), (8, 3, 2, 1, 1))[0]
        a, b, lo = 0.0, 0.0, 16
        if kind == "lognormal":
            a, b = round(_log_uniform(rng, 32, 2048), 1), round(rng.uniform(0.6, 1.3), 2)
        elif kind == "mixture":
            a, b = round(_log_uniform(rng, 64, 512), 1), 1.0
        elif kind == "cuts":
            a, lo = rng.randint(2, 6), 8
        elif kind == "equal":
            a = rng.choice([96, 128, 250, 512, 1000, 2048])
        case = _case("", mode, tokens, kind, rng.randint(1, 1 << 30), q_heads, kv_heads, rng.choice([64, 128, 128]),
                     a=a, b=b, lo=lo, std=rng.choice([1.0, 1.0, 0.5]), no_split=rng.random() < 0.08)
        del case["name"]
        if work(case)["flops"] > most:
            continue
        if mode == "forward_static":
            layout = binding.varlen_attn_workspace_regions(_params(case))
            if layout.col_partials_offset > binding.STATIC_SCRATCH_BYTES:
                continue
        return case


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    n, hq, hkv, d = case["tokens"], case["q_heads"], case["kv_heads"], case["head_dim"]

    def values(heads):
        return torch.randn((n, heads, d), generator=gen, device=dev).mul_(case["std"]).to(torch.bfloat16)

    s = {"mode": case["mode"], "params": _params(case)}
    s["q"], s["k"], s["v"], s["do"] = values(hq), values(hkv), values(hkv), values(hq)
    s["cu"] = torch.from_numpy(W.lengths_to_cu(_lengths(case)).copy()).to(dev)
    s["o"] = torch.zeros_like(s["q"])
    s["lse"] = torch.zeros((hq, n), dtype=torch.float32, device=dev)
    if case["mode"] != "forward_static":
        s["workspace"] = torch.empty(binding.varlen_attn_workspace_bytes(s["params"]), dtype=torch.uint8, device=dev)
    if case["mode"] in ("step", "layer", "backward"):
        s["dq"], s["dk"], s["dv"] = torch.zeros_like(s["q"]), torch.zeros_like(s["k"]), torch.zeros_like(s["v"])
        p = s["params"]
        s["kept"] = binding.make_params(p.total_tokens, p.num_docs, p.num_q_heads, p.num_kv_heads, p.head_dim,
                                        p.softmax_scale, p.flags | binding.FLAG_REUSE_PLAN)
    if case["mode"] == "layer":
        binding.check(binding.varlen_attn_plan(s["params"], s["cu"], s["workspace"]))
    if case["mode"] == "backward":
        _forward(s, s["params"])
    return s


def _forward(s, params):
    binding.check(binding.varlen_attn_fwd(params, s["q"], s["k"], s["v"], s["cu"], s["o"], s["lse"], s["workspace"]))


def _backward(s, params):
    binding.check(binding.varlen_attn_bwd(params, s["q"], s["k"], s["v"], s["o"], s["lse"], s["do"], s["cu"],
                                          s["dq"], s["dk"], s["dv"], s["workspace"]))


def run(state):
    s = state
    if s["mode"] == "forward_static":
        binding.check(binding.varlen_attn_fwd_static(s["params"], s["q"], s["k"], s["v"], s["cu"], s["o"], s["lse"]))
        return {"o": s["o"], "lse": s["lse"]}
    if s["mode"] == "forward":
        _forward(s, s["params"])
        return {"o": s["o"], "lse": s["lse"]}
    if s["mode"] == "step":
        _forward(s, s["params"])
    elif s["mode"] == "layer":
        _forward(s, s["kept"])
    _backward(s, s["kept"])
    if s["mode"] == "backward":
        return {"dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}
    return {"o": s["o"], "lse": s["lse"], "dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}


def work(case):
    """Bytes: every input read once and every output written once in the pass (O and LSE are results
    of a step, inputs of a backward).  Flops: 2 d per (query, key) pair of the causal document mask
    and contraction, two contractions forward and five backward."""
    n, hq, hkv, d = case["tokens"], case["q_heads"], case["kv_heads"], case["head_dim"]
    q, kv, lse = 2 * d * n * hq, 2 * d * n * hkv, 4 * n * hq
    pair = 2 * d * hq * _pairs(case)
    if case["mode"] in ("forward", "forward_static"):
        return {"bytes": 2 * q + 2 * kv + lse, "flops": 2 * pair}
    if case["mode"] == "backward":
        return {"bytes": 4 * q + 4 * kv + lse, "flops": 5 * pair}
    return {"bytes": 4 * q + 4 * kv + lse, "flops": 7 * pair}


def tolerance(case):
    # P and dS are rounded to bf16 before their contraction, O and the gradients are stored in bf16,
    # the backward reads the O of the forward: the distance to fp64 arithmetic on the same inputs
    # (2-norm over 2-norm) is 1.9e-3 to 2.6e-3 for the bf16 results and 5e-8 for LSE
    return {"rel": 1.0e-2}
