"""The calls of the MoE layer whose speed matters, as cases that a timing or comparison program can run.

A case is a batch of N tokens through one layer (d, h, E experts, top-k) in one of three uses:

  forward  moe_plan + moe_forward: serving, from a handful of tokens to a long ragged prefill batch
  train    moe_plan + moe_forward + moe_backward (+ moe_bias_backward when the experts have biases, + moe_balance_stats
           when the statistics are asked for): one training step's work, gradients included
  move     moe_plan and the four data movements on their own, for callers that put another expert network between them

Options: storage type, skew of the expert load (the gate bias of synth.gate_bias), expert biases, scores over all
experts, load-balance statistics, and weight gradients added up in fp32 over micro-batches.

`listed()` holds the workloads C0 to C4 of synth.WORKLOADS (the layer's benchmark configurations) and, around them, the
uses that they leave out; `draw(rng)` gives further ones of the same ranges.
"""
import math

import torch

from paper_2103_13262_amd import binding as B
from paper_2103_13262_amd.synth import WORKLOADS, Workload, gate_bias

_DEFAULTS = {"use": "train", "dtype": "bf16", "zipf": 0.0, "biases": False, "score_all": False, "balance": False, "accumulate": False}


def _case(name, N, d, h, E, k, **options):
    c = {"name": name, "N": N, "d": d, "h": h, "E": E, "k": k, **_DEFAULTS}
    c.update(options)
    return c


def _workload(name, key):
    w = WORKLOADS[key]
    return _case(name, w.N, w.d, w.h, w.E, w.k, dtype=w.dtype, zipf=w.zipf_s)


def listed():
    return [
        # C0, the tiny fp32 layer: a step is nothing but launches and latency
        _workload("train_tiny_f32", "C0"),
        # a few sequences decoding through the paper-shape layer: every touched expert's weights for a row or two each
        _case("decode_8_tokens", 8, 1024, 4096, 16, 2, use="forward"),
        # a larger decode batch through the layer of many small experts (C3's): most experts see one row or none
        _case("decode_200_small_experts", 200, 512, 1024, 256, 1, use="forward"),
        # an odd-length prefill through the paper-shape layer whose experts have biases, as trained ones do
        _case("prefill_1777_biases", 1777, 1024, 4096, 16, 2, use="forward", biases=True),
        # a long prompt through the large shard of C4 at its own skew: the forward direction at matrix-core rates
        _case("prefill_8192_large", 8192, 2048, 8192, 32, 2, use="forward", zipf=0.8),
        # C1, the paper's own shape
        _workload("train_paper_shape", "C1"),
        # C2, a skewed load over 64 experts: hundreds of rows for some, next to none for others
        _workload("train_skewed_64", "C2"),
        # C3, many small experts, top-1
        _workload("train_256_small_top1", "C3"),
        # C4, the large one-GPU shard: the largest case
        _workload("train_large_shard", "C4"),
        # a micro-batch of odd length in a layer with biases and widths that are no powers of two, its weight gradients
        # added up in fp32
        _case("train_micro_accumulate", 1000, 768, 3072, 8, 2, biases=True, accumulate=True),
        # scores over all experts with the load-balance statistics of the step
        _case("train_scores_all_balance", 2048, 1024, 2048, 64, 2, score_all=True, balance=True),
        # the data movements alone, around somebody else's experts, at C4's tokens
        _case("move_large", 32768, 2048, 8192, 32, 2, use="move"),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` from lo to hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(v / step) * step)))


def draw(rng):
    largest = work(_workload("", "C4"))
    while True:
        kind = rng.choice(("forward", "forward", "train", "train", "train", "train_f32", "move"))
        c = _case("", _log(rng, 1, 32768), _log(rng, 256, 2048, 32), _log(rng, 512, 8192, 32), _log(rng, 2, 256), rng.choice((1, 2, 2, 4)))
        if kind == "train_f32":                       # fp32 is the layer's type for small models and for checking others
            c.update(N=_log(rng, 64, 4096), d=_log(rng, 64, 512, 32), h=_log(rng, 64, 1024, 32), E=_log(rng, 2, 32), dtype="f32")
        elif kind == "train":                         # (a training step has at least a short sequence in it)
            c["N"] = _log(rng, 256, 32768)
        if kind == "move":
            c.update(use="move", N=_log(rng, 64, 32768))
        elif kind == "forward":
            c["use"] = "forward"
        c["k"] = min(c["k"], c["E"])
        c["zipf"] = rng.choice((0.0, 0.0, round(rng.uniform(0.2, 1.2), 2)))
        if c["use"] != "move":
            c["biases"] = rng.random() < 0.25
            c["score_all"] = rng.random() < 0.15
        if c["use"] == "train":
            c["balance"] = c["score_all"] and rng.random() < 0.5
            c["accumulate"] = rng.random() < 0.25
        del c["name"]
        w = work(c)
        # a layer has at most some billions of parameters and fits the card several times over
        if w["bytes"] <= largest["bytes"] and w["flops"] <= largest["flops"] and c["E"] * c["d"] * c["h"] <= 32 * 2048 * 8192:
            return c


class _State:
    pass


def prepare(case, seed):
    """A program's tensors on the GPU: activations N(0,1), weights N(0,0.02) in the storage type, and the layer's buffers."""
    s = _State()
    s.case = case
    N, d, h, E, k = (case[n] for n in ("N", "d", "h", "E", "k"))
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    act = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    dt = B.MOE_BF16 if case["dtype"] == "bf16" else B.MOE_F32

    def normal(shape, std=1.0, dtype=act):
        return torch.empty(shape, dtype=dtype, device=dev).normal_(0.0, std, generator=gen)

    s.desc = B.make_desc(N, d, h, E, k, dt, B.MOE_F32 if case["accumulate"] else dt, int(case["accumulate"]), int(case["score_all"]),
                         int(case["balance"]))
    s.buf = B.MoeLayerBuffers(s.desc, dev)
    s.stream = s.buf.stream()
    s.X, s.Wg = normal((N, d)), normal((d, E), 0.02)
    s.bg = torch.from_numpy(gate_bias(Workload("", N, d, h, E, k, case["dtype"], case["zipf"]))).to(dev)
    s.Y = torch.empty((N, d), dtype=act, device=dev)
    grad = torch.float32 if case["accumulate"] else act
    make = torch.zeros if case["accumulate"] else torch.empty     # (added to: a program clears them once per optimizer step)
    s.b1 = s.b2 = None
    if case["use"] != "move":
        s.W1, s.W2 = normal((E, d, h), 0.02), normal((E, h, d), 0.02)
        if case["biases"]:
            s.b1, s.b2 = normal((E, h), 0.1), normal((E, d), 0.1)
    if case["use"] != "forward":
        s.dY, s.dX = normal((N, d)), torch.empty((N, d), dtype=act, device=dev)
        s.dWg, s.dbg = make((d, E), dtype=grad, device=dev), make(max(E, 4), dtype=torch.float32, device=dev)
    if case["use"] == "train":
        s.dW1, s.dW2 = make((E, d, h), dtype=grad, device=dev), make((E, h, d), dtype=grad, device=dev)
        if case["biases"]:
            s.db1, s.db2 = make((E, h), dtype=torch.float32, device=dev), make((E, d), dtype=torch.float32, device=dev)
        if case["balance"]:
            s.fraction, s.mean_prob = torch.empty(E, dtype=torch.float32, device=dev), torch.empty(E, dtype=torch.float32, device=dev)
            s.loss = torch.empty(1, dtype=torch.float32, device=dev)
    if case["use"] == "move":
        M = N * k
        s.Ys, s.dXs = normal((M, d)), normal((M, d))
        s.Xs, s.dYs = torch.empty((M, d), dtype=act, device=dev), torch.empty((M, d), dtype=act, device=dev)
        s.dl = torch.empty(max(M, 4), dtype=torch.float32, device=dev)
    return s


def run(s):
    """One pass through the layer's public calls; returns its outputs (the state's own buffers)."""
    c, buf, E = s.case, s.buf, s.case["E"]
    ws, nws, st = buf.workspace, buf.ws_bytes, s.stream
    B.moe_plan(s.desc, s.X, s.Wg, s.bg, buf.plan, ws, nws, st)
    out = {"topk_idx": buf.topk_idx, "topk_w": buf.topk_w}
    if c["use"] == "move":
        B.moe_scatter(s.desc, buf.plan, s.X, s.Xs, st)
        B.moe_gather(s.desc, buf.plan, s.Ys, s.Y, st)
        B.moe_gather_backward(s.desc, buf.plan, s.dY, s.Ys, s.dYs, s.dl, st)
        B.moe_scatter_backward(s.desc, buf.plan, s.Wg, s.Xs, s.dXs, s.dl, s.dX, s.dWg, s.dbg, ws, nws, st)
        out.update(Xs=s.Xs, Y=s.Y, dYs=s.dYs, dl=s.dl[:c["N"] * c["k"]], dX=s.dX)
    else:
        B.moe_forward(s.desc, buf.plan, s.X, s.W1, s.W2, s.b1, s.b2, s.Y, ws, nws, st)
        out["Y"] = s.Y
    if c["use"] == "train":
        B.moe_backward(s.desc, buf.plan, s.X, s.Wg, s.W1, s.W2, s.dY, s.dX, s.dWg, s.dbg, s.dW1, s.dW2, ws, nws, st)
        out.update(dX=s.dX, dW1=s.dW1, dW2=s.dW2)
        if c["biases"]:
            B.moe_bias_backward(s.desc, buf.plan, s.db1, s.db2, ws, nws, st)
            out.update(db1=s.db1, db2=s.db2)
        if c["balance"]:
            B.moe_balance_stats(s.desc, buf.plan, s.fraction, s.mean_prob, s.loss, ws, nws, st)
            out.update(fraction=s.fraction, mean_prob=s.mean_prob, loss=s.loss)
    if c["use"] != "forward" and (c["k"] > 1 or c["score_all"] or c["accumulate"]):   # (otherwise the gate's gradient is exactly zero)
        out.update(dWg=s.dWg, dbg=s.dbg[:E])
    return out


def work(case):
    """Bytes and operations that a pass cannot do without: inputs read once, outputs written once, expert and gate products."""
    N, d, h, E, k = (case[n] for n in ("N", "d", "h", "E", "k"))
    b = 2 if case["dtype"] == "bf16" else 4
    g = 4 if case["accumulate"] else b                    # weight gradients
    M = N * k
    nbytes = N * d * b + d * E * b + M * 8                # X, W_g, the routing
    flops = 2.0 * N * d * E
    if case["use"] == "move":
        nbytes += 4 * M * d * b + 3 * N * d * b + 2 * d * E * b + M * 4      # Xs, Ys, dYs, dXs; Y, dY, dX; W_g again, dW_g; dl
        return {"bytes": nbytes, "flops": flops + 6.0 * M * d}
    # experts that at least one token reaches (p: an expert's share of the tokens, after the gate bias of the case)
    p = [(e + 1.0) ** -case["zipf"] for e in range(E)]
    p = [min(1.0, k * v / sum(p)) for v in p]
    touched = sum(1.0 - (1.0 - v) ** N for v in p)
    nbytes += 2 * touched * d * h * b + N * d * b         # W1, W2 of those; Y
    flops += 4.0 * M * d * h
    if case["biases"]:
        nbytes += touched * (d + h) * b
    if case["use"] == "train":
        nbytes += 2 * N * d * b + d * E * g + 2 * E * d * h * g * (2 if case["accumulate"] else 1)   # dY, dX, dW_g, dW1, dW2 (added to: read as well)
        flops += 8.0 * M * d * h + (4.0 * N * d * E if case["score_all"] else 4.0 * M * d)
        if case["biases"]:
            nbytes += E * (d + h) * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what the path differs by from itself with its sums in another order (the model and hidden dimensions and the
    tokens permuted), over the listed cases and some two hundred drawn ones.  fp32: 1.5e-6 of a tensor's norm, 1e-5 for a single
    value; bf16: 1.1e-3 (the gate's gradients; 6e-4 for the others) and 3.2e-2.  The gate-bias gradient is a short vector of
    sums that largely cancel: with few experts it moved by up to 1.5e-2 (bf16) and 5e-6 (fp32) of its norm.  The selection is that
    of exact arithmetic, so the chosen experts stay the same."""
    few = case["use"] != "forward" and case["E"] <= 8
    if case["dtype"] == "f32":
        return {"rel": 2e-5 if few else 6e-6, "max": 5e-5}
    return {"rel": 0.03 if few else 5e-3, "max": 0.13}
