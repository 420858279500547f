"""What this library is timed on: one MoE layer on one GPU, from single decode steps to the largest training layer.

Every case goes through `MoELayer` (paper_2304_03946_amd/layer.py), whose methods are the sequences of C-ABI calls a
user's program makes.  Inputs follow workloads.py: x ~ N(0, 1) with a constant last feature that carries the gate's
skew bias, W_g ~ N(0, 1) / sqrt(d), expert weights ~ N(0, 0.02^2), dY ~ N(0, 1); expert loads follow a Zipf law (the
paper's load trace: ten of 64 experts take about three quarters of the tokens), and the placement table is the greedy
capacity rule on the expected loads.

Passes:
  infer       forward only, nothing kept for a backward pass (top-1 layers and gathered loads where they are supported)
  train       forward, then the backward pass of the expert path: dX, dW1, dW2
  train_full  forward with biases, then every gradient of a trainable layer: also db1, db2, dW_g and the gate's share of dX
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2304_03946_amd import binding as B
from paper_2304_03946_amd import workloads as W
from paper_2304_03946_amd.layer import MoELayer

_ACT = {"relu": B.RELU, "gelu": B.GELU_ERF, "gelu_tanh": B.GELU_TANH}


def _case(name, mode, dtype, N, d, f, E, k, V, zipf, act="gelu"):
    c = {"mode": mode, "dtype": dtype, "N": N, "d": d, "f": f, "E": E, "k": k, "V": V, "zipf": zipf, "act": act}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the fp32 layer of workloads.CONFIGS: a call so small that launches are all it costs
        _case("tiny_fp32", "infer", "f32", 256, 64, 256, 4, 1, 4, 0.0, "relu"),
        # fp32 training of a small layer: gradient checks, reference runs
        _case("fp32_train", "train_full", "f32", 1000, 256, 1024, 8, 2, 10, 1.0),
        # one decode step of a small serving batch on the GPT-medium-like layer
        _case("decode_16", "infer", "bf16", 16, 1024, 4096, 32, 2, 48, 1.2),
        # one decode step of a large serving batch on the GPT-XL-like layer: every expert's weights for a few rows each
        _case("decode_xl_256", "infer", "bf16", 256, 2048, 8192, 64, 2, 96, 1.5),
        # a prompt of ragged length through the same layer
        _case("prefill_xl_2000", "infer", "bf16", 2000, 2048, 8192, 64, 2, 96, 1.5),
        # the BERT-like layer, forward
        _case("bert_infer", "infer", "bf16", 8192, 768, 3072, 16, 2, 18, 1.2),
        # many small experts, four per token
        _case("fine_grained", "infer", "bf16", 4096, 512, 1024, 128, 4, 160, 0.8),
        # a narrow layer whose sizes are no multiples of the usual tile sizes, every gradient
        _case("narrow_full", "train_full", "bf16", 5003, 192, 768, 12, 2, 15, 0.8, "gelu_tanh"),
        # a small training batch of odd length on the GPT-medium-like layer, every gradient
        _case("gpt_m_1500_full", "train_full", "bf16", 1500, 1024, 4096, 32, 2, 48, 1.2),
        # the Swin-like layer (top-1), training
        _case("swin_train", "train", "bf16", 32768, 512, 2048, 32, 1, 40, 1.0),
        # the GPT-medium-like layer, training
        _case("gpt_m_train", "train", "bf16", 16384, 1024, 4096, 32, 2, 48, 1.2),
        # the GPT-XL-like layer, training: the largest configuration, and the benchmark's default
        _case("gpt_xl_train", "train", "bf16", 65536, 2048, 8192, 64, 2, 96, 1.5),
    ]


def _cost(c):
    return (3 if c["mode"] != "infer" else 1) * c["N"] * c["k"] * c["d"] * c["f"]


def draw(rng):
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        fp32 = rng.random() < 0.2
        mode = rng.choice(["infer", "infer", "train", "train", "train_full"])
        step = rng.choice([8, 64, 128, 128])                       # granularity of the feature sizes
        d = max(step, log_uniform(64, 512 if fp32 else 2048) // step * step)
        f = max(step, d * rng.choice([2, 3, 4, 4, 4]) // step * step)
        E = log_uniform(4, 16 if fp32 else 128)
        k = rng.choice([1, 2, 2, 2, 4])
        V = E + rng.randrange(0, E // 2 + 1)
        N = log_uniform(8, 4096 if fp32 else 65536)
        zipf = round(rng.uniform(0.5, 1.5), 2)
        act = rng.choice(["gelu", "gelu", "gelu", "gelu_tanh", "relu"])
        c = _case(None, mode, "f32" if fp32 else "bf16", N, d, f, E, k, V, zipf, act)
        largest = 3 * 131072 * 2048 * 8192
        if _cost(c) * (64 if fp32 else 1) <= largest and E * d * f <= 64 * 2048 * 8192:
            return c


def _shares(E, k, zipf):
    """Share of the assignments per load rank: rank^-zipf, no expert above what k distinct experts per token allow."""
    p = (np.arange(E) + 1.0) ** (-zipf)
    p /= p.sum()
    cap = 0.98 / k if k > 1 else 1.0
    for _ in range(E):
        over = p > cap
        if not over.any():
            break
        rest = 1.0 - cap * over.sum()
        p = np.where(over, cap, p * rest / p[~over].sum())
    return p


@functools.lru_cache(maxsize=64)
def _bias(E, k, zipf):
    """Gate bias per load rank under which the expected loads follow `_shares` (logit noise of variance 1), on a
    coarser quadrature than workloads.solve_bias takes for its configurations: loads within a few per cent."""
    if k == E or zipf == 0.0:
        return np.zeros(E)
    p = _shares(E, k, zipf)
    sigma = np.ones(E)
    b = np.log(p / p.max())
    slope = np.ones(E)
    want = np.log(np.minimum(k * p, 1.0 - 1e-9))
    got = np.log(np.maximum(W.inclusion_probabilities(b, sigma, k, 65), 1e-12))
    for _ in range(12):
        if np.max(np.abs(want - got)) < 0.05:
            break
        b_new = b + np.clip((want - got) / slope, -1.0, 1.0)
        b_new -= b_new.max()
        got_new = np.log(np.maximum(W.inclusion_probabilities(b_new, sigma, k, 65), 1e-12))
        db = b_new - b
        est = np.where(np.abs(db) > 1e-9, (got_new - got) / np.where(np.abs(db) > 1e-9, db, 1.0), slope)
        slope = np.clip(np.where(np.isfinite(est) & (est > 0), est, slope), 0.2, 20.0)
        b, got = b_new, got_new
    return b


def prepare(case, seed):
    N, d, f, E, k, V = (case[n] for n in ("N", "d", "f", "E", "k", "V"))
    k = min(k, E)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, std):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)

    ranks = np.random.default_rng(seed).permutation(E)             # load rank of each expert
    x = normal((N, d), 1.0)
    wg = normal((d, E), 1.0 / math.sqrt(d))
    x[:, d - 1] = 1.0
    wg[d - 1] = torch.from_numpy(_bias(E, k, case["zipf"])[ranks]).to(wg)
    loads = N * k * _shares(E, k, case["zipf"])[ranks]
    rep_off, rep_ids = W.placement_from_loads(loads, V, 8)
    train = case["mode"] != "infer"
    state = {
        "mode": case["mode"], "x": x, "wg": wg, "w1": normal((E, d, f), 0.02), "w2": normal((E, f, d), 0.02),
        "rep_off": rep_off, "rep_ids": rep_ids, "b1": None, "b2": None,
        "layer": MoELayer(N, d, f, E, k, V, B.BF16 if case["dtype"] == "bf16" else B.F32, _ACT[case["act"]], backward=train),
    }
    if train:
        state["dy"] = normal((N, d), 1.0)
    if case["mode"] == "train_full":
        state["b1"], state["b2"] = normal((E, f), 0.02), normal((E, d), 0.02)
    return state


def run(state):
    L, x, wg, w1, w2 = (state[n] for n in ("layer", "x", "wg", "w1", "w2"))
    rep, b1, b2 = (state["rep_off"], state["rep_ids"]), state["b1"], state["b2"]
    if state["mode"] == "infer":
        if L.top1_supported():
            L.forward_top1(x, wg, w1, w2, *rep, keep_hpre=False)
        elif L.gather_supported() and L.d % 128 == 0:
            L.forward_fused(x, wg, w1, w2, *rep, keep_hpre=False)
        else:
            L.forward(x, wg, w1, w2, *rep, keep_hpre=False)
        return {"y": L.y, "topk_idx": L.topk_idx, "topk_w": L.topk_w}
    L.forward(x, wg, w1, w2, *rep, b1=b1, b2=b2)
    if state["mode"] == "train_full":
        grads = L.backward_full(state["dy"], wg, w1, w2)
        return {"y": L.y, **{n: grads[n] for n in ("dx", "dw1", "dw2", "db1", "db2", "dwg")}}
    step = L.backward_top1 if L.top1_supported() else L.backward
    dx, dw1, dw2 = step(state["dy"], w1, w2)
    return {"y": L.y, "dx": dx, "dw1": dw1, "dw2": dw2}


def work(case):
    N, d, f, E = (case[n] for n in ("N", "d", "f", "E"))
    k = min(case["k"], E)
    A = N * k
    s = 2 if case["dtype"] == "bf16" else 4
    # experts that get at least one token: the others' weights are never read
    p = np.minimum(k * _shares(E, k, case["zipf"]), 1.0)
    active = float((1.0 - (1.0 - p) ** N).sum())
    weights = 2.0 * d * f * s
    b = 2 * N * d * s + d * E * s + 8 * A + active * weights
    flops = 2.0 * N * d * E + 4.0 * A * d * f
    if case["mode"] != "infer":
        b += 2 * N * d * s + E * weights
        flops += 8.0 * A * d * f
    if case["mode"] == "train_full":
        b += 2 * E * (d + f) * s + d * E * s
        flops += 6.0 * A * d + 2.0 * A * (d + f)
    return {"bytes": b, "flops": flops}


def tolerance(case):
    # Measured against a 64-bit evaluation of the same inputs with the same selection: bf16 (a rounding of 2^-9 at each of
    # the stored intermediates, four between x and y, six between dY and dW) at most 3.7e-3 in norm and 0.12 in the worst
    # element of dX; fp32 at most 6.8e-7 and 1.1e-5 on sums of a thousand products, longer ones grow with the root.
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.3, "differ": 1e-3}
    return {"rel": 5e-6, "max": 1e-4, "differ": 1e-3}
