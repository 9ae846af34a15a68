"""The calls this library is timed on: Gated MLP and Softmax+MatMul as a
serving program makes them, from one decode token to a prefill of thousands.

A case is a dict of plain values:

    op          "forward" (the whole MLP), "gate_up" or "down" (one of its two
                steps alone), or "softmax" (Softmax+MatMul)
    T, D, F     forward / gate_up / down: tokens, model width, hidden width;
                softmax: T rows of X, F the contracted width, D output columns
    activation  "silu", "swish" (with beta) or "sigmoid"; rmsnorm: RMSNorm of
                X in front
    plain       True: the call without workspace and output arguments, which
                allocates both; False: the serving form, which keeps a
                workspace per layer and writes into a buffer of its own

bf16 is the library's only data type, and it computes forward passes only.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2606_26344_amd import gmlp, softmax_matmul as smm

BETA = 1.702  # the swish slope of the SwiGLU variant
EPS = 1e-6


def _case(name, op, T, D, F, activation="silu", rmsnorm=False, plain=False):
    c = {"op": op, "T": T, "D": D, "F": F, "activation": activation, "rmsnorm": rmsnorm, "plain": plain}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a toy layer, bound by launches and host work.
        _case("tiny", "forward", 16, 256, 512, plain=True),
        # Single-stream decode of an 8B-class layer: one token, bound by the
        # weight stream.
        _case("decode", "forward", 1, 4096, 14336),
        # Decode of four sequences with the family's options: SwiGLU behind a
        # fused RMSNorm.
        _case("decode_4_swiglu_rms", "forward", 4, 4096, 14336, activation="swish", rmsnorm=True),
        # Batched decode: a few tens of sequences, one token each.
        _case("batch_24", "forward", 24, 4096, 14336),
        # A small model's batched decode, an odd batch, through the call that
        # allocates for itself.
        _case("batch_51_small", "forward", 51, 2048, 8192, plain=True),
        # The benchmark's small-batch workload.
        _case("batch_128", "forward", 128, 4096, 14336),
        # A ragged prompt on a 13B-class layer, RMSNorm in front.
        _case("prompt_300_rms", "forward", 300, 5120, 13824, rmsnorm=True),
        # A chunk of a prompt, ragged, gate/up step alone (the paper's
        # MM+MM+SiLU+Mul kernel) with the GLU gate.
        _case("gate_up_1000_glu", "gate_up", 1000, 4096, 14336, activation="sigmoid"),
        # Prefill, the benchmark's compute-bound workload.
        _case("prefill_4096", "forward", 4096, 4096, 14336),
        # Prefill of a 70B-class layer.
        _case("large_prefill_2048", "forward", 2048, 8192, 28672),
        # Softmax+MatMul at the paper's largest shape ...
        _case("softmax_8192", "softmax", 8192, 8192, 8192),
        # ... and near its smallest, with ragged rows.
        _case("softmax_2000", "softmax", 2000, 2048, 4096, plain=True),
    ]


# (D, F) of the repository's workloads and tests, and of the same class.
_WIDTHS = [(256, 512), (1024, 4096), (1032, 2056), (2048, 8192), (3072, 8192), (4096, 11008), (4096, 12288),
           (4096, 14336), (4096, 16384), (5120, 13824), (8192, 28672)]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    largest = work(_case(None, "forward", 2048, 8192, 28672))["flops"]
    while True:
        if rng.random() < 0.8:
            op = rng.choice(["forward", "forward", "forward", "forward", "gate_up", "down"])
            D, F = rng.choice(_WIDTHS)
            if rng.random() < 0.4:  # widths of no particular class
                D = 8 * _log_uniform(rng, 32, 1024)
                F = 8 * max(64, min(3584, int(D / 8 * rng.uniform(2.0, 4.0))))
            T = _log_uniform(rng, 1, 4096)
            if op == "down":
                c = _case(None, op, T, D, F, plain=rng.random() < 0.3)
            else:
                c = _case(None, op, T, D, F, activation=rng.choice(["silu", "silu", "silu", "swish", "sigmoid"]),
                          rmsnorm=rng.random() < 0.3, plain=rng.random() < 0.3)
        else:  # 2K to 8K in every dimension, fewer rows too
            c = _case(None, "softmax", _log_uniform(rng, 8, 8192), 8 * _log_uniform(rng, 128, 1024),
                      8 * _log_uniform(rng, 256, 1024), plain=rng.random() < 0.3)
        if work(c)["flops"] <= largest:
            return c


def _inputs(case, seed):
    """bf16 inputs with the distributions of the repository's generator:
    activations N(0, 1), weights N(0, 1/fan_in); for Softmax+MatMul N(0, 1)
    logits and right operand."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(rows, cols, scale):
        t = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
        step = max(1, (1 << 26) // cols)
        for r in range(0, rows, step):
            n = min(step, rows - r)
            t[r:r + n] = torch.randn((n, cols), generator=gen, device="cuda") * scale
        return t

    op, T, D, F = case["op"], case["T"], case["D"], case["F"]
    if op == "softmax":
        return {"x": normal(T, F, 1.0), "y": normal(F, D, 1.0)}
    if op == "down":
        # H as the gate/up step leaves it: a product of two unit-scale factors.
        h = normal(T, F, 0.6) * normal(T, F, 1.0)
        return {"h": h, "wd": normal(F, D, F ** -0.5)}
    t = {"x": normal(T, D, 1.0), "wg": normal(D, F, D ** -0.5), "wu": normal(D, F, D ** -0.5)}
    if op == "forward":
        t["wd"] = normal(F, D, F ** -0.5)
    return t


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    op, T, D, F = case["op"], case["T"], case["D"], case["F"]
    s["kw"] = {}
    if op in ("forward", "gate_up"):
        if case["activation"] != "silu":
            s["kw"]["activation"] = case["activation"]
        if case["activation"] == "swish":
            s["kw"]["beta"] = BETA
        if case["rmsnorm"]:
            s["kw"].update(rmsnorm=True, eps=EPS)
    if not case["plain"]:
        if op == "softmax":
            s["kw"]["workspace"] = smm.make_workspace(T, F, D)
        else:
            s["kw"]["workspace"] = gmlp.Workspace(T, D, F)
        s["kw"]["out"] = torch.empty((T, F if op == "gate_up" else D), dtype=torch.bfloat16, device="cuda")
    return s


def run(s):
    op, kw = s["case"]["op"], s["kw"]
    if op == "forward":
        return gmlp.forward(s["x"], s["wg"], s["wu"], s["wd"], **kw)
    if op == "gate_up":
        return gmlp.gate_up(s["x"], s["wg"], s["wu"], **kw)
    if op == "down":
        return gmlp.down(s["h"], s["wd"], **kw)
    return smm.softmax_matmul(s["x"], s["y"], **kw)


def work(case):
    op, T, D, F = case["op"], case["T"], case["D"], case["F"]
    if op == "softmax":
        return {"bytes": 2.0 * (T * F + F * D + T * D), "flops": 2.0 * T * F * D}
    if op == "down":
        return {"bytes": 2.0 * (T * F + F * D + T * D), "flops": 2.0 * T * F * D}
    if op == "gate_up":
        return {"bytes": 2.0 * (T * D + 2 * D * F + T * F), "flops": 4.0 * T * D * F}
    return {"bytes": 2.0 * (3 * D * F + 2 * T * D), "flops": 6.0 * T * D * F}


def tolerance(case):
    """bf16 results (and a bf16 H inside the whole MLP) of fp32 sums: two
    implementations that add in another order differ by single bf16 steps
    here and there.  Measured between the library's GEMV and MFMA paths on the
    same inputs (T = 2..8, widths 256 to 28672): rel at most 4.1e-4, max 7.8e-3;
    four times that."""
    return {"rel": 2e-3, "max": 3.2e-2}


def exact(case, seed):
    s = {k: v.double() for k, v in _inputs(case, seed).items()}
    op = case["op"]
    if op == "softmax":
        return torch.softmax(s["x"], dim=1) @ s["y"]
    if op == "down":
        return s["h"] @ s["wd"]
    x = s["x"]
    r = torch.rsqrt(x.square().mean(dim=1, keepdim=True) + EPS) if case["rmsnorm"] else 1.0
    g, u = (x * r) @ s["wg"], (x * r) @ s["wu"]
    if case["activation"] == "sigmoid":
        h = torch.sigmoid(g) * u
    else:
        h = g * torch.sigmoid(g * (BETA if case["activation"] == "swish" else 1.0)) * u
    return h if op == "gate_up" else h @ s["wd"]
