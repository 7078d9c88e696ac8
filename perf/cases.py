"""Performance cases of the MoE expert layer: the calls a training or serving program makes, over the range of
sizes, storage types and options it makes them with.

A case is a dict of plain values.  `prepare` builds what such a program holds before a call (weights, inputs, the
layer or engine object with its buffers), `run` makes ONE pass through the public entry points and returns the
outputs, `work` states the bytes and operations the pass cannot do without, `tolerance` how far two correct
implementations of the same precision may differ.

Fields: op      "step" forward + backward, "ckpt" the same with activation checkpointing, "fwd" forward alone,
                "zebra" one iteration of the micro-batched engine (L layers, R micro-batches of T tokens)
        T d f E k, dtype "f32" | "bf16" | "f16", act "gelu" | "swiglu"
        cap     capacity factor (0 = unlimited), zipf skew of the router bias (0 = none),
        partial this GPU computes the lower half of the experts in full and of the upper half only the tail
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_03871_amd import binding as B
from paper_2504_03871_amd.layer import MoELayer
from paper_2504_03871_amd.zebra import ZebraExpertEngine

DTYPES = {"f32": B.DTYPE_F32, "bf16": B.DTYPE_BF16, "f16": B.DTYPE_F16}
ACTS = {"gelu": B.ACT_GELU, "swiglu": B.ACT_SWIGLU}


def _case(op, T, d, f, E, k, dtype="bf16", act="gelu", cap=0.0, zipf=0.0, partial=False, L=1, R=1, name=None):
    c = dict(op=op, T=T, d=d, f=f, E=E, k=k, dtype=dtype, act=act, cap=cap, zipf=zipf, partial=partial, L=L, R=R)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the full-precision configuration: small-model runs and gradient checks; every call is short
        _case("step", 512, 128, 256, 8, 2, dtype="f32", name="f32_step_small"),
        # full precision at the size of a small training run, sizes that are multiples of four and nothing more
        _case("step", 2000, 516, 1540, 8, 2, dtype="f32", act="swiglu", name="f32_step_odd"),
        # generation: one forward pass over the few tokens of a decode batch, Mixtral-like layer
        _case("fwd", 16, 4096, 14336, 8, 2, act="swiglu", name="fwd_decode"),
        # a short prompt or an evaluation batch: forward alone, an odd number of tokens
        _case("fwd", 1001, 2048, 8192, 16, 2, dtype="f16", name="fwd_prompt"),
        # the micro-batched engine on its streams: weight gradients accumulate over the micro-batches.  One layer: a
        # second one routes on the first one's rounded output, where a last-bit difference can move whole tokens
        _case("zebra", 2048, 1024, 4096, 8, 2, R=4, name="zebra_microbatches"),
        # ordinary training steps: the hidden sizes of the paper's models
        _case("step", 8192, 1024, 4096, 8, 2, name="step_1024"),
        # the paper's own setting: FP16 storage, activation checkpointing, a skewed router
        _case("ckpt", 8192, 2048, 8192, 16, 2, dtype="f16", zipf=1.2, name="ckpt_f16_skewed"),
        # one GPU's share under asymmetric expert assignment: some experts in full, of the others a slice
        _case("step", 16384, 2048, 8192, 32, 4, cap=1.25, partial=True, name="step_partial"),
        # ragged everything: odd token count, widths that are multiples of 64 only, capacity drops, top-3 of six
        _case("step", 3001, 1088, 2880, 6, 3, act="swiglu", cap=0.8, zipf=0.7, name="step_ragged"),
        # many small experts, top-8
        _case("step", 8192, 2048, 1024, 128, 8, act="swiglu", name="step_many_experts"),
        # the headline workload of the benchmark, the largest that is run
        _case("step", 32768, 4096, 14336, 8, 2, act="swiglu", name="step_large"),
    ]


def _log_int(rng, lo, hi, mult=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // mult * mult, max(-(-lo // mult) * mult, int(round(v / mult)) * mult))


def draw(rng):
    """One more case of the listed ranges; sizes over their logarithm, never dearer than the largest listed."""
    while True:
        op = rng.choice(["step", "step", "step", "fwd", "fwd", "ckpt", "zebra"])
        act = rng.choice(["gelu", "swiglu"])
        cap, zipf = rng.choice([0.0, 0.0, 0.8, 1.25]), rng.choice([0.0, 0.0, 0.7, 1.2])
        partial = op == "step" and rng.random() < 0.25
        if op != "zebra" and rng.random() < 0.2:
            E = _log_int(rng, 4, 32)
            c = _case(op, _log_int(rng, 64, 4096), _log_int(rng, 64, 1024, 4), _log_int(rng, 128, 4096, 4), E,
                      rng.randint(1, min(E, 4)), "f32", act, cap, zipf, partial)
        elif op == "zebra":
            E = _log_int(rng, 4, 32)
            c = _case(op, _log_int(rng, 512, 4096), _log_int(rng, 512, 2048, 64), _log_int(rng, 1024, 8192, 64), E,
                      rng.randint(1, min(E, 4)), rng.choice(["bf16", "bf16", "f16"]), act, R=rng.randint(2, 6))
        else:
            many = rng.random() < 0.25
            E = _log_int(rng, 64, 256) if many else _log_int(rng, 4, 48)
            k = rng.randint(2, 8) if many else rng.randint(1, 4)
            T = _log_int(rng, 1 if op == "fwd" else 256, 32768)
            c = _case(op, T, _log_int(rng, 512, 4096, 64), _log_int(rng, 512, 2048, 64) if many else
                      _log_int(rng, 1024, 14336, 64), E, k, rng.choice(["bf16", "bf16", "f16"]), act, cap, zipf, partial)
        big = listed()[-1]
        w, b = work(c), work(big)
        if w["flops"] <= b["flops"] / 4 and w["bytes"] <= b["bytes"] / 2:
            return c


# ---- inputs --------------------------------------------------------------------------------------------------

def _capacity(c):
    return math.ceil(c["cap"] * c["T"] * c["k"] / c["E"]) if c["cap"] > 0 else 0


def _bias(c):
    if c["zipf"] <= 0:
        return None
    return torch.tensor([-c["zipf"] * math.log(e + 1) for e in range(c["E"])], dtype=torch.float32)


def _normal_(t, gen, std):
    """N(0, std^2), drawn in fp32 and rounded once to the storage type, a piece of the tensor at a time."""
    flat, step = t.view(-1), 1 << 27
    for i in range(0, flat.numel(), step):
        p = flat[i:i + step]
        p.copy_(torch.randn(p.numel(), generator=gen, device=t.device, dtype=torch.float32).mul_(std))


def _fill_params(m, c, gen):
    _normal_(m.Wr, gen, c["d"] ** -0.5)
    for w in (m.W1, m.W1b, m.W2):
        if w is not None:
            _normal_(w, gen, 0.02)
    b = _bias(c)
    m.bias = b.to(m.device) if b is not None else None


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    dt, act = DTYPES[c["dtype"]], ACTS[c["act"]]
    if c["op"] == "zebra":
        eng = ZebraExpertEngine(c["L"], c["R"], c["T"], c["d"], c["f"], c["E"], c["k"], dtype=dt, act=act)
        for m in eng.params:
            _fill_params(m, c, gen)
        for j in range(c["R"]):
            _normal_(eng.act[0][j], gen, 1.0)
            _normal_(eng.grad[c["L"]][j], gen, 1.0)
        return dict(op="zebra", engine=eng, L=c["L"], R=c["R"])
    m = MoELayer(c["T"], c["d"], c["f"], c["E"], c["k"], dtype=dt, act=act, capacity=_capacity(c))
    _fill_params(m, c, gen)
    _normal_(m.x, gen, 1.0)
    if c["op"] != "fwd":
        _normal_(m.d_out, gen, 1.0)
    if c["partial"]:
        cut = int(0.6 * c["T"] * c["k"] / c["E"])      # the last 40 % of an evenly loaded expert's rows
        lo = [0 if e < c["E"] // 2 else cut for e in range(c["E"])]
        m.set_slices(lo, [2 ** 31 - 1] * c["E"])
    return dict(op=c["op"], layer=m)


def _param_grads(m):
    out = dict(dW1=m.dW1, dW2=m.dW2, dWr=m.dWr)
    if m.dW1b is not None:
        out["dW1b"] = m.dW1b
    return out


def run(state):
    if state["op"] == "zebra":
        eng = state["engine"]
        eng.run_iteration()
        out = {f"out{j}": eng.act[state["L"]][j] for j in range(state["R"])}
        out.update({f"dx{j}": eng.grad[0][j] for j in range(state["R"])})
        for i, m in enumerate(eng.params):
            out.update({f"{n}_{i}": t for n, t in _param_grads(m).items()})
        return out
    m = state["layer"]
    if state["op"] == "fwd":
        m.forward()
        return dict(out=m.out, logits=m.logits, topk_idx=m.topk_idx, topk_w=m.topk_w)
    if state["op"] == "ckpt":
        m.step_checkpointed()
    else:
        m.step()
    return dict(out=m.out, logits=m.logits, topk_idx=m.topk_idx, topk_w=m.topk_w, dx=m.dx, **_param_grads(m))


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def _rows(c):
    """Expected assignment rows this GPU computes and expected experts that have any, from the routing statistics
    (standard normal logits plus the bias) of a fixed sample of tokens."""
    n = 2048
    logits = np.random.default_rng(1).standard_normal((n, c["E"]))
    b = _bias(c)
    if b is not None:
        logits += b.numpy()
    top = np.argpartition(-logits, c["k"] - 1, axis=1)[:, :c["k"]]
    p = np.bincount(top.ravel(), minlength=c["E"]) / n           # chance that a token goes to expert e
    rows = p * c["T"]
    cap = _capacity(c)
    if cap > 0:
        rows = np.minimum(rows, cap)
    if c["partial"]:
        rows[c["E"] // 2:] = np.maximum(rows[c["E"] // 2:] - int(0.6 * c["T"] * c["k"] / c["E"]), 0)
    return float(rows.sum()), float((1.0 - (1.0 - p) ** c["T"]).sum())


def work(case):
    c = case
    s = 4 if c["dtype"] == "f32" else 2
    mats = 3 if c["act"] == "swiglu" else 2
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    S, live = _rows(c)
    weights, grads = live * mats * d * f * s, E * mats * d * f * 4
    gate = T * d * E * 2
    fwd = dict(flops=2 * mats * S * d * f + gate, bytes=2 * T * d * s + T * k * 8 + d * E * 4)
    if c["op"] == "fwd":
        return dict(flops=fwd["flops"], bytes=fwd["bytes"] + weights)
    flops = 3 * fwd["flops"]
    if c["op"] == "ckpt":                                        # the first GEMM(s) and the gate once more
        flops += 2 * (mats - 1) * S * d * f + gate
    act = 4 * T * d * s + T * k * 8                              # x, d_out in; out, dx and the routing out
    if c["op"] == "zebra":
        L, R = c["L"], c["R"]
        return dict(flops=flops * L * R, bytes=R * 4 * T * d * s + L * (weights + grads + 2 * d * E * 4))
    return dict(flops=flops, bytes=act + weights + grads + 2 * d * E * 4)


def tolerance(case):
    # Measured against the same layer evaluated in fp64 (largest over out, dx and the weight gradients; 2-norm):
    # fp32 3.8e-7 at d 128, f 256 and 1.1e-6 at d 516, f 1540, growing with the length of the sums; bf16 3.9e-3 and
    # fp16 4.9e-4, from the roundings of the intermediate tensors to the storage type.  Stated: about four times
    # that (fp32: at its longest sums).  Largest single difference in fp32: 7.8e-6 of the rms.  None is stated for
    # 16-bit storage: a token whose k-th and next logits lie within rounding of each other may go to either expert.
    tol = {"f32": {"rel": 1e-5, "max": 5e-5}, "bf16": {"rel": 1.6e-2}, "f16": {"rel": 2e-3}}[case["dtype"]]
    return dict(tol, differ=1e-4)
