"""Timed cases of the MoE layer: what a program that uses this package has it do, through its public entry points.

Two kinds of case.  A "forward" case is one pass of the whole layer (`binding.forward`) on weights, buffers and a
workspace that the program keeps, with the epoch raised on every pass.  A "pieces" case is a program that computes the
experts itself and takes the gate, the dispatch and the combine from here as three calls.  Inputs follow the
package's workloads: x ~ N(0,1), weights ~ N(0,0.02), an fp32 offset per expert on the gate logits where load is
skewed, pre-routed rows with Zipf(1.1) popularity of the local experts.
"""
from __future__ import annotations

import math

import torch

from paper_2605_00686_amd import binding as B

W_STD = 0.02
_DEFAULTS = dict(kind="forward", dtype="bf16", tile_m=0, bias_std=0.0, prerouted=False, capacity=0, ready_queue=False)


def _case(**kw):
    return {**_DEFAULTS, **kw}


def listed():
    return [
        # the smallest layer anybody runs, in fp32 (a unit test or a reference run of a program that uses the package)
        _case(name="tiny_f32", T=256, d=512, E=8, k=2, f=1024, R=2, dtype="f32"),
        # serving a handful of sequences: one decode step of 8 tokens on a layer of many small experts; latency
        _case(name="decode_8", T=8, d=2048, E=128, k=8, f=768, R=8, tile_m=32, bias_std=0.5),
        # serving: a decode step of 128 sequences on the same layer; every expert is reached, each by a few rows
        _case(name="decode_128", T=128, d=2048, E=128, k=8, f=768, R=8, tile_m=32, bias_std=0.5),
        # serving: a decode step on one rank of a wide expert-parallel layer that publishes to 64 destinations
        _case(name="decode_wide", T=128, d=7168, E=32, k=8, f=2048, R=64, tile_m=32),
        # a short prompt or a mixed prefill/decode step: odd sizes, tens of rows per expert, padded layout of the rows
        _case(name="mixed_odd", T=1001, d=1024, E=48, k=6, f=1408, R=7, capacity=256),
        # prefill of 4096 tokens on the layer of many small experts, skewed load
        _case(name="prefill_small_experts", T=4096, d=2048, E=128, k=8, f=768, R=8, bias_std=0.5),
        # prefill on a layer whose dimensions are no powers of two (ragged column tiles)
        _case(name="prefill_odd_dims", T=4096, d=2880, E=128, k=4, f=2880, R=8),
        # rows that arrive already routed from 64 peers at a rank that holds four experts
        _case(name="arriving_rows", T=8192, d=7168, E=4, k=1, f=2048, R=64, prerouted=True),
        # the largest: 16384 tokens on few large experts, bound by the matrix cores
        _case(name="large_experts", T=16384, d=4096, E=8, k=2, f=14336, R=8),
        # the same prefill on ready queues: what a layer with peers whose rows arrive at unknown times would run
        _case(name="prefill_ready_queue", T=2048, d=2048, E=64, k=8, f=1024, R=8, ready_queue=True),
        # gate, dispatch and combine around a program's own expert computation: prefill ...
        _case(name="pieces_prefill", kind="pieces", T=4096, d=2048, E=128, k=8, f=768, R=8, bias_std=0.5),
        # ... and a decode step of 128 tokens
        _case(name="pieces_decode", kind="pieces", T=128, d=2048, E=128, k=8, f=768, R=8, bias_std=0.5),
    ]


def _log_uniform(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    """One more case of the ranges above: 1 to 16384 tokens, 4 to 256 experts, d and f from 512 up."""
    while True:
        dtype = "f32" if rng.random() < 0.12 else "bf16"
        kind = "pieces" if rng.random() < 0.2 else "forward"
        prerouted = kind == "forward" and rng.random() < 0.12
        T = _log_uniform(rng, 1, 16384)
        E = _log_uniform(rng, 4, 16 if prerouted else 256)
        k = 1 if prerouted else rng.choice([k for k in (1, 2, 2, 4, 6, 8, 8) if k <= E])
        d = _log_uniform(rng, 512, 7168, 64)
        f = _log_uniform(rng, 512, 14336, 64)
        # few large experts or many small ones, no larger than the largest layer above; fp32 layers are small
        if 3 * E * d * f * 2 > 12e9 or T * k * 6 * d * f > 1.1e13 or T * k * d > 1.2e8:
            continue
        if dtype == "f32" and (E * d * f > 1.5e8 or T * k * 6 * d * f > 3e10):
            continue
        R = rng.choice([r for r in range(1, 65) if T % r == 0])
        rows = T * k / E
        capacity = 0
        if kind == "forward" and not prerouted and rng.random() < 0.2:
            capacity = min(T, 64 * (int(3 * rows) // 64 + 2))
        return _case(kind=kind, dtype=dtype, T=T, d=d, E=E, k=k, f=f, R=R, prerouted=prerouted,
                     tile_m=32 if rows < 96 and dtype == "bf16" and rng.random() < 0.7 else 0,
                     bias_std=0.0 if capacity or prerouted else rng.choice([0.0, 0.5]), capacity=capacity,
                     ready_queue=kind == "forward" and rng.random() < 0.15)


def prepare(case, seed):
    T, d, E, k, f = (case[n] for n in ("T", "d", "E", "k", "f"))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=1.0, dtype=dt):
        t = torch.empty(shape, dtype=dtype, device="cuda")
        for part in (t if len(shape) == 3 else (t,)):
            part.normal_(0.0, std, generator=gen)
        return t

    p = B.problem(T, d, E, k, f, case["R"], dt, tile_m=case["tile_m"], capacity=case["capacity"],
                  scheduler=B.MOE_SCHED_READY_QUEUE if case["ready_queue"] else B.MOE_SCHED_STATIC)
    s = {"kind": case["kind"], "p": p, "buf": B.Buffers(p), "x": normal(T, d), "Wg": None, "bias": None}
    if case["prerouted"]:
        # popularity of the local experts: the first E ranks of a Zipf law; a row's weight is one share of a top-8 gate
        pmf = torch.arange(1, E + 1, dtype=torch.float32, device="cuda").pow(-1.1)
        s["buf"].topk_idx.copy_(torch.multinomial(pmf, T, replacement=True, generator=gen).reshape(T, 1))
        shares = torch.rand(T, 8, generator=gen, device="cuda") + 0.05
        s["buf"].topk_w.copy_(shares[:, :1] / shares.sum(dim=1, keepdim=True))
    else:
        s["Wg"] = normal(d, E, std=W_STD)
        if case["bias_std"] > 0:
            s["bias"] = normal(E, std=case["bias_std"], dtype=torch.float32)
    if case["kind"] == "forward":
        s["W1"], s["W3"], s["W2"] = normal(E, d, f, std=W_STD), normal(E, d, f, std=W_STD), normal(E, f, d, std=W_STD)
    else:
        s["buf"].staging.normal_(0.0, 0.5, generator=gen)  # the expert outputs, computed by the program itself
        s["x_perm"] = torch.empty((T * k, d), dtype=dt, device="cuda")
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return s


def run(s):
    p, b = s["p"], s["buf"]
    if s["kind"] == "pieces":
        B.moe_route(p, s["x"], s["Wg"], s["bias"], b.topk_idx, b.topk_w)
        B.moe_dispatch(p, s["x"], b.topk_idx, b.counts, b.offsets, b.perm, b.inv_perm, s["x_perm"], s["status"], b.workspace)
        B.moe_combine(p, b.staging, None, None, b.topk_w, b.out, s["status"])
        return {"topk_idx": b.topk_idx, "topk_w": b.topk_w, "counts": b.counts, "offsets": b.offsets, "perm": b.perm,
                "inv_perm": b.inv_perm, "x_perm": s["x_perm"], "out": b.out, "status": s["status"]}
    p.epoch += 1  # (flags are left out of what is returned: their value is the number of the pass)
    B.forward(p, b, s["x"], s["Wg"], s["bias"], s["W1"], s["W3"], s["W2"])
    return {"topk_idx": b.topk_idx, "topk_w": b.topk_w, "counts": b.counts, "offsets": b.offsets, "perm": b.perm,
            "inv_perm": b.inv_perm, "slot_flag": b.slot_flag, "staging": b.staging, "out": b.out}


def work(case):
    T, d, E, k, f = (case[n] for n in ("T", "d", "E", "k", "f"))
    N, sz = T * k, 4 if case["dtype"] == "f32" else 2
    gate_bytes = 0 if case["prerouted"] else d * E * sz
    gate_flops = 0 if case["prerouted"] else 2 * T * d * E
    rows = case["E"] * case["capacity"] if case["capacity"] else N
    ints = 4 * (2 * N + rows + N + 2 * E)  # choices and their weights, both permutations, counts and offsets
    if case["kind"] == "pieces":
        return {"bytes": T * d * sz + gate_bytes + 2 * N * d * sz + T * d * sz + ints, "flops": gate_flops + 2 * N * d}
    reached = E * (1.0 - (1.0 - k / E) ** T)  # experts whose weights are read, for even routing
    return {"bytes": T * d * sz + gate_bytes + reached * 3 * d * f * sz + N * d * sz + T * d * sz + ints + 4 * N,
            "flops": gate_flops + N * 6 * d * f}


def tolerance(case):
    # Measured against the same layer with its sums in another order (torch matrix products per expert; fp64 ones for
    # fp32 layers), about four times what that showed; whole numbers (routing, counts, permutations, flags) agree.
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5}  # seen: 8.3e-7 and 4.6e-6
    # other orders of the fp32 sums flip a few roundings of h and of the rows by one unit in the last place, which is up
    # to 2^-7 of a value; seen: rel 4.1e-4, max 1.6e-2
    return {"rel": 2e-3, "max": 4e-2}
