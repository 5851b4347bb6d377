"""The layer's work that is measured: what a user of the framework has it do, through its public calls.

A case names an operation and a layer shape (notation of include/lazarus_moe.h: T tokens, model
dimension d, hidden dimension ffn, E experts, top-k, N ranks of c replica slots each).  Operations:

  forward        MoELayer.forward: route, dispatch, permute, expert FFN, combine
  forward_fused  MoELayer.forward_fused: the same, the reshuffle read by the first GEMM
  train          MoELayer.forward_train and backward: one training step of the layer
  accumulate     one optimizer step over two micro-batches with fp32 gradient accumulators
  dispatch       MoELayer.route and plan_dispatch alone: the integer half of the layer, for a
                 program that brings its own experts
  replan         ranks are lost: lz_replan on the survivors, then the replica copies of its plan

Inputs follow the synthetic workloads of this repository: logits N(0, 1) plus a Zipf(s) popularity
bias over a seeded ranking of the experts, x and dy N(0, 1), weights N(0, 0.02), every slot holding
its own copy of its expert, plan = Eq. 1 and MRO placement on the loads of an earlier batch of the
same popularity (a plan is made from history, not from the batch it serves).
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import paper_2407_04656_amd as lz

DEV = "cuda:0"
WEIGHT_STD = 0.02


def _case(name, op, dtype, act, T, d, ffn, E, k, N, c, zipf=1.0, lost=0):
    out = dict(op=op, dtype=dtype, act=act, T=T, d=d, ffn=ffn, E=E, k=k, N=N, c=c, zipf=zipf, lost=lost)
    return dict(out, name=name) if name else out


def listed():
    return [
        # the smallest call: the fp32 test layer, a few kernel launches
        _case("forward_f32_tiny", "forward", "f32", "gelu", 256, 128, 256, 8, 2, 4, 4, 0.5),
        # a few sequences' next tokens, or the last fragment of a batch: every slot's weights for a handful of rows
        _case("forward_small", "forward", "bf16", "swiglu", 64, 1024, 4096, 8, 2, 8, 2),
        # the headline layer: one batch through eight large experts
        _case("forward_c2", "forward", "bf16", "swiglu", 8192, 4096, 14336, 8, 2, 8, 2),
        # many GELU experts with a skewed load (32 experts on 48 slots)
        _case("forward_c3", "forward", "bf16", "gelu", 16384, 2048, 8192, 32, 2, 8, 6, 1.2),
        # fine-grained experts, top-6, with the reshuffle fused into the first GEMM
        _case("forward_fused_c4", "forward_fused", "bf16", "swiglu", 16384, 2048, 1408, 64, 6, 16, 8, 1.1),
        # feature sizes that no power of two divides, a ragged batch
        _case("forward_odd", "forward", "bf16", "swiglu", 3001, 1000, 2664, 8, 2, 6, 2),
        # the headline layer's training step (the most arithmetic)
        _case("train_c2", "train", "bf16", "swiglu", 8192, 4096, 14336, 8, 2, 8, 2),
        # a small language model's layer as it is trained: top-1, batch 4 x 1024 tokens on each of 10 ranks of 6 slots
        _case("train_top1", "train", "bf16", "gelu", 40960, 768, 3072, 8, 1, 10, 6),
        # fine-grained experts trained with two micro-batches per optimizer step
        _case("accumulate_c4", "accumulate", "bf16", "swiglu", 4096, 2048, 1408, 64, 6, 16, 8, 1.1),
        # full-precision training: gradient checks, ablations at small width
        _case("train_f32", "train", "f32", "gelu", 1024, 512, 2048, 8, 2, 4, 4),
        # routing and dispatch of a wide mixture: 256 experts, top-8, 32 ranks
        _case("dispatch_wide", "dispatch", "bf16", "swiglu", 32768, 256, 256, 256, 8, 32, 10),
        # two of eight ranks are lost: new plan, 48 slots filled from the survivors
        _case("replan_c5", "replan", "bf16", "gelu", 16384, 2048, 8192, 32, 2, 8, 6, 1.2, 2),
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer multiple of `step` in [lo, hi], uniform over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, int(round(v / step)) * step)


def draw(rng):
    """A case of the same ranges: every operation, both types and activations, sizes over their logarithm."""
    while True:
        op = rng.choices(["forward", "forward_fused", "train", "accumulate", "dispatch", "replan"], [6, 3, 6, 2, 2, 1])[0]
        dtype = "bf16" if op in ("dispatch", "replan") or rng.random() < 0.85 else "f32"
        act = rng.choice(["gelu", "swiglu"])
        # widths: mostly multiples of 256 and 64, sometimes only of 8 (fp32: of anything)
        step = rng.choices([256, 64, 8], [6, 2, 2])[0] if dtype == "bf16" else rng.choices([64, 8, 1], [4, 3, 3])[0]
        d = _log_int(rng, 256, 4096, step) if dtype == "bf16" else _log_int(rng, 64, 1024, step)
        ffn = _log_int(rng, max(128, d // 2), 4 * d, 64 if step == 256 and rng.random() < 0.4 else step)
        E = _log_int(rng, 4, 64)
        k = rng.randint(1, min(E, 8))
        N = rng.randint(2, 16)
        c = -(-E // N) + rng.randint(0, 4)
        T = _log_int(rng, 32, 32768)
        lost = 0
        if op == "dispatch":
            T, E, N = _log_int(rng, 256, 65536), _log_int(rng, 8, 256), rng.randint(2, 64)
            k = rng.randint(1, 8)
            d = ffn = 256
            c = -(-E // N) + rng.randint(0, 4)
        if op == "replan":
            N, lost = rng.randint(4, 12), 1
            c = -(-2 * E // N) + rng.randint(0, 3)
        if c > 64:
            continue
        case = _case(None, op, dtype, act, T, d, ffn, E, k, N, c, round(rng.uniform(0.0, 1.3), 2), lost)
        # no dearer than the largest listed case: its flops and weights, less where fp32 gradients are
        # accumulated, much less in fp32 and at widths that are not multiples of 64
        slot_params = N * c * _params(case)
        most_flops = 17e12 if dtype == "bf16" and d % 256 == 0 and ffn % 64 == 0 else 1.0e11
        most_params = {"accumulate": 1.1e9, "train": 2.0e9, "replan": 1.6e9}.get(op, 2.8e9)
        if op == "dispatch" or (work(case)["flops"] <= most_flops and slot_params <= most_params):
            return case


def _params(case):
    return case["d"] * case["ffn"] * (3 if case["act"] == "swiglu" else 2)


def work(case):
    T, d, E, k, N, c = (case[n] for n in ("T", "d", "E", "k", "N", "c"))
    b = 4 if case["dtype"] == "f32" else 2
    S, P, params = N * c, T * k, _params(case)
    used = min(S, P)  # slots that can have rows
    route = T * E * 4 + P * 8
    if case["op"] == "dispatch":
        return {"bytes": route + P * 8 + S * 12 + E * N * 4 + E * N * N * 4, "flops": 0}
    if case["op"] == "replan":  # each expert read once, every new slot written once
        return {"bytes": (E + _new_slots(case)) * params * b, "flops": 0}
    if case["op"] in ("forward", "forward_fused"):
        return {"bytes": route + 2 * T * d * b + used * params * b, "flops": 2 * P * params}
    batch = route + T * E * 4 + 4 * T * d * b  # logits and their gradient; x, dy read, y, dx written
    if case["op"] == "train":
        return {"bytes": batch + used * params * b + E * params * b, "flops": 6 * P * params}
    # accumulators of every slot and their sum over replicas, both fp32
    return {"bytes": 2 * batch + used * params * b + (S + E) * params * 4, "flops": 12 * P * params}


def tolerance(case):
    """Against the same operations in fp64 (all listed operations, reduced and odd sizes): fp32 rel 0.4e-6 to
    1.3e-6, largest difference 9e-6; bf16, which stores z, h, yp and their gradients between the
    GEMMs, rel 0.003 to 0.0042, largest difference 0.058 (weight gradients)."""
    if case["op"] in ("replan", "dispatch"):
        return {"rel": 1e-6}  # indices and copied bytes are exact; the fp32 gates are a few exponentials
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.2}


# ------------------------------------------------------------------------------------------ state
def _new_c(case):
    return -(-case["N"] * case["c"] // (case["N"] - case["lost"]))


def _new_slots(case):
    return (case["N"] - case["lost"]) * _new_c(case)


def _bias(case, gen):
    ranking = torch.randperm(case["E"], generator=gen, device=DEV).float()
    return -case["zipf"] * torch.log(ranking + 1.0)


def _logits(case, gen, bias):
    return torch.randn((case["T"], case["E"]), generator=gen, device=DEV) + bias


def _loads(case, logits):
    """Tokens per expert of a batch."""
    T, E, k = case["T"], case["E"], case["k"]
    ids = torch.empty((T, k), dtype=torch.int32, device=DEV)
    gates = torch.empty((T, k), dtype=torch.float32, device=DEV)
    lz.lz_route(logits, T, E, k, ids, gates)
    return torch.bincount(ids.reshape(-1), minlength=E).cpu().numpy().astype(np.int64)


def _normal(gen, shape, dtype, std=1.0):
    return torch.randn(shape, generator=gen, device=DEV).mul_(std).to(dtype)


def _slot_weights(case, gen, slot_expert):
    """w1 [S, d, n1], w2 [S, ffn, d]: every slot its own copy of its expert's weights."""
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    d, ffn, S = case["d"], case["ffn"], len(slot_expert)
    n1 = ffn * (2 if case["act"] == "swiglu" else 1)
    w1 = torch.empty((S, d, n1), dtype=dtype, device=DEV)
    w2 = torch.empty((S, ffn, d), dtype=dtype, device=DEV)
    for e in range(case["E"]):
        a, b = _normal(gen, (d, n1), dtype, WEIGHT_STD), _normal(gen, (ffn, d), dtype, WEIGHT_STD)
        for s in np.flatnonzero(np.asarray(slot_expert) == e):
            w1[s].copy_(a)
            w2[s].copy_(b)
    return w1, w2


def _prepare_replan(case, gen, shape):
    N, c, lost = case["N"], case["c"], case["lost"]
    bias = _bias(case, gen)
    before, now = (_loads(case, _logits(case, gen, bias)) for _ in range(2))
    f = 2 if N * c >= 2 * case["E"] else 1
    plan = lz.lz_place_mro(lz.lz_allocate_replicas(before, N, c, f), before, N, c)
    # the ranks that are lost: the last set that leaves every expert a replica
    for dead in itertools.combinations(range(N - 1, -1, -1), lost):
        alive = np.ones(N, dtype=np.uint8)
        alive[list(dead)] = 0
        if set(plan.reshape(N, c)[alive == 1].reshape(-1).tolist()) == set(range(case["E"])):
            break
    w1, w2 = _slot_weights(case, gen, plan)
    S_new = _new_slots(case)
    return dict(case=case, shape=shape, plan=plan, alive=alive, loads=now, w1=w1, w2=w2, c_new=_new_c(case),
                w1_new=torch.empty((S_new, *w1.shape[1:]), dtype=w1.dtype, device=DEV),
                w2_new=torch.empty((S_new, *w2.shape[1:]), dtype=w2.dtype, device=DEV))


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    N, c, T = case["N"], case["c"], case["T"]
    shape = lz.Shape(T, case["d"], case["ffn"], case["E"], case["k"], N, c,
                     lz.LZ_F32 if case["dtype"] == "f32" else lz.LZ_BF16,
                     lz.LZ_GELU if case["act"] == "gelu" else lz.LZ_SWIGLU)
    if case["op"] == "replan":
        return _prepare_replan(case, gen, shape)
    bias = _bias(case, gen)
    history = _loads(case, _logits(case, gen, bias))
    plan = lz.lz_place_mro(lz.lz_allocate_replicas(history, N, c, 1), history, N, c)
    layer = lz.MoELayer(shape, DEV)
    layer.set_plan(plan, np.array([(i * T) // N for i in range(N + 1)], dtype=np.int32))
    state = dict(case=case, layer=layer)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    if case["op"] != "dispatch":
        layer.set_slot_weights(*_slot_weights(case, gen, plan))
    batches = 2 if case["op"] == "accumulate" else 1
    state["logits"] = [_logits(case, gen, bias) for _ in range(batches)]
    if case["op"] != "dispatch":
        state["x"] = [_normal(gen, (T, case["d"]), dtype) for _ in range(batches)]
    if case["op"] in ("train", "accumulate"):
        state["dy"] = [_normal(gen, (T, case["d"]), dtype) for _ in range(batches)]
        layer.enable_training()
    if case["op"] == "accumulate":
        layer.enable_accumulation()
    return state


def run(state):
    op = state["case"]["op"]
    if op == "replan":
        r = lz.lz_replan(state["plan"], state["case"]["N"], state["case"]["c"], state["alive"], state["loads"],
                         state["c_new"], 1)
        lz.lz_apply_transfers(r["transfers"], state["w1"], state["w2"], len(state["plan"]), state["w1_new"],
                              state["w2_new"], len(r["new_slot_expert"]), state["shape"])
        return {"plan": r["new_slot_expert"], "nodes": r["plan2phys"], "w1": state["w1_new"], "w2": state["w2_new"]}
    layer = state["layer"]
    if op == "dispatch":
        layer.route(state["logits"][0])
        layer.plan_dispatch()
        return {n: getattr(layer, n) for n in ("topk_ids", "topk_gates", "slot_counts", "slot_offsets", "pair_to_row",
                                               "row_to_pair", "Tej", "D", "status")}
    if op == "forward":
        y = layer.forward(state["logits"][0], state["x"][0])
        return {"y": y, "ids": layer.topk_ids, "gates": layer.topk_gates}
    if op == "forward_fused":
        y = layer.forward_fused(state["logits"][0], state["x"][0])
        return {"y": y, "ids": layer.topk_ids, "gates": layer.topk_gates}
    if op == "train":
        y = layer.forward_train(state["logits"][0], state["x"][0])
        dx = layer.backward(state["dy"][0])
        return {"y": y, "dx": dx, "dlogits": layer.dlogits, "dw1": layer.dw1, "dw2": layer.dw2}
    layer.dw1_acc.zero_()
    layer.dw2_acc.zero_()
    for logits, x, dy in zip(state["logits"], state["x"], state["dy"]):
        y = layer.forward_train(logits, x)
        dx = layer.backward_accumulate(dy)
    dw1, dw2 = layer.reduce_accumulated()
    return {"y": y, "dx": dx, "dlogits": layer.dlogits, "dw1": dw1, "dw2": dw2, "dw1_slots": layer.dw1_acc,
            "dw2_slots": layer.dw2_acc}
