"""Performance cases: what users of the library run, at the sizes they run it.

A network is optimised once (match, measure every candidate kernel, op-level
search, compile, graph-level search: the steps of bench.py) and then executed
for input after input, so an optimised network is built once per process and
shared by all inputs made for it, as in a serving program: weights and plan
stay, inputs and outputs change.  One pass is one clg_execute.  The other kind
of case is the placement search itself (match enumeration and dynamic
programme), which runs on the host.
"""
import functools
import math

import numpy as np
import torch

import paper_2111_00655_amd as clg
import workloads as wl
from paper_2111_00655_amd import binding as B

# the kernel-variant backends the benchmark registers
VARIANTS = ("igemm", "igemm_s", "igemm_s8", "igemm_s16", "igemm_m", "igemm_l", "igemm_s_nk", "igemm_s8_nk",
            "igemm_s16_nk", "igemm_r32", "igemm_r16", "igemm_r32_w4", "igemm_r32_w8", "igemm_r16_w4", "igemm_r16_w8",
            "igemm_r16x2_w4", "igemm_r16x2_w8", "igemm_r16_sk", "igemm_r16_sk_w4", "igemm_r32_sk")


def listed():
    return [
        # the smallest network: latency and launches only
        {"name": "tiny_cnn", "model": "tiny_cnn", "image": 32},
        # image generation, one sample (weight-bound) and a batch (compute-bound)
        {"name": "dcgan b1", "model": "dcgan", "batch": 1},
        {"name": "dcgan b64", "model": "dcgan", "batch": 64},
        # image classification, one image at a time: the headline workload
        {"name": "resnet50 b1", "model": "resnet50", "batch": 1, "image": 224},
        # a few images of a size nothing is aligned to
        {"name": "resnet50 b5 197", "model": "resnet50", "batch": 5, "image": 197},
        # grouped convolutions, one image and the largest batch of the batch sweep
        {"name": "resnext50 b1", "model": "resnext50", "batch": 1, "image": 224},
        {"name": "resnext50 b32", "model": "resnext50", "batch": 32, "image": 224},
        # transformer encoder: the usual sequence, and a long ragged one
        {"name": "bert_base s128", "model": "bert_base", "seq": 128},
        {"name": "bert_base s389", "model": "bert_base", "seq": 389},
        # many small kernels: separable convolutions and pools
        {"name": "nasnet_a b1", "model": "nasnet_a", "batch": 1, "image": 224},
        # video clip: 3-D convolutions
        {"name": "resnet3d_50", "model": "resnet3d_50", "batch": 1, "frames": 16, "image": 112},
        # the placement search of the network with the most operators, on the host (separable convolutions operator by
        # operator, the registry's default)
        {"name": "placement nasnet_a", "task": "placement", "model": "nasnet_a", "cells": 4, "filters": 44},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("tiny_cnn", "dcgan", "resnet50", "resnext50", "bert_base", "nasnet_a", "resnet3d_50", "placement"))
    if kind == "tiny_cnn":
        return {"model": kind, "image": rng.randint(16, 96)}
    if kind == "dcgan":
        return {"model": kind, "batch": _log_int(rng, 2, 256)}
    if kind in ("resnet50", "resnext50"):
        image = rng.randint(96, 256)
        return {"model": kind, "batch": _log_int(rng, 1, min(32, 32 * 224 * 224 // (image * image))), "image": image}
    if kind == "bert_base":
        return {"model": kind, "seq": _log_int(rng, 16, 512)}
    if kind == "nasnet_a":
        return {"model": kind, "batch": _log_int(rng, 1, 4), "image": rng.randint(96, 256)}
    if kind == "resnet3d_50":
        return {"model": kind, "batch": rng.randint(1, 2), "frames": rng.randint(8, 24), "image": rng.randint(64, 128)}
    if rng.random() < 0.5:
        return {"task": "placement", "model": "bert_base", "layers": rng.randint(1, 12), "seq": _log_int(rng, 16, 512)}
    return {"task": "placement", "model": "nasnet_a", "cells": rng.randint(1, 4), "filters": 4 * rng.randint(6, 16)}


def _describe(case):
    """The network as a graph description (seeded weights; the inputs in it only give the shapes)."""
    sizes = {k: v for k, v in case.items() if k not in ("name", "task", "model")}
    desc = {"tiny_cnn": wl.tiny_cnn, "dcgan": wl.dcgan, "resnet50": wl.resnet50, "resnext50": wl.resnext50,
            "bert_base": wl.bert_base, "nasnet_a": wl.nasnet_a, "resnet3d_50": wl.resnet3d_50}[case["model"]](0, **sizes)
    # random weights make logits of thousands and a softmax that is one-hot; a trained classifier's are of order ten
    gain = {"resnet50": 1e-3, "resnext50": 1e-3, "nasnet_a": 1e-4, "resnet3d_50": 1e-2}.get(case["model"])
    for n, nd in enumerate(desc.nodes):
        if gain and nd["name"] == "fc.w":
            desc.tensors[n] = (desc.tensors[n] * gain).astype(np.float32)
    return desc


def _key(case):
    return tuple(sorted((k, v) for k, v in case.items() if k != "name"))


def _registry(sepconv):
    return wl.default_registry(VARIANTS, sepconv=sepconv, attention=True)


@functools.lru_cache(maxsize=None)
def _network(key):
    """The optimised network: session, compiled plan under the placement found for it, and one workspace."""
    s = clg.Session(_describe(dict(key)), _registry(True), device=0)
    s.match()
    total, ids = s.search(s.profile(B.ProfileOpts(warmup=3, batches=3, min_batch_us=200, max_launches=500)), 0)
    plan = s.compile(ids).bind()
    # graph level: which sibling kernels share a launch, priced by timing the sequence (fewer repeats of a long one)
    rand = np.random.default_rng(0).integers(0, 2 ** 32, 1 << 17, dtype=np.uint64).tolist()
    plan.search_graph_level(B.make_es_opts(population=12, generations=12, tournament=3, patience=5, p_init=0.5, p_mutate=0.5,
                                           p_flip=0.1, p_cross=0.5, seed_ones=True),
                            rand, lanes=1, warmup=3, batches=3, reps=max(4, min(20, int(20e6 / total))))
    ws = torch.empty(max(plan.ws_bytes, 256), dtype=torch.uint8, device="cuda:0")
    return s, plan, ws


@functools.lru_cache(maxsize=None)
def _host_session(key):
    """A host-only session for the placement search, and the number of its matches."""
    s = clg.Session(_describe(dict(key)), _registry(False), device=None)
    return s, len(s.match())


def prepare(case, seed):
    key = _key(case)
    if case.get("task") == "placement":
        s, n = _host_session(key)
        costs = np.random.default_rng(seed).integers(2000, 20000, n)         # measured nanoseconds of a cost log
        return {"session": s, "costs": costs}
    s, plan, ws = _network(key)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    inputs = []
    for n in s.input_nodes:
        nd = s.desc.nodes[n]
        if nd["dtype"] == "int32":                                           # token ids
            inputs.append(torch.randint(0, 30522, nd["shape"], generator=gen, device="cuda:0", dtype=torch.int32))
        else:
            inputs.append(torch.randn(nd["shape"], generator=gen, device="cuda:0"))
    outputs = [torch.empty(shape, device="cuda:0") for shape in s.out_shapes]
    return {"plan": plan, "inputs": inputs, "outputs": outputs, "workspace": ws}


def run(state):
    if "session" in state:
        s = state["session"]
        s.match()
        total, ids = s.search(state["costs"], 0)
        chosen = np.full(len(s.desc.op_nodes()), -1, np.int64)               # a placement has at most one match per operator
        chosen[:len(ids)] = ids
        return [np.array([total], np.int64), chosen]
    ws = state["workspace"]
    B.clg_execute(state["plan"].h, [t.data_ptr() for t in state["inputs"]], [t.data_ptr() for t in state["outputs"]],
                  ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    return state["outputs"]


@functools.lru_cache(maxsize=None)
def _work(key):
    """Inputs, weights (table rows that are gathered) and outputs once; two flops per multiply-add of the contractions."""
    desc = _describe(dict(key))
    s = clg.Session(desc, [], device=None)
    shape = [B.clg_graph_node_shape(s.graph, n)[1] for n in range(len(desc))]
    size = [math.prod(sh) for sh in shape]
    tables = {nd["inputs"][0] for nd in desc.nodes if nd["kind"] == "take"}
    values = sum(size[n] for n in desc.outputs)
    values += sum(size[n] for n, nd in enumerate(desc.nodes) if nd["kind"] in ("input", "const") and n not in tables)
    flops = 0
    for n, nd in enumerate(desc.nodes):
        if nd["kind"] == "take":
            values += size[n]
        elif nd["kind"] in ("conv2d", "conv3d", "dense"):
            flops += 2 * size[n] * math.prod(shape[nd["inputs"][1]][1:])
        elif nd["kind"] == "conv2d_transpose":
            flops += 2 * size[nd["inputs"][0]] * math.prod(shape[nd["inputs"][1]][1:])
        elif nd["kind"] == "batch_matmul":
            flops += 2 * size[n] * shape[nd["inputs"][0]][-1]
    ops = len(desc.op_nodes())
    s.close()
    return 4 * values, flops, ops


def work(case):
    nbytes, flops, ops = _work(_key(case))
    if case.get("task") == "placement":
        # a cost per match and backend variant of each operator read, a match id per operator written
        return {"bytes": 8 * ops * len(VARIANTS) + 4 * ops, "flops": ops * len(VARIANTS)}
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case.get("task") == "placement":
        return "exact"
    return {"rel": 1e-5}       # 32-bit sums of up to 13824 terms, in another order in every kernel variant
