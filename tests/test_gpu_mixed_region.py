"""Regions of siblings of unlike kinds in one launch: depthwise and separable convolutions of every filter size, window pools and 1x1 convolutions over one tensor, where a kind's tiles, waves and
remainders can go wrong beside the others.  Against the oracle; the kinds that run unchanged (all but 1x1 convolutions) bit for bit as one by one."""
import numpy as np
import pytest
import torch

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg
from paper_2111_00655_amd import binding as B
from oracle.graph import Graph
from parity_util import OP_TOL, check_outputs, norm_err

pytestmark = pytest.mark.gpu

TAILS = [(), ("bias_add",), ("bias_add", "add"), ("bias_add", "relu")]
CASES = [
    # batch, channels, height, width, branches: (kind, filter, stride, relu in front, output channels, tail)
    # one and two 16-pixel tiles per problem; channels that are not a multiple of four (the any-filter path), a wave per tile
    (1, 11, 5, 5, [("dw", 3, 1, True, 0, ()), ("max", 3, 1, False, 0, ()), ("conv", 1, 1, False, 11, ("bias_add",)), ("sep", 3, 1, True, 11, ("bias_add",)),
                   ("conv", 1, 2, False, 7, ("bias_add", "add"))]),
    # every depthwise and separable filter size, four and eight waves, an odd number of pixel tiles, two images
    (2, 44, 9, 11, [("dw", 7, 1, True, 0, ("bias_add",)), ("sep", 5, 1, True, 44, ("bias_add", "add")), ("sep", 7, 1, False, 20, ("bias_add",)), ("conv", 1, 1, True, 33, ("bias_add",)),
                    ("avg", 3, 2, False, 0, ("add",)), ("dw", 5, 2, False, 0, ()), ("sep", 3, 2, True, 50, ())]),
    # two, four and eight waves per tile of 1x1 convolutions (two to more than eight chunks), with and without a relu, without wide kinds
    (1, 88, 14, 13, [("conv", 1, 1, False, 88, ("bias_add",)), ("conv", 1, 1, True, 90, ("bias_add", "add")), ("max", 3, 1, False, 0, ("add",)), ("sep", 3, 1, True, 88, ("bias_add",))]),
    (3, 176, 7, 7, [("conv", 1, 1, False, 176, ("bias_add", "relu")), ("conv", 1, 2, True, 16, ("bias_add",)), ("dw", 3, 1, True, 0, ("bias_add", "add")), ("avg", 3, 1, False, 0, ())]),
    (1, 600, 6, 4, [("conv", 1, 1, False, 40, ("bias_add",)), ("conv", 1, 1, True, 24, ()), ("dw", 5, 1, True, 0, ()), ("max", 2, 2, False, 0, ())]),
    # long any-filter channel ranges; more branches than a region holds
    (1, 90, 8, 8, [("conv", 1, 1, False, 18, ("bias_add",)), ("dw", 3, 1, False, 0, ()), ("dw", 7, 2, True, 0, ()), ("sep", 5, 2, True, 90, ("bias_add",)), ("avg", 5, 1, False, 0, ()),
                   ("max", 3, 1, False, 0, ()), ("sep", 3, 1, False, 16, ()), ("conv", 1, 2, False, 90, ()), ("dw", 5, 1, False, 0, ("bias_add",)), ("conv", 1, 1, False, 5, ())]),
]


@pytest.mark.parametrize("ci", range(len(CASES)))
def test_region_of_siblings_of_unlike_kinds(ci):
    n_img, c, h, w, branches = CASES[ci]
    r = np.random.default_rng([91, ci])
    f32 = lambda *shape, scale=1.0: (r.standard_normal(shape) * scale).astype(np.float32)
    d = wl.GraphDesc("region_mixed")
    x = d.input(f32(n_img, c, h, w))
    for kind, k, stride, pre, cout, tail in branches:
        pad, ho, wo = (k - 1) // 2, (h + 2 * ((k - 1) // 2) - k) // stride + 1, (w + 2 * ((k - 1) // 2) - k) // stride + 1
        cout = cout or c
        y = d.op("relu", [x]) if pre else x
        if kind in ("dw", "sep"):
            y = d.op("conv2d", [y, d.const(f32(c, 1, k, k, scale=1.0 / k))], stride=(stride, stride), pad=(pad, pad), groups=c)
        if kind in ("sep", "conv"):
            s1 = stride if kind == "conv" else 1
            y = d.op("conv2d", [y, d.const(f32(cout, c, 1, 1, scale=c ** -0.5))], stride=(s1, s1), pad=(0, 0), groups=1)
        if kind in ("max", "avg"):
            y = d.op(kind + "_pool2d", [x], kernel=(k, k), stride=(stride, stride), pad=(pad, pad))
        for op in tail:
            operand = [d.const(f32(cout))] if op == "bias_add" else ([d.input(f32(n_img, cout, ho, wo))] if op == "add" else [])
            y = d.op(op, [y] + operand, **({"axis": 1} if op == "bias_add" else {}))
        d.mark_output(y)

    def tails(anchor):
        out = []
        for t in TAILS:
            p = anchor
            for op in t:
                p = P(op, p, W) if op in ("bias_add", "add") else P(op, p)
            out.append(p)
        return out
    dw = P("conv2d", P("relu", W), W)
    reg = [("sepconv", p) for a in (P("conv2d", dw, W), P("conv2d", P("conv2d", W, W), W), dw) for p in tails(a)]
    reg += [("direct", p) for p in tails(P("conv2d", W, W, groups=(c, c)))] + [("igemm_r16", p) for p in tails(P("conv2d", W, W, groups=(1, 1)))]
    reg += [("direct", p) for k in ("avg_pool2d", "max_pool2d") for p in (P(k, W), P("add", P(k, W), W))]
    reg += [("eltwise", P("relu", W)), ("eltwise", P("add", W, W)), ("eltwise", P("bias_add", W, W))]
    s = clg.Session(d, reg, device=0)
    ms = s.match()
    _, ids = s.search([100] * len(ms), 0)                   # fewest kernels: every branch is one
    plan = s.compile(ids).bind()
    n, regions = plan.n_kernels, plan.regions()
    names = [k["name"] for k in plan.kernels()]
    assert n == len(branches), names
    assert sum(g == 0 for g in regions) == min(n, 8), (regions, names)
    ref = Graph(d).run()
    one_by_one = plan.run()
    check_outputs(one_by_one, ref, OP_TOL, (ci, "one by one"))
    for digits in ([1] * n, [i % 2 for i in range(n)], [1, 1] + [0] * (n - 2), [0] * (n - 2) + [1, 1], [1] * n):
        plan.set_handover(digits, lanes=1)
        saved = sum(max(sum(dg for dg, g in zip(digits, regions) if g == q) - 1, 0) for q in range(max(regions) + 1))
        assert plan.n_launches == n - saved, (digits, regions, plan.n_launches)
        got = plan.run()
        check_outputs(got, ref, OP_TOL, (ci, digits))
        for k, (a, b) in enumerate(zip(got, one_by_one)):
            assert branches[k][0] == "conv" or np.array_equal(a, b), (ci, digits, branches[k])
    s.close()


# 1x1 convolutions of grouped channels (whole tiles, several groups per tile, groups that take the any-filter path) and with padding, beside pools
def test_grouped_and_padded_convolutions_in_a_region_of_unlike_kinds():
    r = np.random.default_rng(17)
    f32 = lambda *shape: r.standard_normal(shape).astype(np.float32)
    c, d = 48, wl.GraphDesc("region_grouped")
    x = d.input(f32(2, c, 9, 7))
    for cout, groups, stride, pad in ((48, 3, 1, 0), (48, 12, 2, 0), (32, 16, 1, 0), (20, 1, 2, 1), (96, 3, 1, 1)):
        y = d.op("conv2d", [x, d.const(f32(cout, c // groups, 1, 1))], stride=(stride, stride), pad=(pad, pad), groups=groups)
        d.mark_output(d.op("bias_add", [y, d.const(f32(cout))], axis=1))
    d.mark_output(d.op("max_pool2d", [x], kernel=(3, 3), stride=(1, 1), pad=(1, 1)))
    d.mark_output(d.op("avg_pool2d", [x], kernel=(3, 3), stride=(2, 2), pad=(1, 1)))
    s = clg.Session(d, [("igemm_r16", P("bias_add", P("conv2d", W, W), W)), ("direct", P("max_pool2d", W)), ("direct", P("avg_pool2d", W))], device=0)
    plan = s.compile(list(range(len(s.match())))).bind()
    assert plan.regions() == [0] * 7
    ref = Graph(d).run()
    one_by_one = plan.run()
    check_outputs(one_by_one, ref, OP_TOL, "one by one")
    plan.set_handover([1] * 7, lanes=1)
    assert plan.n_launches == 1
    got = plan.run()
    check_outputs(got, ref, OP_TOL, "one launch")
    assert all(np.array_equal(a, b) for a, b in zip(got[5:], one_by_one[5:]))
    s.close()


# in the order of their levels, with and without digits, on several streams: the kernels of the sequence, bit for bit
def test_order_by_level_on_several_lanes():
    d = wl.nasnet_a(0, image=48, stem=8, filters=8, cells=1, classes=5, batch=2)
    s = clg.Session(d, wl.default_registry(("igemm_r16",), sepconv=True), device=0)
    plan = s.compile(s.search([1] * len(s.match()), 0)[1]).bind()
    n = plan.n_kernels
    want = plan.run()
    assert max(norm_err(a, b) for a, b in zip(want, Graph(d).run())) <= 1e-3
    for lanes, digits in ((2, [1] * n), (4, [1] * n), (4, [i % 2 for i in range(n)]), (3, [int(i % 3 > 0) for i in range(n)])):
        plan.set_handover(digits, lanes=lanes)
        assert plan.n_launches >= n - sum(k["name"].endswith("_alias") for k in plan.kernels()) - 2, "regions share launches on one lane only"
        for _ in range(3):
            assert all(np.array_equal(a, b) for a, b in zip(plan.run(), want)), (lanes, digits)
    plan.set_lanes(4)
    assert all(np.array_equal(a, b) for a, b in zip(plan.run(), want))
    s.close()


@pytest.mark.parametrize("missing", ["weights", "bias"])
def test_a_constant_without_device_memory_is_refused_in_a_region_too(missing):
    """Depthwise convolutions and a pool over one tensor: the members of a region are checked as kernels launched one by one are, and so are the operands of
    fused tails (host-side checks: nothing is launched)."""
    r = np.random.default_rng(5)
    d = wl.GraphDesc("no_memory")
    x = d.input(r.standard_normal((1, 8, 6, 6)).astype(np.float32))
    w, b = d.const(r.standard_normal((8, 1, 3, 3)).astype(np.float32)), d.const(r.standard_normal(8).astype(np.float32))
    d.mark_output(d.op("bias_add", [d.op("conv2d", [x, w], stride=(1, 1), pad=(1, 1), groups=8), b], axis=1))
    d.mark_output(d.op("max_pool2d", [x], kernel=(3, 3), stride=(1, 1), pad=(1, 1)))
    reg = [("direct", P("bias_add", P("conv2d", W, W), W)), ("direct", P("max_pool2d", W))]
    ctx = B.clg_create(0)
    g = B.clg_graph_create(ctx)
    for be, pat in reg:
        B.clg_register_pattern(ctx, B.clg_register_backend(ctx, be), pat)
    keep = {n: torch.from_numpy(t).to("cuda:0") for n, t in d.tensors.items() if n in (w, b)}
    for n, nd in enumerate(d.nodes):
        if nd["kind"] == "input":
            B.clg_graph_input(g, B.F32, nd["shape"])
        elif nd["kind"] == "const":
            B.clg_graph_const(g, B.F32, d.tensors[n].shape, 0 if n == (w if missing == "weights" else b) else keep[n].data_ptr())
        else:
            B.clg_graph_op(g, nd["kind"], nd["inputs"], B.make_attrs(**nd["attrs"]))
    for o in d.outputs:
        B.clg_graph_mark_output(g, o)
    plan = B.clg_compile(ctx, g, list(range(len(B.clg_match_all(ctx, g)))))
    xs = torch.zeros(1, 8, 6, 6, device="cuda:0")
    outs = [torch.zeros(1, 8, 6, 6, device="cuda:0") for _ in d.outputs]
    for digits in ([0, 0], [1, 1]):
        B.clg_plan_set_handover(plan, digits, 1)
        assert B.clg_plan_num_launches(plan) == 2 - digits[0]
        with pytest.raises(clg.ClgError, match="device pointer") as e:
            B.clg_execute(plan, [xs.data_ptr()], [t.data_ptr() for t in outs], 0, 0, torch.cuda.current_stream().cuda_stream)
        assert e.value.status == "INVALID_ARG"
    B.clg_plan_destroy(plan)
    B.clg_graph_destroy(g)
    B.clg_destroy(ctx)
