"""Kernels that share launches with what reads them: [global average pool,] dense layer and softmax in one, and a dense layer with K split whose partial
results the layer norm behind it adds up."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg
from paper_2111_00655_amd import binding as B

pytestmark = pytest.mark.gpu


def timed(plan):
    """Outputs of an execution that times its kernels."""
    ns = np.asarray(plan.execute_timed())
    torch.cuda.synchronize()
    assert (ns > 0).all()                                    # one by one
    return [t.cpu().numpy() for t in plan._out]


def launches(plan):
    """Kernels that one execution launches, counted in a graph that it is captured into."""
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64.so" in line))
    plan.execute()                                           # (what a first call sets up)
    torch.cuda.synchronize()
    g, st, n = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream(), ctypes.c_size_t()
    with torch.cuda.stream(st), torch.cuda.graph(g, stream=st):
        plan.execute()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def same_on_two_lanes(plan, got):
    plan.set_lanes(2)
    assert all(np.array_equal(a, b) for a, b in zip(plan.run(), got))
    n = plan.n_kernels
    for digits in ([0] + [1] * (n - 1), [1] * (n - 1) + [0]):
        plan.set_handover(digits, lanes=2)
        assert all(np.array_equal(a, b) for a, b in zip(plan.run(), got))


# classes and channels at the ends of what the kernel takes, images of all remainders of four and eight loads, weights as they lie and in both packed orders
@pytest.mark.parametrize("backend", ["igemm_s8", "igemm_r16", "igemm_r32", "igemm_r16x2_w4"])
@pytest.mark.parametrize("n,c,h,w,classes", [(1, 32, 32, 32, 10), (3, 16, 7, 9, 64), (2, 256, 2, 3, 8), (1, 48, 1, 1, 1), (5, 128, 4, 6, 33), (2, 130, 9, 9, 63), (1, 3, 130, 130, 5)])
def test_classifier(n, c, h, w, classes, backend):
    r = np.random.default_rng(n * c + h)
    xv, wv, bv = r.standard_normal((n, c, h, w)).astype(np.float32) + 1, r.standard_normal((classes, c)).astype(np.float32), r.standard_normal(classes).astype(np.float32)
    d = wl.GraphDesc("classifier")
    y = d.op("dense", [d.op("global_avg_pool2d", [d.input(xv)]), d.const(wv)])
    logits = d.op("bias_add", [y, d.const(bv)], axis=-1)
    d.mark_output(logits)
    d.mark_output(d.op("softmax", [logits]))
    s = clg.Session(d, [("direct", P("global_avg_pool2d", W)), (backend, P("bias_add", P("dense", W, W), W)), ("rowwise", P("softmax", W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    assert plan.n_kernels == 3 and plan.n_launches == 1
    p = xv.astype(np.float64).mean((2, 3))
    want = p @ wv.T.astype(np.float64) + bv
    # means of up to 17000 values, added 8 ways and over the lanes (60 terms in a chain at most), then products of 256 terms, 16 in a chain
    bound = 140 * 2.0 ** -24 * (np.abs(xv).astype(np.float64).mean((2, 3)) @ np.abs(wv).T.astype(np.float64) + np.abs(bv))
    e = np.exp(want - want.max(-1, keepdims=True))
    prob = e / e.sum(-1, keepdims=True)
    got = plan.run()
    for y in (got, timed(plan)):
        assert (np.abs(y[0] - want) <= bound).all()
        assert (np.abs(y[1] - prob) <= prob * (4 * bound.max(-1, keepdims=True) + 80 * 2.0 ** -24)).all()
    same_on_two_lanes(plan, got)
    s.close()


def test_classifier_without_a_pool_and_with_outputs_over_its_input():
    r = np.random.default_rng(2)
    xv, wv = r.standard_normal((6, 20)).astype(np.float32), r.standard_normal((20, 20)).astype(np.float32)
    d = wl.GraphDesc("dense_softmax")
    d.mark_output(d.op("softmax", [d.op("dense", [d.input(xv), d.const(wv)])]))
    s = clg.Session(d, [("igemm_s", P("dense", W, W)), ("rowwise", P("softmax", W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    assert plan.n_launches == 1
    e = np.exp(xv.astype(np.float64) @ wv.T.astype(np.float64))
    want = e / e.sum(-1, keepdims=True)
    assert np.allclose(plan.run()[0], want, rtol=1e-5, atol=0)
    plan._in[0].copy_(torch.from_numpy(xv))
    plan._out[0] = plan._in[0]                               # the softmax of all rows over the input: the kernels run one by one
    plan.execute()
    torch.cuda.synchronize()
    assert np.allclose(plan._out[0].cpu().numpy(), want, rtol=1e-5, atol=0)
    s.close()


def test_what_is_no_small_classifier():
    for classes, c, hw in ((65, 16, 4), (10, 260, 4), (10, 32, 2052)):
        d = wl.GraphDesc("large")
        y = d.op("dense", [d.op("global_avg_pool2d", [d.input(np.ones((1, c, hw, 1), np.float32))]), d.const(np.ones((classes, c), np.float32))])
        d.mark_output(d.op("softmax", [y]))
        s = clg.Session(d, [("direct", P("global_avg_pool2d", W)), ("igemm_s8", P("dense", W, W)), ("rowwise", P("softmax", W))], device=0)
        plan = s.compile(list(range(len(s.match()))))
        assert plan.n_launches == (2 if hw == 2052 else 3), (classes, c, hw)
        assert np.allclose(plan.run()[0], 1 / classes, rtol=1e-5, atol=0)
        s.close()


# both sides of the row counts up to which a workgroup per row pays: compute units, twice as many with a pool of 32 channels and more
@pytest.mark.parametrize("c,hw,rows,joined", [(40, 0, 1, 1), (40, 0, 0, 2), (40, 5, 1, 1), (40, 5, 2, 1), (40, 5, 3, 3), (31, 5, 1, 1), (31, 5, 0, 3)])
def test_classifier_rows(c, hw, rows, joined):
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    m = {0: n_cus + 1, 1: n_cus, 2: 2 * n_cus, 3: 2 * n_cus + 1}[rows]
    r = np.random.default_rng(m)
    xv, wv = r.standard_normal((m, c, hw, 1) if hw else (m, c)).astype(np.float32), r.standard_normal((10, c)).astype(np.float32)
    d = wl.GraphDesc("classifier_rows")
    x = d.input(xv)
    d.mark_output(d.op("softmax", [d.op("dense", [d.op("global_avg_pool2d", [x]) if hw else x, d.const(wv)])]))
    s = clg.Session(d, [("direct", P("global_avg_pool2d", W)), ("igemm_s8", P("dense", W, W)), ("rowwise", P("softmax", W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    assert plan.n_launches == joined
    e = np.exp((xv.astype(np.float64).mean((2, 3)) if hw else xv.astype(np.float64)) @ wv.T.astype(np.float64))
    assert np.allclose(plan.run()[0], e / e.sum(-1, keepdims=True), rtol=1e-4, atol=0)
    s.close()


# rows and lengths with partly empty tiles and waves, two to sixteen slices, one to eight loads per lane; bias and residual before and in the layer norm's prologue.  igemm_r32_sk has tiles
# that are not split: no join, the same results
@pytest.mark.parametrize("rows,k,hid,head,pro,slices", [(389, 3072, 768, (), ("bias_add", "add"), 3), (161, 2048, 64, ("bias_add",), ("add",), 16), (200, 512, 260, ("bias_add", "add"), (), 4),
                                                        (160, 4096, 128, (), (), 16), (333, 1024, 516, ("bias_add",), ("add",), 4), (170, 1024, 1028, (), ("add",), 4),
                                                        (162, 2048, 2048, ("bias_add",), ("add",), 2)])
@pytest.mark.parametrize("backend", ["igemm_r16_sk", "igemm_r32_sk"])
def test_layer_norm_of_partial_results(rows, k, hid, head, pro, slices, backend):
    r = np.random.default_rng(rows + hid)
    f = lambda *sh: r.standard_normal(sh).astype(np.float32)
    d = wl.GraphDesc("split_norm")
    pat, npat = P("dense", W, W), W
    xv, wv = f(rows, k), f(hid, k) / np.float32(k ** 0.5)
    y, ref = d.op("dense", [d.input(xv), d.const(wv)]), xv.astype(np.float64) @ wv.T.astype(np.float64)
    for n, op in enumerate(head + pro):
        t = f(hid) if op == "bias_add" else f(rows, hid)
        ref = ref + t
        y = d.op("bias_add", [y, d.const(t)], axis=-1) if op == "bias_add" else d.op("add", [y, d.input(t)])
        if n < len(head):
            pat = P(op, pat, W)
        else:
            npat = P(op, npat, W)
    g, b = f(hid), f(hid)
    d.mark_output(d.op("layer_norm", [y, d.const(g), d.const(b)], eps=1e-5))
    c = ref - ref.mean(-1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(-1, keepdims=True) + 1e-5) * g + b
    s = clg.Session(d, [(backend, pat), ("rowwise", P("layer_norm", npat, W, W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    split = backend == "igemm_r16_sk"
    assert plan.kernels()[0]["name"].endswith(f"_k{slices}") == split
    got = plan.run()
    assert plan.n_kernels == 2 and launches(plan) == 2
    assert np.linalg.norm(got[0] - ref) < 2e-6 * np.linalg.norm(ref)      # (chains of 1024 products and less: as below)
    assert np.array_equal(got[0], timed(plan)[0])            # one by one: the same sums in the same order
    same_on_two_lanes(plan, got)
    plan.set_lanes(1)
    # operands at addresses that 16-byte loads do not take: one by one
    if "add" in pro:
        n = len(plan._in) - 1
        odd = torch.empty(rows * hid + 1, device="cuda:0")[1:].view(rows, hid)
        odd.copy_(plan._in[n])
        plan._in[n] = odd
        assert launches(plan) == (3 if split else 2)
        plan.execute()
        torch.cuda.synchronize()
        assert np.linalg.norm(plan._out[0].cpu().numpy() - ref) < 2e-6 * np.linalg.norm(ref)
    s.close()


# fp32 dense layers that are split for the layer norm behind them: both ends of both ranges of tiles, a last slice that is short (33 chunks, three per wave: eleven waves of twelve), other tiles, K and
# widths that stay
@pytest.mark.parametrize("rows,k,hid,head,pro,slices", [(1, 2048, 64, (), ("bias_add", "add"), 4), (16, 3072, 768, ("bias_add",), ("add",), 4), (42, 2048, 656, ("bias_add", "add"), (), 4),
                                                        (17, 2064, 68, (), ("add",), 3), (96, 3072, 720, (), ("bias_add", "add"), 4), (80, 4096, 1024, (), ("add",), 4), (96, 2560, 720, (), ("add",), 1),
                                                        (96, 2048, 720, (), ("add",), 1), (96, 4096, 1024, (), ("add",), 1), (64, 3072, 1028, (), ("add",), 1), (128, 3072, 768, (), ("add",), 4),
                                                        (64, 3072, 768, (), ("add",), 1), (144, 3072, 768, (), ("add",), 1), (16, 1536, 768, (), ("add",), 1)])
@pytest.mark.parametrize("backend", ["igemm_r16", "igemm_r16x2_w8", "igemm_r32_w4"])
def test_dense_layers_split_for_a_layer_norm(rows, k, hid, head, pro, slices, backend):
    r = np.random.default_rng(rows + hid)
    f = lambda *sh: r.standard_normal(sh).astype(np.float32)
    d = wl.GraphDesc("split_for_norm")
    pat, npat = P("dense", W, W), W
    xv, wv = f(rows, k), f(hid, k) / np.float32(k ** 0.5)
    y, ref = d.op("dense", [d.input(xv), d.const(wv)]), xv.astype(np.float64) @ wv.T.astype(np.float64)
    for n, op in enumerate(head + pro):
        t = f(hid) if op == "bias_add" else f(rows, hid)
        ref = ref + t
        y = d.op("bias_add", [y, d.const(t)], axis=-1) if op == "bias_add" else d.op("add", [y, d.input(t)])
        if n < len(head):
            pat = P(op, pat, W)
        else:
            npat = P(op, npat, W)
    g, b = 1 + f(hid) / 8, f(hid)
    d.mark_output(d.op("layer_norm", [y, d.const(g), d.const(b)], eps=1e-5))
    c = ref - ref.mean(-1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(-1, keepdims=True) + 1e-5) * g + b
    s = clg.Session(d, [(backend, pat), ("rowwise", P("layer_norm", npat, W, W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    got = plan.run()
    # a chain of up to 2048 / 4 products per K-wave and slice, at random: 1e-6 of the values; their spread is about one
    assert np.linalg.norm(got[0] - ref) < 2e-6 * np.linalg.norm(ref)
    apart = timed(plan)[0]                                   # the kernel that the layer has alone
    assert np.linalg.norm(apart - ref) < 2e-6 * np.linalg.norm(ref)
    assert plan.ws_bytes >= slices * rows * hid * 4 and (slices == 1) == np.array_equal(apart, got[0])
    same_on_two_lanes(plan, got)
    s.close()


def over(plan, k, shift, n):
    """Puts the plan's output 0 into the memory of its input k, `shift` floats behind the input's begin; returns the call that fills the inputs."""
    base = torch.zeros(shift + max(plan._in[k].numel(), n), device="cuda:0")
    value, shape = plan._in[k].clone(), plan._in[k].shape
    plan._in[k] = base[:value.numel()].view(shape)
    out = plan._out[0]
    plan._out[0] = base[shift:shift + out.numel()].view(out.shape)
    return lambda: plan._in[k].copy_(value)


# the softmax over the input, over weights and over a bias that are inputs, and over the logits one row further on: rows that run beside each other would overwrite
# what others read
@pytest.mark.parametrize("where", ["input", "weights", "bias", "logits"])
def test_classifier_with_outputs_over_what_other_rows_read(where):
    r = np.random.default_rng(4)
    m, k, n = 40, 48, 24
    xv, wv, bv = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((n, k)).astype(np.float32), r.standard_normal(n).astype(np.float32)
    d = wl.GraphDesc("outputs_over_inputs")
    logits = d.op("bias_add", [d.op("dense", [d.input(xv), d.input(wv)]), d.input(bv)], axis=-1)
    d.mark_output(d.op("softmax", [logits]))
    if where == "logits":
        d.mark_output(logits)
    s = clg.Session(d, [("igemm_s", P("bias_add", P("dense", W, W), W)), ("rowwise", P("softmax", W))], device=0)
    plan = s.compile(list(range(len(s.match())))).bind()
    assert plan.n_launches == 1
    z = xv.astype(np.float64) @ wv.T.astype(np.float64) + bv
    e = np.exp(z - z.max(-1, keepdims=True))
    want = e / e.sum(-1, keepdims=True)
    fill = lambda: None
    if where == "logits":
        both = torch.zeros((m + 1) * n, device="cuda:0")
        plan._out = [both[n:].view(m, n), both[:m * n].view(m, n)]
    else:
        fill = over(plan, ("input", "weights", "bias").index(where), 8, m * n)
    for _ in range(3):
        fill()
        plan.execute()
        torch.cuda.synchronize()
        assert np.allclose(plan._out[0].cpu().numpy(), want, rtol=1e-4, atol=1e-7)
    s.close()


# the layer norm's result over the residual of the dense layer in front of it (its own row: joined; a row further on: not) and over its bias
@pytest.mark.parametrize("where,shift", [(1, 0), (1, 260), (2, 0)], ids=["residual", "residual a row on", "bias"])
@pytest.mark.parametrize("backend,rows", [("igemm_r16_sk", 200), ("igemm_r16", 16)], ids=["split", "split for it"])
def test_layer_norm_over_what_its_dense_layer_adds(backend, rows, where, shift):
    r = np.random.default_rng(6)
    f = lambda *sh: r.standard_normal(sh).astype(np.float32)
    k, hid = 2048, 260
    xv, av, bv, wv, g, b = f(rows, k), f(rows, hid), f(hid), f(hid, k) / np.float32(k ** 0.5), f(hid), f(hid)
    d = wl.GraphDesc("norm_over_inputs")
    x, a, bias = d.input(xv), d.input(av), d.input(bv)
    y = d.op("add", [d.op("bias_add", [d.op("dense", [x, d.const(wv)]), bias], axis=-1), a])
    d.mark_output(d.op("layer_norm", [y, d.const(g), d.const(b)], eps=1e-5))
    s = clg.Session(d, [(backend, P("add", P("bias_add", P("dense", W, W), W), W)), ("rowwise", P("layer_norm", W, W, W))], device=0)
    plan = s.compile(list(range(len(s.match())))).bind()
    z = xv.astype(np.float64) @ wv.T.astype(np.float64) + bv + av
    z -= z.mean(-1, keepdims=True)
    want = z / np.sqrt((z * z).mean(-1, keepdims=True) + 1e-5) * g + b
    fill = over(plan, where, shift, rows * hid)
    for _ in range(3):
        fill()
        plan.execute()
        torch.cuda.synchronize()
        assert np.linalg.norm(plan._out[0].cpu().numpy() - want) < 2e-6 * np.linalg.norm(want)       # (as below)
    s.close()
