"""Networks whose weights exceed the memory-side cache: layer norms and attention carry workgroups that read later kernels' weights ahead.  Rows at
the ends of where they do (below, the smallest, more rows than read-ahead waves, attention that leaves few compute units or none), against float64."""
import numpy as np
import pytest

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg

pytestmark = pytest.mark.gpu

PAIRS, HID, MID = 17, 1024, 2048          # 17 x 2 x 8.4 MB of weights: 285 MB
HEADS, D = 12, 64


@pytest.fixture(scope="module")
def weights():
    r = np.random.default_rng(7)
    return [(r.standard_normal((MID, HID)) / 32).astype(np.float32) if k % 2 == 0 else (r.standard_normal((HID, MID)) / 45).astype(np.float32)
            for k in range(2 * PAIRS)]


@pytest.mark.parametrize("rows", [95, 96, 389, 512, 700])
def test_a_network_larger_than_the_memory_side_cache(weights, rows):
    r = np.random.default_rng(rows)
    d = wl.GraphDesc("read_ahead")
    xv = r.standard_normal((rows, HID)).astype(np.float32)
    keys = min(rows, 512)
    qkv = [r.standard_normal((HEADS, keys, D)).astype(np.float32) for _ in range(3)]
    g, b = (1 + 0.1 * r.standard_normal(HID)).astype(np.float32), (0.1 * r.standard_normal(HID)).astype(np.float32)
    x = d.input(xv)
    q, k, v = (d.input(t) for t in qkv)
    gn, bn = d.const(g), d.const(b)
    a = d.op("batch_matmul", [q, k], transpose_b=True)
    a = d.op("softmax", [d.op("mul_scalar", [a], scalar=0.125)])
    d.mark_output(d.op("batch_matmul", [a, v], transpose_b=False))
    y, ref = x, xv.astype(np.float64)
    for n, w in enumerate(weights):
        if n % 2 == 0:
            y = d.op("layer_norm", [y, gn, bn], eps=1e-5)
            c = ref - ref.mean(-1, keepdims=True)
            ref = c / np.sqrt((c * c).mean(-1, keepdims=True) + 1e-5) * g + b
        y = d.op("dense", [y, d.const(w)])
        ref = ref @ w.T.astype(np.float64)
    d.mark_output(y)
    att = P("batch_matmul", P("softmax", P("mul_scalar", P("batch_matmul", W, W))), W)
    s = clg.Session(d, [("attention", att), ("igemm_r16_w4", P("dense", W, W)), ("rowwise", P("layer_norm", W, W, W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    assert any("attention" in kk["name"] for kk in plan.kernels())
    got = plan.run()
    again = plan.run()
    s.close()
    assert all(np.array_equal(a, c) for a, c in zip(got, again))
    p = np.einsum("hqd,hkd->hqk", qkv[0].astype(np.float64), qkv[1].astype(np.float64)) * 0.125
    p = np.exp(p - p.max(-1, keepdims=True))
    want = np.einsum("hqk,hkd->hqd", p / p.sum(-1, keepdims=True), qkv[2].astype(np.float64))
    assert np.linalg.norm(got[0] - want) < 3e-6 * np.linalg.norm(want)
    # 34 fp32 products of up to 2048 terms and 17 normalisations one after the other: 2e-7 each, adding up at random
    assert np.linalg.norm(got[1] - ref) < 1e-5 * np.linalg.norm(ref)


def test_weights_of_a_region_are_read_ahead_in_the_copy_that_runs():
    """Layer norms in front of three dense siblings whose own kernels are fp32 ones and whose region is a split-operand launch with packed copies of its own:
    launched apart, one of them handed over (still its own kernel), two and all three.  Every choice of digits against float64, and again bit for bit."""
    blocks, rows, hid, mid = 24, 320, 1024, 768               # 24 x 4 x 3.1 MB of weights as fp32: 302 MB
    r = np.random.default_rng(11)
    ws = [(r.standard_normal((mid, hid)) / 32).astype(np.float32) for _ in range(3)] + [(r.standard_normal((hid, mid)) / 48).astype(np.float32)]
    xv = r.standard_normal((rows, hid)).astype(np.float32)
    g, b = (1 + 0.1 * r.standard_normal(hid)).astype(np.float32), (0.1 * r.standard_normal(hid)).astype(np.float32)
    d = wl.GraphDesc("read_ahead_region")
    y, ref = d.input(xv), xv.astype(np.float64)
    gn, bn = d.const(g), d.const(b)
    for _ in range(blocks):
        y = d.op("layer_norm", [y, gn, bn], eps=1e-5)
        p = [d.op("dense", [y, d.const(w)]) for w in ws[:3]]
        y = d.op("dense", [d.op("add", [d.op("add", p[:2]), p[2]]), d.const(ws[3])])
        c = ref - ref.mean(-1, keepdims=True)
        ref = c / np.sqrt((c * c).mean(-1, keepdims=True) + 1e-5) * g + b
        ref = sum(ref @ w.T.astype(np.float64) for w in ws[:3]) @ ws[3].T.astype(np.float64)
    d.mark_output(y)
    s = clg.Session(d, [("igemm_r16_w4", P("dense", W, W)), ("rowwise", P("layer_norm", W, W, W)), ("eltwise", P("add", W, W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    assert all((by >= 3 * 4 * hid * mid) == (gr == 256) == k["name"].startswith("layer_norm") for k, (by, gr) in zip(plan.kernels(), plan.read_ahead()))
    rg, n = plan.regions(), plan.n_kernels
    assert len(set(rg)) == blocks + 1 and all(rg.count(k) == 3 for k in range(blocks)), rg
    nth = [rg[:i].count(rg[i]) if rg[i] >= 0 else 3 for i in range(n)]      # place of a member in its region
    for handed, launches in ((0, n), (1, n), (2, n - blocks), (3, n - 2 * blocks)):
        plan.set_handover([int(k < handed) for k in nth], 1)
        assert plan.n_launches == launches
        got = plan.run()[0]
        assert np.array_equal(got, plan.run()[0]), handed
        # 48 products of up to 1024 terms and 24 normalisations one after the other: 2e-7 each, adding up at random
        assert np.linalg.norm(got - ref) < 1e-5 * np.linalg.norm(ref), handed
    s.close()


@pytest.mark.parametrize("rows", [304, 305, 336, 384, 385])
def test_lengths_at_which_attention_covers_most_compute_units(rows):
    """One encoder layer's attention beside more weights than the cache holds, with few, no and (two row tiles) many compute units to read ahead on."""
    r = np.random.default_rng(rows)
    d = wl.GraphDesc("read_ahead_attention")
    qkv = [r.standard_normal((HEADS, rows, D)).astype(np.float32) for _ in range(3)]
    q, k, v = (d.input(t) for t in qkv)
    a = d.op("softmax", [d.op("mul_scalar", [d.op("batch_matmul", [q, k], transpose_b=True)], scalar=0.125)])
    y = d.op("reshape", [d.op("transpose", [d.op("batch_matmul", [a, v], transpose_b=False)], dims=(1, 0, 2))], dims=(rows, HEADS * D))
    p = np.einsum("hqd,hkd->hqk", qkv[0].astype(np.float64), qkv[1].astype(np.float64)) * 0.125
    p = np.exp(p - p.max(-1, keepdims=True))
    ref = np.einsum("hqk,hkd->qhd", p / p.sum(-1, keepdims=True), qkv[2].astype(np.float64)).reshape(rows, HEADS * D)
    ws = [(r.standard_normal((HEADS * D, HEADS * D)) / 28).astype(np.float32) for _ in range(2)]
    for n in range(128):                                      # 128 x 2.4 MB as fp32: 302 MB; two products of them in a row
        y, ref = (d.op("dense", [y, d.const(ws[n % 2])]), ref @ ws[n % 2].T.astype(np.float64)) if n < 2 else (y, ref)
        if n >= 2:
            d.mark_output(d.op("dense", [y, d.const(ws[n % 2])]))
    d.mark_output(y)
    att = P("reshape", P("transpose", P("batch_matmul", P("softmax", P("mul_scalar", P("batch_matmul", W, W))), W)))
    s = clg.Session(d, [("attention", att), ("igemm_r16_w4", P("dense", W, W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    nbytes, groups = plan.read_ahead()[0]
    assert (groups > 0) == (rows not in (305, 336, 384)) and (nbytes > 0) == (groups > 0)
    got = plan.run()[-1]
    s.close()
    assert np.linalg.norm(got - ref) < 3e-6 * np.linalg.norm(ref)
