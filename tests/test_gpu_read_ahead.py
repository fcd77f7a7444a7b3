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
