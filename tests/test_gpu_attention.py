"""One-kernel attention where its launch changes: up to 128 keys and beyond, the most keys, one and two row tiles per
workgroup (two where single ones are more than the 256 compute units), ragged rows and keys, every head size.  Against float64:
scores of d products, probabilities and sums of up to 512 terms in fp32, exp to two units in the last place of
arguments up to 8: 3e-6 of the result's norm."""
import numpy as np
import pytest

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg

pytestmark = pytest.mark.gpu

# heads, queries, keys, head size
CASES = [(12, 128, 128, 64), (12, 129, 129, 64), (12, 336, 336, 64), (12, 337, 389, 64), (12, 512, 512, 64), (1, 7, 130, 64),
         (17, 250, 300, 32), (40, 100, 512, 32), (3, 40, 97, 32), (9, 470, 144, 128), (2, 31, 128, 128), (300, 17, 3, 64),
         # more workgroups than compute units: slices of k of both widths (heads of 32, on both sides of 448 keys), every count of key tiles per wave
         (80, 100, 470, 32), (80, 100, 512, 32), (80, 100, 448, 32), (300, 5, 9, 128), (40, 130, 70, 128), (40, 130, 250, 128), (30, 150, 300, 128), (70, 150, 250, 64)]


@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_attention_against_float64(case, merged):
    h, sq, sk, dd = case
    r = np.random.default_rng([59, *case])
    q, k, v = (r.standard_normal((h, n, dd)).astype(np.float32) for n in (sq, sk, sk))
    s = q.astype(np.float64) @ k.astype(np.float64).transpose(0, 2, 1) * np.float64(np.float32(dd ** -0.5))
    p = np.exp(s - s.max(-1, keepdims=True))
    ref = p / p.sum(-1, keepdims=True) @ v.astype(np.float64)
    d = wl.GraphDesc("attention")
    y = d.op("batch_matmul", [d.input(q), d.input(k)], transpose_b=True)
    y = d.op("softmax", [d.op("mul_scalar", [y], scalar=float(np.float32(dd ** -0.5)))])
    y = d.op("batch_matmul", [y, d.input(v)], transpose_b=False)
    pat = P("batch_matmul", P("softmax", P("mul_scalar", P("batch_matmul", W, W))), W)
    if merged:
        y = d.op("reshape", [d.op("transpose", [y], dims=(1, 0, 2))], dims=(sq, h * dd))
        pat, ref = P("reshape", P("transpose", pat)), ref.transpose(1, 0, 2).reshape(sq, h * dd)
    d.mark_output(y)
    sess = clg.Session(d, [("attention", pat)], device=0)
    sess.match()
    plan = sess.compile([0])
    got, again = plan.run()[0], plan.run()[0]
    sess.close()
    assert np.array_equal(got, again)
    assert np.linalg.norm(got - ref) < 3e-6 * np.linalg.norm(ref)
