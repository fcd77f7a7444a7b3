"""3x3 convolutions of a few channels per group on the vector units (four output rows per thread): heights that are no
multiple of four, strides and pads, groups of unequal input and output widths, tails.  Against float64; K is at
most 9 * 32 products in one fp32 chain, whose rounding is below sqrt(288) / 2 * 2^-24 of the result's norm (5e-7)."""
import numpy as np
import pytest

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg

pytestmark = pytest.mark.gpu

# images, in, out channels, groups, height, width, stride, pad
CASES = [
    (1, 128, 128, 32, 56, 56, 1, 1),       # ResNeXt-50's groups of four
    (3, 64, 64, 8, 13, 17, 1, 1),          # groups of eight, ragged rows
    (2, 32, 64, 16, 9, 10, 2, 1),          # two in, four out, stride 2
    (5, 12, 24, 3, 3, 3, 1, 0),            # one output row
    (1, 96, 48, 3, 31, 7, 2, 0),           # groups of 32 in, 16 out
    (2, 8, 8, 2, 1, 1, 1, 1),              # everything but one value is padding
    (1, 18, 36, 3, 6, 300, 1, 2),          # groups of six, more padding than the filter needs
]


@pytest.mark.parametrize("tail", [(), ("bias_add", "relu"), ("bias_add", "add", "relu")], ids=lambda t: "+".join(t) or "none")
@pytest.mark.parametrize("case", CASES)
def test_narrow_groups_against_float64(case, tail):
    import torch
    n, cin, cout, g, h, w, s, p = case
    r = np.random.default_rng([53, *case])

    def f32(*shape, scale=1.0):
        return (r.standard_normal(shape) * scale).astype(np.float32)

    x, wt = f32(n, cin, h, w), f32(cout, cin // g, 3, 3, scale=(cin // g * 9) ** -0.5)
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wt).double(), stride=s, padding=p, groups=g).numpy()
    d = wl.GraphDesc("grouped")
    y = d.op("conv2d", [d.input(x), d.const(wt)], stride=(s, s), pad=(p, p), groups=g)
    pat = P("conv2d", W, W)
    for op in tail:
        if op == "bias_add":
            b = f32(cout)
            ref = ref + b.astype(np.float64).reshape(1, -1, 1, 1)
            y, pat = d.op("bias_add", [y, d.const(b)], axis=1), P("bias_add", pat, W)
        elif op == "add":
            a = f32(*ref.shape)
            ref = ref + a
            y, pat = d.op("add", [y, d.input(a)]), P("add", pat, W)
        else:
            ref, y, pat = np.maximum(ref, 0), d.op("relu", [y]), P("relu", pat)
    d.mark_output(y)
    sess = clg.Session(d, [("direct", pat)], device=0)
    full = [i for i, m in enumerate(sess.match()) if m.n_nodes == len(d.op_nodes())]
    got = sess.compile(full).run()[0]
    sess.close()
    assert np.linalg.norm(got - ref) < 5e-7 * np.linalg.norm(ref) + 1e-30
