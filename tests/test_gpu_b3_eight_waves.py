"""Split-operand kernels of eight waves per 64x64 tile for 3x3 filters and the 2x2-tap phases of transposed convolutions: 256 channels and more, tiles for more than
half of the compute units but no more than there are, against float64."""
import numpy as np
import pytest
import torch

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg

pytestmark = pytest.mark.gpu


# (transposed, images, channels in and out, size, stride, whether the rule takes it): stages that end inside a block of channels, rows and columns that end inside a
# tile, tiles on both sides of the rule, a patch (stride 2) of which 64 channels do not fit
@pytest.mark.parametrize("t,n,cin,cout,h,stride,w8", [(0, 16, 256, 256, 14, 1, 1), (0, 17, 264, 250, 13, 1, 1), (0, 30, 272, 200, 21, 2, 0), (0, 7, 320, 256, 15, 1, 0), (0, 17, 240, 250, 13, 1, 0),
                                                      (0, 24, 256, 256, 14, 1, 0), (1, 40, 512, 256, 4, 2, 1), (1, 31, 256, 120, 8, 2, 1), (1, 34, 256, 120, 8, 2, 0)])
def test_eight_waves(t, n, cin, cout, h, stride, w8):
    r = np.random.default_rng(n * cin)
    k = 4 if t else 3
    xv = r.standard_normal((n, cin, h, h)).astype(np.float32)
    wv = (r.standard_normal((cin, cout, k, k) if t else (cout, cin, k, k)) / (cin * 9) ** 0.5).astype(np.float32)
    bv = r.standard_normal(cout).astype(np.float32)
    kind = "conv2d_transpose" if t else "conv2d"
    d = wl.GraphDesc("eight_waves")
    y = d.op(kind, [d.input(xv), d.const(wv)], stride=(stride, stride), pad=(1, 1))
    d.mark_output(d.op("relu", [d.op("bias_add", [y, d.const(bv)], axis=1)]))
    s = clg.Session(d, [("igemm_r16_sk", P("relu", P("bias_add", P(kind, W, W), W)))], device=0)
    s.match()
    plan = s.compile([0])
    assert ("m64n64w8" in plan.kernels()[0]["name"]) == bool(w8), plan.kernels()[0]["name"]
    got = plan.run()[0]
    f = torch.nn.functional.conv_transpose2d if t else torch.nn.functional.conv2d
    want = torch.relu(f(torch.from_numpy(xv).double(), torch.from_numpy(wv).double(), torch.from_numpy(bv).double(), stride=stride, padding=1)).numpy()
    # sums of up to 4608 products, rounded once per 16 of them: the square root of 288 roundings of half a unit, 5e-7
    assert np.linalg.norm(got - want) < 1e-6 * np.linalg.norm(want)
    s.close()
