"""Transposed convolutions with 4x4 filters, stride 2, pad 1 and one to four output channels in the direct backend."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

import paper_2111_00655_amd as clg
import workloads as wl
from workloads.patterns import P, W

pytestmark = pytest.mark.gpu


def run(x, w, tail=()):
    d = wl.GraphDesc("few_convt")
    y = d.op("conv2d_transpose", [d.input(x), d.const(w)], stride=(2, 2), pad=(1, 1))
    pat = P("conv2d_transpose", W, W)
    for op, operand in tail:
        y = d.op(op, [y] if operand is None else [y, d.const(operand)], **({"axis": 1} if op == "bias_add" else {}))
        pat = P(op, pat) if operand is None else P(op, pat, W)
    d.mark_output(y)
    s = clg.Session(d, [("direct", pat)], device=0)
    whole = [i for i, m in enumerate(s.match()) if m.n_nodes == len(d.op_nodes())]
    got = s.compile(whole).run()[0]
    s.close()
    return got


def data(n, cin, cout, hw, seed):
    r = np.random.default_rng(seed)
    return r.standard_normal((n, cin) + hw).astype(np.float32), (r.standard_normal((cin, cout, 4, 4)) * (4 * cin) ** -0.5).astype(np.float32), r


# (images, channels in, out, (height, width), tail): one position; a workgroup's 64 positions exactly, one more; fewer channels than
# waves, channels that the waves cannot share evenly; more than 512 workgroups of one position per lane: two, at odd and even heights
CASES = [(1, 1, 1, (1, 1), ""), (1, 64, 3, (8, 8), "bt"), (1, 33, 3, (5, 13), "bt"), (2, 3, 2, (1, 65), "br"), (1, 40, 4, (7, 9), "ba"),
         (3, 17, 4, (65, 1), "b"), (1, 100, 1, (16, 16), "bar"), (17, 33, 3, (31, 33), "bt"), (34, 33, 3, (31, 33), "bt"),
         (35, 5, 4, (31, 33), "ba"), (33, 6, 1, (32, 32), ""), (9, 64, 2, (64, 64), "b")]


@pytest.mark.parametrize("n,cin,cout,hw,tail", CASES)
def test_against_64_bits(n, cin, cout, hw, tail):
    x, w, r = data(n, cin, cout, hw, 7)
    bias = r.standard_normal(cout).astype(np.float32)
    add = r.standard_normal((n, cout, 2 * hw[0], 2 * hw[1])).astype(np.float32)
    steps = {"b": ("bias_add", bias), "a": ("add", add), "r": ("relu", None), "t": ("tanh", None)}
    got = run(x, w, [steps[t] for t in tail])
    ref = F.conv_transpose2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), stride=2, padding=1).numpy()
    mag = F.conv_transpose2d(torch.from_numpy(abs(x)).double(), torch.from_numpy(abs(w)).double(), stride=2, padding=1).numpy()
    for t in tail:
        ref = {"b": lambda v: v + bias[:, None, None], "a": lambda v: v + add, "r": lambda v: np.maximum(v, 0), "t": np.tanh}[t](ref)
    # at most 4 * cin roundings of a partial sum that is no larger than the sum of absolute products; the tail's few on values of size one
    np.testing.assert_array_less(abs(got - ref), 4 * cin * 2.0 ** -24 * mag + 8 * 2.0 ** -24 * (1 + abs(ref)))


@pytest.mark.parametrize("n,hw", [(2, (4, 6)), (34, (31, 33))])
def test_infinities_stay_where_their_taps_are(n, hw):
    x, w, _ = data(n, 5, 3, hw, 8)
    x[0, 2, 0, 0], x[1, 1, 3, 5], w[3, 1, 0, 2], w[4, 2, 3, 3] = np.inf, np.nan, np.inf, -np.inf
    got = run(x, w)
    ref = F.conv_transpose2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), stride=2, padding=1).numpy()
    fin = np.isfinite(ref)
    np.testing.assert_array_equal(np.isfinite(got), fin)
    np.testing.assert_array_equal(np.nan_to_num(got[~fin], posinf=2, neginf=-2), np.nan_to_num(ref[~fin], posinf=2, neginf=-2))
    np.testing.assert_allclose(got[fin], ref[fin], rtol=0, atol=1e-5)
