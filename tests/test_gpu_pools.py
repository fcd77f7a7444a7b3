"""Pools where their kernels branch: 3x3 and 3x3x3 windows (all loads at once) over images smaller than a window, windows that hang over every edge, other windows beside them;
global averages of one wave's lanes, one more, and more than eight rounds of loads.  Against the oracle: maxima are the same values, averages of n terms agree to n roundings."""
import numpy as np
import pytest

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg
from oracle.graph import Graph

pytestmark = pytest.mark.gpu

WINDOWS = [((2, 3, 1, 1), 3, 1, 1), ((1, 2, 2, 5), 3, 2, 1), ((3, 5, 14, 9), 3, 3, 0), ((1, 4, 33, 31), 3, 2, 1), ((2, 2, 7, 8), 2, 2, 0), ((1, 3, 9, 9), 5, 1, 2),
           ((1, 2, 1, 1, 1), 3, 1, 1), ((2, 3, 5, 4, 7), 3, 2, 1), ((1, 2, 4, 6, 5), 2, 2, 0)]


@pytest.mark.parametrize("avg", [False, True], ids=["max", "avg"])
@pytest.mark.parametrize("case", WINDOWS, ids=str)
def test_window_pools(case, avg):
    shape, k, st, pad = case
    n = len(shape) - 2
    if avg and n == 3:
        pytest.skip("no 3-D average window pool")
    d = wl.GraphDesc("pool")
    x = d.input(np.random.default_rng(len(shape) * 100 + k).standard_normal(shape).astype(np.float32))
    kind = "avg_pool2d" if avg else f"max_pool{n}d"
    d.mark_output(d.op(kind, [x], kernel=(k,) * n, stride=(st,) * n, pad=(pad,) * n))
    s = clg.Session(d, [("direct", P(kind, W))], device=0)
    s.match()
    got, ref = s.compile([0]).run()[0], Graph(d).run()[0]
    s.close()
    if avg:
        np.testing.assert_allclose(got, ref, rtol=0, atol=k * k * 2.0 ** -24 * 4)
    else:
        np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("hw", [(1, 1), (7, 7), (8, 8), (5, 13), (24, 24), (31, 33), (90, 77)])
def test_global_average(hw):
    d = wl.GraphDesc("gap")
    x = d.input(np.random.default_rng(hw[1]).standard_normal((3, 5) + hw).astype(np.float32))
    d.mark_output(d.op("global_avg_pool2d", [x]))
    s = clg.Session(d, [("direct", P("global_avg_pool2d", W))], device=0)
    s.match()
    got, ref = s.compile([0]).run()[0], Graph(d).run()[0]
    s.close()
    # sums of hw terms of size one, rounded once per addition of a lane's and the lanes' partial sums
    np.testing.assert_allclose(got, ref, rtol=0, atol=4 * 2.0 ** -24 * (hw[0] * hw[1]) ** 0.5)


@pytest.mark.parametrize("case,avg", [(c, avg) for c in WINDOWS for avg in (False, True) if not (avg and len(c[0]) == 5)], ids=str)
def test_windows_of_values_that_are_not_finite(case, avg):
    """A maximum passes over NaN (nothing but NaN: minus infinity) and takes infinities and the lowest float as they are; an average is of the pixels inside the image,
    whatever lies behind the edge."""
    shape, k, st, pad = case
    n = len(shape) - 2
    r = np.random.default_rng(len(shape) * 100 + k)
    lowest = np.finfo(np.float32).min
    xv = r.choice(np.array([-np.inf, lowest, -1, 2, np.nan] + ([] if avg else [np.inf]), np.float32), shape, p=[.2, .2, .3, .2, .1] if avg else [.3, .2, .1, .05, .3, .05])
    d = wl.GraphDesc("pool")
    kind = "avg_pool2d" if avg else f"max_pool{n}d"
    d.mark_output(d.op(kind, [d.input(xv)], kernel=(k,) * n, stride=(st,) * n, pad=(pad,) * n))
    s = clg.Session(d, [("direct", P(kind, W))], device=0)
    s.match()
    got = s.compile([0]).run()[0]
    s.close()
    wide = [(0, 0), (0, 0)] + [(pad, pad)] * n
    win = np.lib.stride_tricks.sliding_window_view(np.pad(xv.astype(np.float64), wide), (k,) * n, axis=tuple(range(2, n + 2)))
    ins = np.lib.stride_tricks.sliding_window_view(np.pad(np.ones(shape, bool), wide), (k,) * n, axis=tuple(range(2, n + 2)))
    step = (slice(None), slice(None)) + (slice(None, None, st),) * n
    win, ins, axes = win[step], ins[step], tuple(range(-n, 0))
    if avg:
        with np.errstate(invalid="ignore"):
            sums = np.where(ins, win, 0).sum(axes)
        ref = np.where(sums < 1.5 * float(lowest), -np.inf, sums) / ins.sum(axes)                # (two of the lowest float are below the range)
        np.testing.assert_allclose(got, ref, rtol=k * k * 2.0 ** -24, atol=k * k * 2.0 ** -24 * 4)
    else:
        np.testing.assert_array_equal(got, np.where(ins & ~np.isnan(win), win, -np.inf).max(axes))
