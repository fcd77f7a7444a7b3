"""Register-fed dense layers whose K is a multiple of 4 but not of the group that an MFMA round takes, against float64."""
import numpy as np
import pytest
import torch

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg

pytestmark = pytest.mark.gpu

BACKENDS = ["igemm_r16", "igemm_r16_w4", "igemm_r32", "igemm_r32_w4"]


def dense(m, k, n, xv, wv, tail, backend):
    r = np.random.default_rng(n)
    d = wl.GraphDesc("ragged_dense")
    bv, av = r.standard_normal(n).astype(np.float32), r.standard_normal((m, n)).astype(np.float32)
    y, pat = d.op("dense", [d.input(xv), d.const(wv)]), P("dense", W, W)
    with np.errstate(invalid="ignore"):
        ref = xv.astype(np.float64) @ wv.T.astype(np.float64)
    if tail:
        y, pat, ref = d.op("bias_add", [y, d.const(bv)], axis=-1), P("bias_add", pat, W), ref + bv
        y, pat, ref = d.op("add", [y, d.input(av)]), P("add", pat, W), ref + av
        y, pat, ref = d.op("relu", [y]), P("relu", pat), np.where(ref > 0, ref, 0)
    d.mark_output(y)
    s = clg.Session(d, [(backend, pat)], device=0)
    ids = [i for i, mt in enumerate(s.match()) if mt.n_nodes == len(d.op_nodes())]
    plan = s.compile(ids)
    return s, plan, ref


# last groups of one to three parts of 16 bytes (one of two with 32x32 tiles), one group and many, waves without work; rows and columns that end inside a tile
@pytest.mark.parametrize("m,k,n,tail", [(1, 20, 5, 0), (16, 20, 300, 1), (5, 100, 130, 1), (33, 100, 64, 0), (64, 100, 1000, 1), (17, 36, 48, 0), (40, 60, 33, 1), (9, 1028, 70, 1), (64, 2100, 17, 0)])
@pytest.mark.parametrize("backend", BACKENDS)
def test_ragged(m, k, n, tail, backend):
    r = np.random.default_rng(k * n + m)
    xv, wv = r.standard_normal((m, k)).astype(np.float32), (r.standard_normal((n, k)) / k ** 0.5).astype(np.float32)
    s, plan, ref = dense(m, k, n, xv, wv, tail, backend)
    assert plan.kernels()[0]["name"].startswith("dense4_rf" if k % (8 if "r32" in backend else 16) else "dense_rf")
    got = plan.run()[0]
    bound = (k / 4 + 24) * 2.0 ** -24 * (np.abs(xv).astype(np.float64) @ np.abs(wv).T + 6)       # an MFMA adds two or four products at a time; bias and residual are below 6
    assert (np.abs(got - ref) <= bound).all()
    if plan.kernels()[0]["name"].startswith("dense4"):       # rows at an address that is a float's only
        odd = torch.empty(m * k + 1, device="cuda:0")[1:].view(m, k)
        odd.copy_(torch.from_numpy(xv))
        plan._in[0] = odd
        plan.execute()
        torch.cuda.synchronize()
        assert np.array_equal(plan._out[0].cpu().numpy(), got)
    s.close()


@pytest.mark.parametrize("value", [np.inf, np.nan], ids=str)
@pytest.mark.parametrize("backend", BACKENDS)
def test_values_that_are_not_finite(value, backend):
    """What is read again behind K meets zero weights: it must not make an infinity NaN, nor NaN out of another row's value."""
    m, k, n = 20, 100, 40
    r = np.random.default_rng(3)
    xv, wv = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((n, k)).astype(np.float32)
    xv[3, 99], xv[7, 96], xv[11, 0], xv[18, 50] = value, value, value, value
    wv[:, [0, 50, 96, 99]] = np.abs(wv[:, [0, 50, 96, 99]]) + 0.5
    s, plan, ref = dense(m, k, n, xv, wv, 0, backend)
    got = plan.run()[0]
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    ok = np.isfinite(ref)
    assert ok.sum() == (m - 4) * n and np.abs(got - ref)[ok].max() < 1e-4
    s.close()
