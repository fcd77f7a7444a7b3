"""Dense layers of one to four rows and 64 <= K < 512 (sixteen lanes per output column), against float64."""
import numpy as np
import pytest
import torch

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg

pytestmark = pytest.mark.gpu


# K at the ends of one, two, four and eight loads per lane; N with a last workgroup and a last wave that are partly empty; the row counts
# on both sides of the rule
@pytest.mark.parametrize("m,k,n,tail", [(1, 64, 1, ()), (1, 100, 8192, ("bias_add", "relu")), (2, 128, 17, ("bias_add",)), (3, 132, 35, ("bias_add", "add")),
                                        (4, 252, 130, ("bias_add", "tanh")), (4, 256, 66, ()), (1, 260, 5, ("bias_add", "gelu")), (4, 508, 70, ("bias_add", "add", "relu"))])
def test_short_rows(m, k, n, tail):
    r = np.random.default_rng(k * n + m)
    d = wl.GraphDesc("short_rows")
    xv, w, b, add = (r.standard_normal(s) for s in ((m, k), (n, k), (n,), (m, n)))
    xv, w, b, add = (t.astype(np.float32) for t in (xv, w / k ** 0.5, b, add))
    y, pat = d.op("dense", [d.input(xv), d.const(w)]), P("dense", W, W)
    size = np.abs(xv).astype(np.float64) @ np.abs(w).T.astype(np.float64)
    ref = torch.from_numpy(xv.astype(np.float64) @ w.T.astype(np.float64))
    for op in tail:
        if op == "bias_add":
            y, ref = d.op(op, [y, d.const(b)], axis=-1), ref + torch.from_numpy(b).double()
        elif op == "add":
            y, ref = d.op(op, [y, d.input(add)]), ref + torch.from_numpy(add).double()
        else:
            y, ref = d.op(op, [y]), {"relu": torch.relu, "tanh": torch.tanh, "gelu": torch.nn.functional.gelu}[op](ref)
        pat = P(op, pat, W) if op in ("bias_add", "add") else P(op, pat)
    d.mark_output(y)
    s = clg.Session(d, [("igemm_s8", pat)], device=0)
    ids = [i for i, mt in enumerate(s.match()) if mt.n_nodes == len(d.op_nodes())]
    plan = s.compile(ids)
    assert [c["name"] for c in plan.kernels()] == ["gemv16_nt"]
    # a lane adds at most 4 x 8 products one after the other, then sixteen partial sums; the tail rounds a few times more
    bound = 40 * 2.0 ** -24 * (size + np.abs(add) + np.abs(b) + 1)
    got = plan.run()[0]
    assert (np.abs(got - ref.numpy()) <= bound).all()
    # the input at an address that 16-byte loads do not take
    shifted = torch.empty(m * k + 1, device="cuda:0")[1:].view(m, k)
    shifted.copy_(torch.from_numpy(xv))
    plan._in[0] = shifted
    plan.execute()
    torch.cuda.synchronize()
    assert (np.abs(plan._out[0].cpu().numpy() - ref.numpy()) <= (2 * k + 8) * 2.0 ** -24 * (size + np.abs(add) + np.abs(b) + 1)).all()
    s.close()


def test_five_rows_stay_with_the_tiled_kernels():
    r = np.random.default_rng(0)
    d = wl.GraphDesc("five_rows")
    d.mark_output(d.op("dense", [d.input(r.standard_normal((5, 100)).astype(np.float32)), d.const(r.standard_normal((64, 100)).astype(np.float32))]))
    s = clg.Session(d, [("igemm_s8", P("dense", W, W))], device=0)
    s.match()
    assert s.compile([0]).kernels()[0]["name"].startswith("gemm_nt")
    s.close()
