"""A split dense layer whose partial results the layer norm behind it adds up: one by one (timed) and joined."""
import numpy as np
import pytest
import torch

import workloads as wl
from workloads.patterns import P, W
import paper_2111_00655_amd as clg
from paper_2111_00655_amd import binding as B

pytestmark = pytest.mark.gpu


def both(plan):
    """Outputs of a joined execution and of one kernel after the other."""
    got = plan.run()
    ns = plan.execute_timed()
    torch.cuda.synchronize()
    assert (np.asarray(ns) > 0).all()
    return got, [t.cpu().numpy() for t in plan._out]


# rows and lengths with partly empty tiles and waves, two to sixteen slices, one to eight loads per lane; bias and residual before and in the layer norm's prologue
@pytest.mark.parametrize("rows,k,hid,head,pro", [(389, 3072, 768, (), ("bias_add", "add")), (161, 2048, 64, ("bias_add",), ("add",)), (200, 512, 260, ("bias_add", "add"), ()),
                                                 (160, 4096, 128, (), ()), (333, 1024, 516, ("bias_add",), ("add",)), (170, 1024, 1028, (), ("add",)), (162, 2048, 2048, ("bias_add",), ("add",))])
@pytest.mark.parametrize("backend", ["igemm_r16_sk", "igemm_r32_sk"])
def test_layer_norm_of_partial_results(rows, k, hid, head, pro, backend):
    r = np.random.default_rng(rows + hid)
    f = lambda *sh: r.standard_normal(sh).astype(np.float32)
    d = wl.GraphDesc("split_norm")
    pat = P("dense", W, W)
    y = d.op("dense", [d.input(f(rows, k)), d.const(f(hid, k) / k ** 0.5)])
    for op in head:
        y = d.op("bias_add", [y, d.const(f(hid))], axis=-1) if op == "bias_add" else d.op("add", [y, d.input(f(rows, hid))])
        pat = P(op, pat, W)
    npat = W
    for op in pro:
        y = d.op("bias_add", [y, d.const(f(hid))], axis=-1) if op == "bias_add" else d.op("add", [y, d.input(f(rows, hid))])
        npat = P(op, npat, W)
    d.mark_output(d.op("layer_norm", [y, d.const(f(hid)), d.const(f(hid))], eps=1e-5))
    s = clg.Session(d, [(backend, pat), ("rowwise", P("layer_norm", npat, W, W))], device=0)
    plan = s.compile(list(range(len(s.match()))))
    got, apart = both(plan)
    assert plan.n_kernels == 2
    assert np.array_equal(got[0], apart[0])                  # the same sums in the same order
    # operands at addresses that 16-byte loads do not take: one by one
    if "add" in pro:
        n = len(plan._in) - 1
        odd = torch.empty(rows * hid + 1, device="cuda:0")[1:].view(rows, hid)
        odd.copy_(plan._in[n])
        plan._in[n] = odd
        plan.execute()
        torch.cuda.synchronize()
        assert np.allclose(plan._out[0].cpu().numpy(), got[0], rtol=1e-4, atol=1e-5)
    s.close()
