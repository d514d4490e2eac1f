"""Untuned calls that leave the GPU nearly idle, on plans whose delay spans no finely
tiled kernel but the wide lane tiles takes, and of so few rows that the direct kernel is
taken: forward and adjoint bit-identical to the oracle, the allocation-free adjoint
to the one with a workspace."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _rows(x):
    import paper_1601_01165_amd as dd

    t = dd.empty_rows(*x.shape, torch.float32, "cuda")
    t.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return t


# the direct kernel (a few rows), the wide lane tiles (the adjoint's spans fit the wide windows, no
# narrower lane kernel), and a plan that no tile fits
@pytest.mark.parametrize("nc,nd,ns,band", [(9, 14, 500, "lofar"), (18, 12, 2387, "lofar"), (30, 102, 1728, "l"),
                                           (28, 99, 4001, "l"), (4, 3, 37, "l"), (23, 9, 493, "lofar"), (60, 40, 301, "p")])
def test_small_calls(nc, nd, ns, band):
    import paper_1601_01165_amd as dd

    lo, hi, ts, step = {"l": (1270.0, 1570.0, 50e-6, 0.25), "lofar": (134.875, 141.125, 5e-6, 0.01),
                        "p": (300.0, 400.0, 50e-6, 2.0)}[band]
    f = lo + (np.arange(nc) + 0.5) * (hi - lo) / nc
    dms = np.arange(nd) * step
    delta = oracle.delay_table(f, ts, dms)
    plan = dd.Plan(f, ts, dms)
    plan.prepare("f32", adjoint=True)
    rng = np.random.default_rng(nc)
    w = rng.uniform(0.5, 1.5, nc).astype(np.float32)
    wg = torch.from_numpy(w).cuda()
    nin = ns + int(delta.max())
    x = rng.standard_normal((2, nc, nin)).astype(np.float32)
    g = rng.standard_normal((2, nd, ns)).astype(np.float32)
    for wh, wt in ((None, None), (w, wg)):
        got = dd.dedisperse(_rows(x), plan, wt, nsamp=ns).cpu().numpy()
        assert np.array_equal(got, oracle.forward_f32(x, delta, ns, wh))
        gi, gw = dd.adjoint(_rows(g), plan, nin, wt, _rows(x))
        assert np.array_equal(gi.cpu().numpy(), oracle.adjoint_gather_f32(g, delta, nin, wh))
        ref, scale = oracle.grad_w(x, g, delta)
        assert (np.abs(gw.cpu().numpy() - ref) <= 1e-5 * scale + 1e-6 * np.abs(ref)).all()
        gi2 = dd.empty_rows(2, nc, nin, torch.float32, "cuda")
        gw2 = torch.empty(nc, device="cuda")
        dd.adjoint_noalloc(_rows(g), plan, nin, wt, _rows(x), gi2, gw2)
        assert torch.equal(gi2, gi) and torch.equal(gw2, gw)
