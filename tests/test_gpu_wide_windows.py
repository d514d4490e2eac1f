"""Untuned calls on plans with 8 to 12 samples between neighbouring rows, whose default is a
wide window: the calls of few blocks and rows go to tiles of 16 rows, the others stay.
Forward, weighted and adjoint bit-identical to the oracle, at the edges of the tiles."""
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


# DM step 0.55: 7.6 to 9.8 samples between the trials in the lowest channels; channels of
# 60 MHz / nc at 100 pc/cm^3: as many between the channels for the gradient
@pytest.mark.parametrize("nbeam,nc,nd,ns,step", [(8, 20, 256, 2305, 0.55), (1, 20, 17, 769, 0.55), (3, 33, 49, 1281, 0.55),
                                                 (1, 8, 400, 5121, 0.6), (2, 24, 40, 3000, 1.2), (1, 9, 65, 513, 0.5)])
def test_wide_windows(nbeam, nc, nd, ns, step):
    import paper_1601_01165_amd as dd

    f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
    dms = np.arange(nd) * step
    delta = oracle.delay_table(f, 50e-6, dms)
    plan = dd.Plan(f, 50e-6, dms)
    rng = np.random.default_rng(ns)
    w = rng.uniform(0.5, 1.5, nc).astype(np.float32)
    wg = torch.from_numpy(w).cuda()
    nin = ns + int(delta.max())
    x = rng.standard_normal((nbeam, nc, nin)).astype(np.float32)
    g = rng.standard_normal((nbeam, nd, ns)).astype(np.float32)
    for wh, wt in ((None, None), (w, wg)):
        got = dd.dedisperse(_rows(x), plan, wt, nsamp=ns).cpu().numpy()
        assert np.array_equal(got, oracle.forward_f32(x, delta, ns, wh))
        gi, gw = dd.adjoint(_rows(g), plan, nin, wt, _rows(x))
        assert np.array_equal(gi.cpu().numpy(), oracle.adjoint_gather_f32(g, delta, nin, wh))
        ref, scale = oracle.grad_w(x, g, delta)
        assert (np.abs(gw.cpu().numpy() - ref) <= 1e-5 * scale + 1e-6 * np.abs(ref)).all()
