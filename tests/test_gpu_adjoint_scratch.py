"""The allocation-free adjoint where the short tiles that a call of few channels
takes would need more partial sums than the fixed scratch holds: the call runs with
the longer tiles, and gives the bits of the adjoint with a workspace."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_few_channels_long_rows():
    import paper_1601_01165_amd as dd

    nb, nc, ns = 3, 8, 12_000_000
    f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
    plan = dd.Plan(f, 50e-6, np.array([0.0, 0.02]))
    plan.prepare("f32", adjoint=True)
    delta = torch.from_numpy(plan.delays().astype(np.int64)).cuda()
    nin = ns + plan.max_delay
    torch.manual_seed(7)
    g = dd.empty_rows(nb, 2, ns, torch.float32, "cuda").normal_()
    x = dd.empty_rows(nb, nc, nin, torch.float32, "cuda").normal_()
    gw = torch.empty(nc, device="cuda")
    assert dd.lib().dedisp_adjoint_noalloc_bytes(plan.handle, nb, nin) <= 8 << 20
    dd.adjoint_noalloc(g, plan, nin, x=x, grad_w=gw)
    _, want = dd.adjoint(g, plan, nin, x=x, want_grad_in=False)
    assert torch.equal(gw, want)
    # and the definition, sum over beams, DM trials and samples of g x, in FP64: the sums of two
    # terms and of the products round at 2^-24 and 2^-53
    for c in range(nc):
        ref = scale = 0.0
        for b in range(nb):
            for j in range(2):
                d = int(delta[j, c])
                prod = g[b, j].double() * x[b, c, d:d + ns].double()
                ref += float(prod.sum())
                scale += float(prod.abs().sum())
        assert abs(float(gw[c]) - ref) <= 2.0 ** -22 * scale
