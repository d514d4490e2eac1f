"""The kernel choice by size of untuned plans, and the kernels it chooses from
(lane kernels, wide register windows), against the oracle bit for bit: sizes one
either side of the tile edges, few and many rows, delay spans from narrow to
wider than the register windows.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _dd():
    import paper_1601_01165_amd as dd

    return dd


def _rows(x):
    t = _dd().empty_rows(*x.shape, torch.from_numpy(x[:0]).dtype, "cuda", zero=True)
    t.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return t


def _setup(nc, nd, step):
    f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
    dms = np.arange(nd) * step
    return f, dms, oracle.delay_table(f, 50e-6, dms)


@pytest.mark.parametrize("nc,nd,step", [(1, 1, 0.25), (9, 7, 0.25), (40, 70, 0.25), (17, 33, 4.0)])
@pytest.mark.parametrize("weighted", [False, True])
def test_forward_choice_by_size(nc, nd, step, weighted):
    dd = _dd()
    rng = np.random.default_rng(nc + nd)
    f, dms, delta = _setup(nc, nd, step)
    plan = dd.Plan(f, 50e-6, dms)
    w = rng.uniform(0.5, 1.5, nc).astype(np.float32) if weighted else None
    wg = torch.from_numpy(w).cuda() if weighted else None
    for nb, ns in [(1, 1), (2, 255), (1, 257), (1, 1281), (3, 4099)]:
        x = rng.standard_normal((nb, nc, ns + int(delta.max()))).astype(np.float32)
        got = dd.dedisperse(_rows(x), plan, wg, nsamp=ns).cpu().numpy()
        assert np.array_equal(got, oracle.forward_f32(x, delta, ns, w)), (nb, ns)


@pytest.mark.parametrize("nc,nd,step", [(5, 3, 0.25), (40, 70, 0.25), (60, 80, 0.5), (12, 90, 1.0), (33, 41, 4.0)])
def test_adjoint_choice_and_wide_spans(nc, nd, step):
    """The untuned adjoint at several sizes, then every variant that fits (the
    wide register windows and the lane kernels take spans the others refuse; the
    last two set-ups are too wide for any tile and run the direct kernel)."""
    dd = _dd()
    rng = np.random.default_rng(3 * nc + nd)
    f, dms, delta = _setup(nc, nd, step)
    w = rng.uniform(0.5, 1.5, nc).astype(np.float32)
    wg = torch.from_numpy(w).cuda()
    names = dd.variant_names("f32")
    plan = dd.Plan(f, 50e-6, dms)
    seen = set()
    for v in [None] + list(range(39, len(names))):
        try:
            if v is not None:
                plan.set_adjoint_variant(v)
        except dd.DedispError:
            continue
        seen.add(v)
        for nb, ns in [(1, 1), (2, 513), (1, 2051)]:
            nin = ns + int(delta.max()) + 3
            g = rng.standard_normal((nb, nd, ns)).astype(np.float32)
            x = rng.standard_normal((nb, nc, nin)).astype(np.float32)
            gi, gw = dd.adjoint(_rows(g), plan, nin, wg, _rows(x))
            assert np.array_equal(gi.cpu().numpy(), oracle.adjoint_gather_f32(g, delta, nin, w)), (v, nb, ns)
            ref, scale = oracle.grad_w(x, g, delta)
            assert (np.abs(gw.cpu().numpy() - ref) <= 1e-5 * scale + 1e-6 * np.abs(ref)).all(), (v, nb, ns)
    assert None in seen
    if (nc, nd) == (60, 80):
        assert {39, 40} <= seen, seen  # up to 17 samples between neighbouring channels


@pytest.mark.parametrize("nc,nd", [(3, 5), (40, 33), (300, 70)])
def test_u8_choice_by_size(nc, nd):
    dd = _dd()
    rng = np.random.default_rng(nc)
    f, dms, delta = _setup(nc, nd, 0.25)
    plan = dd.Plan(f, 50e-6, dms)
    for nb, ns in [(1, 1), (2, 511), (1, 1025), (3, 5003)]:
        x = rng.integers(0, 256, (nb, nc, ns + int(delta.max())), dtype=np.uint8)
        got = dd.dedisperse(_rows(x), plan, nsamp=ns).cpu().numpy()
        assert np.array_equal(got, oracle.forward_u8(x, delta, ns)), (nb, ns)
