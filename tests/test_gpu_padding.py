"""Rows whose padding (up to the next 16 bytes) holds NaN, as uninitialised memory may: the
adjoint's staging must read every sample past the gradient's last one as zero, also those in
the 16-byte piece that holds the last one, in every kernel that loads rows into LDS."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _rows(x):
    nb, nr, n = x.shape
    buf = torch.full((nb, nr, (n + 3) // 4 * 4 + 4), float("nan"), device="cuda")
    buf[:, :, :n] = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return buf[:, :, :n]


@pytest.mark.parametrize("tail", [0, 1, 2, 3])
def test_adjoint_ignores_the_padding(tail):
    import paper_1601_01165_amd as dd

    nc, nd = 40, 33
    f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
    dms = np.arange(nd) * 0.05
    delta = oracle.delay_table(f, 50e-6, dms)
    plan = dd.Plan(f, 50e-6, dms)
    names = dd.variant_names("f32")
    rng = np.random.default_rng(tail)
    w = rng.uniform(0.5, 1.5, nc).astype(np.float32)
    ran = set()
    for ns in (tail or 4, 252 + tail, 508 + tail, 1280 + tail):
        nin = ns + int(delta.max()) + 2
        g = rng.standard_normal((2, nd, ns)).astype(np.float32)
        x = rng.standard_normal((2, nc, nin)).astype(np.float32)
        want = oracle.adjoint_gather_f32(g, delta, nin, w)
        ref, scale = oracle.grad_w(x, g, delta)
        gg, xg, wg = _rows(g), _rows(x), torch.from_numpy(w).cuda()
        untuned = dd.Plan(f, 50e-6, dms)
        for v in [None] + list(range(len(names))):
            p = untuned if v is None else plan
            if v is not None:
                try:
                    p.set_adjoint_variant(v)
                except dd.DedispError:
                    continue
            ran.add(v)
            gi, gw = dd.adjoint(gg, p, nin, wg, xg)
            assert np.array_equal(gi.cpu().numpy(), want), (ns, v, names[v] if v is not None else "untuned")
            assert (np.abs(gw.cpu().numpy() - ref) <= 1e-5 * scale + 1e-6 * np.abs(ref)).all(), (ns, v)
    assert {None, 44, 45, 46, 47, 48} <= ran
