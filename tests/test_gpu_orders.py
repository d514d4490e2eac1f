"""DM lists and channels in any order: untuned plans take the kernels that branch per
row on regular ascending lists, and those that branch per DM slot on lists whose rows
mostly follow no pattern, forward, backward and batched, bit-identical to the oracle
(float32 sums in channel order) either way."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _dd():
    import paper_1601_01165_amd as dd

    return dd


def _rows(x):
    t = _dd().empty_rows(*x.shape, torch.float32, "cuda")
    t.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return t


def _dms(order, nd, step):
    d = np.arange(nd) * step
    rng = np.random.default_rng(nd)
    if order == "desc":
        return d[::-1].copy()
    if order == "fours":  # shuffled within the rows of a wave
        return rng.permuted(d.reshape(-1, 4), axis=1).ravel()
    if order == "uneven":
        return np.sort(d + rng.uniform(-0.4, 0.4, nd) * step).clip(0)
    return d


def _slots(i):
    return _dd().variant_names("f32")[i].endswith("_slots")


@pytest.mark.parametrize("order,slots", [("asc", False), ("desc", True), ("fours", True), ("uneven", True)])
@pytest.mark.parametrize("fdesc", [False, True])
def test_forward(order, slots, fdesc):
    dd = _dd()
    f = 1270.0 + (np.arange(31) + 0.5) * 300.0 / 31
    f = f[::-1].copy() if fdesc else f
    dms = _dms(order, 196, 0.25)
    delta = oracle.delay_table(f, 50e-6, dms)
    plan = dd.Plan(f, 50e-6, dms)
    assert _slots(plan.variant("f32")) == slots
    rng = np.random.default_rng(5)
    for nb, ns in [(1, 100), (2, 5003), (40, 8000)]:  # lane, middle and coarse tiles
        x = rng.standard_normal((nb, 31, ns + int(delta.max()))).astype(np.float32)
        got = dd.dedisperse(_rows(x), plan, nsamp=ns).cpu().numpy()
        pick = [0, nb - 1]
        assert np.array_equal(got[pick], oracle.forward_f32(x[pick], delta, ns)), (nb, ns)


@pytest.mark.parametrize("fdesc", [False, True])
@pytest.mark.parametrize("order", ["asc", "desc"])
def test_adjoint(order, fdesc):
    dd = _dd()
    nc, nd = 70, 41
    f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
    f = f[::-1].copy() if fdesc else f
    dms = _dms(order, nd, 0.1)
    delta = oracle.delay_table(f, 50e-6, dms)
    plan = dd.Plan(f, 50e-6, dms)
    # output rows are channels here: descending frequencies make their delays descend
    assert _slots(plan.adjoint_variant()) == fdesc
    rng = np.random.default_rng(6)
    for nb, ns in [(1, 100), (40, 20003)]:
        nin = ns + int(delta.max())
        g = rng.standard_normal((nb, nd, ns)).astype(np.float32)
        gi, _ = dd.adjoint(_rows(g), plan, nin)
        pick = [0, nb - 1]
        assert np.array_equal(gi[pick].cpu().numpy(), oracle.adjoint_gather_f32(g[pick], delta, nin)), (nb, ns)


@pytest.mark.parametrize("order,slots", [("asc", False), ("desc", True)])
def test_batch(order, slots):
    dd = _dd()
    rng = np.random.default_rng(7)
    plans, xs, outs, want = [], [], [], []
    for nc, nd, ns in [(20, 60, 1500), (33, 128, 2600)]:
        f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
        dms = _dms(order, nd, 0.25)
        delta = oracle.delay_table(f, 50e-6, dms)
        x = rng.standard_normal((1, nc, ns + int(delta.max()))).astype(np.float32)
        plans.append(dd.Plan(f, 50e-6, dms))
        xs.append(_rows(x))
        outs.append(dd.empty_rows(1, nd, ns, torch.float32, "cuda"))
        want.append(oracle.forward_f32(x, delta, ns))
    b = dd.Batch(plans, xs, outs)
    assert _slots(b.variant) == slots
    b.execute()
    torch.cuda.synchronize()
    for o, w in zip(outs, want):
        assert np.array_equal(o.cpu().numpy(), w)
