"""The workspace of the single-pulse search: one sized for the longest call of a
pipeline serves every shorter one.  Sizes lie either side of the lines where the search
changes its path: the small uint8 tiles (fewer blocks than CUs), the groups of
float32 beams, and float32 beams whose series alone are larger than the groups."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _dd():
    import paper_1601_01165_amd as dd

    return dd


def _plan(nc, nd, step):
    f = 1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc
    return _dd().Plan(f, 50e-6, np.arange(nd) * step)


def _detect(plan, x, ns, ws_bytes):
    """dedisp_detect through the C-ABI with a workspace of exactly ws_bytes."""
    dd = _dd()
    L = dd.lib()
    nb = x.shape[0]
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    o = {"snr": torch.empty((nb, plan.ndm), dtype=torch.float64, device="cuda"),
         "width": torch.empty((nb, plan.ndm), dtype=torch.int32, device="cuda"),
         "start": torch.empty((nb, plan.ndm), dtype=torch.int32, device="cuda")}
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    st = L.dedisp_detect(plan.handle, nb, ns, p(x), 1 if x.dtype == torch.uint8 else 0, x.stride(1), None, 6, p(o["snr"]),
                         p(o["width"]), p(o["start"]), None, None, p(ws), ws_bytes, None)
    torch.cuda.synchronize()
    assert st == 0, (ns, ws_bytes, L.dedisp_last_error())
    return o


def _same(got, want):
    for k in ("width", "start"):
        assert torch.equal(got[k], want[k]), k
    assert torch.allclose(got["snr"], want["snr"], rtol=1e-10, atol=1e-12)  # one-pass FP64 moments


@pytest.mark.parametrize("u8,nc,nd", [(True, 16, 256), (True, 16, 33), (True, 1100, 40), (False, 128, 2048),
                                      (False, 128, 30), (False, 16, 300), (False, 16, 2048)])
def test_size_grows_with_the_call(u8, nc, nd):
    """Up to the series that fit one group, the size asked for never falls as beams or samples grow."""
    L, plan = _dd().lib(), _plan(nc, nd, 0.05)
    beams = [1, 2, 3, 7, 8, 40]
    most = min(1000000, (1 << 28) // nd - 4)  # 1 GiB of series per beam
    sizes = sorted({1, 3, 991, 992, 993, 18700, 20000, 30752, 31744, 31745} | set(range(1, most, most // 97)))
    asked = np.array([[L.dedisp_detect_workspace_bytes(plan.handle, int(u8), nb, ns) for ns in sizes] for nb in beams])
    assert (asked > 0).all()
    assert (np.diff(asked, axis=0) >= 0).all() and (np.diff(asked, axis=1) >= 0).all()


@pytest.mark.parametrize("nb,long,short", [(1, 31744, (30752, 20000, 993, 992, 1)), (3, 12000, (10900, 4000))])
def test_u8_shorter_calls(nb, long, short):
    dd, plan = _dd(), _plan(16, 256, 0.05)
    x = dd.empty_rows(nb, 16, long + plan.max_delay, torch.uint8, "cuda")
    x.copy_(torch.randint(0, 256, x.shape, device="cuda", dtype=torch.uint8))
    ws = dd.lib().dedisp_detect_workspace_bytes(plan.handle, 1, nb, long)
    for ns in (long, *short):
        _same(_detect(plan, x, ns, ws), dd.detect(x, plan, nsamp=ns))


@pytest.mark.parametrize("nb,long,short", [(8, 20000, (18700, 900)), (1, 140000, (130000, 100000, 1))])
def test_f32_shorter_calls(nb, long, short):
    """8 beams of 2048 DM trials go through in groups; one of 140,000 samples has more than 1 GiB of series."""
    dd, plan = _dd(), _plan(128, 2048, 0.01)
    x = dd.empty_rows(nb, 128, long + plan.max_delay, torch.float32, "cuda")
    x.copy_(torch.randint(-3, 4, x.shape, device="cuda"))  # sums are exact in either path
    ws = dd.lib().dedisp_detect_workspace_bytes(plan.handle, 0, nb, long)
    for ns in (long, *short):
        got = _detect(plan, x, ns, ws)
        _same(got, dd.detect(x, plan, nsamp=ns))
        # the binding takes a workspace that the call can run with, and makes another for one that it cannot
        mine = torch.empty(ws, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        _same(dd.detect(x, plan, nsamp=ns, workspace=mine), got)
        assert torch.cuda.max_memory_allocated() - before < 1 << 22
        _same(dd.detect(x, plan, nsamp=ns, workspace=mine[:16]), got)


@pytest.mark.parametrize("nd", [300, 2048])
def test_f32_few_channels(nd):
    """On few channels large calls are searched in place: they run with room for the records alone (64
    bytes per series and tile of at least 1000 samples), and so do the shorter ones."""
    dd, plan = _dd(), _plan(16, nd, 0.01)
    long = 60000000 // nd // 3
    x = dd.empty_rows(3, 16, long + plan.max_delay, torch.float32, "cuda")
    x.copy_(torch.randint(-3, 4, x.shape, device="cuda"))
    plain = _plan(16, nd, 0.01)
    plain.set_detect_variant(-1)
    for ns in (long, long // 14, long // 15, 100, 1):
        got = _detect(plan, x, ns, 3 * nd * (long // 1000 + 1) * 64)
        _same(got, dd.detect(x, plan, nsamp=ns))
        _same(got, dd.detect(x, plain, nsamp=ns))


def test_autotune_times_every_fused_variant_of_a_large_call():
    """512 beams of 1024 DM trials x 16,000 samples: the records of the small tiles take more than
    the series of one group (1 GiB), and every variant that fits is timed all the same."""
    dd, plan = _dd(), _plan(2, 1024, 0.05)
    names, fit = dd.variant_names("u8"), set()
    for i, name in enumerate(names):
        try:
            plan.set_detect_variant(i, "u8")
            fit.add(name)
        except dd.DedispError:
            pass
    assert len(fit) > 10
    times = plan.autotune_detect(512, 16000, "u8")
    assert set(times) == fit | {"unfused"}


@pytest.mark.parametrize("nd", [12, 49, 97])
def test_f32_few_channels_few_dms(nd):
    """Spans of 10 samples between trials, which only tiles of 48 DM trials take: fewer than two of them are
    stored and searched, more searched in place; both give the same."""
    dd = _dd()
    f = 1270.0 + (np.arange(45) + 0.5) * 300.0 / 45
    dms = np.arange(nd) * 0.6
    plan, plain = dd.Plan(f, 50e-6, dms), dd.Plan(f, 50e-6, dms)
    ns = 9000000 // nd  # 36 MB of series
    x = dd.empty_rows(1, 45, ns + plan.max_delay, torch.float32, "cuda")
    x.copy_(torch.randint(-3, 4, x.shape, device="cuda"))
    plain.set_detect_variant(-1)
    for n in (ns, ns // 3):
        _same(dd.detect(x, plan, nsamp=n), dd.detect(x, plain, nsamp=n))
