"""Which path the search takes and its records.  The uint8 search's records, reduced over the lanes for four rows at once while a
window's sum and its start fit 31 bits together: channel counts on both sides of that
limit for each run length (127/128 with 32 samples per lane, 256/257 with 16), rows
saturated for longer than a window so that the largest possible sum occurs and ties, and
row counts that leave a group of rows partly filled.  Sums are exact integers: widths and
first starts must match the oracle's (S/N, mean and std to 1e-10: one-pass FP64
moments)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nchan,ndm", [(127, 6), (128, 5), (256, 7), (257, 1), (257, 9)])
def test_u8_records_of_saturated_rows(nchan, ndm):
    import paper_1601_01165_amd as dd

    ns = 2100
    freqs = 1300.0 + np.arange(nchan) * (200.0 / nchan)
    dms = np.arange(ndm) * 0.5
    delta = oracle.delay_table(freqs, 1e-4, dms)
    rng = np.random.default_rng(nchan + ndm)
    x = rng.integers(0, 40, (1, nchan, ns + int(delta.max()))).astype(np.uint8)
    x[:, :, 1003:1060] = 255
    rows = oracle.forward_u8(x, delta, ns)
    want = oracle.detect(rows, 6)
    g = dd.empty_rows(*x.shape, dtype=torch.uint8, zero=True)
    g.copy_(torch.from_numpy(x))
    plan = dd.Plan(freqs, 1e-4, dms)
    ran = 0
    for i, name in enumerate(dd.variant_names("u8")):
        try:
            plan.set_detect_variant(i, "u8")
        except dd.DedispError:
            continue
        ran += 1
        got = {k: v.cpu().numpy() for k, v in dd.detect(g, plan, nsamp=ns).items()}
        assert np.array_equal(got["width"], want["width"]), name
        assert np.array_equal(got["start"], want["start"]), name
        for k in ("snr", "mean", "std"):
            assert np.allclose(got[k], want[k], rtol=1e-10, atol=1e-12), (name, k)
    assert ran >= 4


@pytest.mark.parametrize("nsamp", [4194000, 4194400])
def test_f32_long_series_are_searched_in_place(nsamp):
    """64 series on both sides of 1 GiB (4,194,304 samples each): stored and searched
    below, searched in the tile kernel above, so that the workspace stays small.  Both
    sum windows by the same doublings: the same widths and starts, moments to rounding."""
    import paper_1601_01165_amd as dd

    plan = dd.Plan(1300.0 + 12.5 * np.arange(8), 1e-4, np.arange(64) * 0.5)
    x = dd.empty_rows(1, 8, nsamp + plan.max_delay)
    x.normal_(generator=torch.Generator("cuda").manual_seed(nsamp))
    x[0, :, 3000000:3000016] += 1.0
    small = dd.lib().dedisp_detect_workspace_bytes(plan.handle, 0, 1, nsamp) < 1 << 29
    assert small == (nsamp > 4194304)
    got = dd.detect(x, plan, nsamp=nsamp)
    plan.set_detect_variant(-1)
    want = dd.detect(x, plan, nsamp=nsamp)
    for k in ("width", "start"):
        assert torch.equal(got[k], want[k]), k
    for k in ("snr", "mean", "std"):
        assert torch.allclose(got[k], want[k], rtol=1e-9, atol=1e-9), k
