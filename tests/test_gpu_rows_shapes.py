"""The search over stored rows where its launches change shape: rows of one tile, one
wave or four per row, one launch or two, and more rows than four waves each can
be launched for (2^32 work items).  The data are small integers, so widths and first
starts must match the oracle, S/N to 1e-10 (one-pass FP64 moments)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _check(x, pick):
    import paper_1601_01165_amd as dd

    got = {k: v[pick].cpu().numpy() for k, v in dd.detect_rows(x).items()}
    want = oracle.detect(x[pick].cpu().numpy().astype(np.float64), 6)
    for k in ("width", "start"):
        assert np.array_equal(got[k], want[k]), k
    for k in ("snr", "mean", "std"):
        assert np.allclose(got[k], want[k], rtol=1e-10, atol=1e-12), k


# rows of 1, 2, 3, 4, 12, 13, 32 and 33 tiles of 992 starts, either side of 192 and 4096 rows
@pytest.mark.parametrize("nrows,tiles", [(3, 1), (4100, 1), (191, 2), (4095, 3), (4096, 2), (4096, 3), (4096, 4),
                                         (191, 12), (191, 13), (192, 13), (192, 32), (192, 33)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.int32])
def test_row_launch_shapes(nrows, tiles, dtype):
    torch.manual_seed(nrows + tiles)
    x = torch.randint(-3, 4, (nrows, 992 * tiles - 1), device="cuda").to(dtype)
    rng = np.random.default_rng(nrows)
    _check(x, np.unique(np.concatenate([[0, nrows - 1], rng.integers(0, nrows, 30)])))


def test_more_rows_than_four_waves_each():
    n = (1 << 24) + 3
    torch.manual_seed(1)
    x = torch.randint(-3, 4, (n, 4), device="cuda", dtype=torch.int32)
    rng = np.random.default_rng(2)
    _check(x, np.unique(np.concatenate([[0, 1, n - 4, n - 3, n - 2, n - 1], rng.integers(0, n, 500)])))
