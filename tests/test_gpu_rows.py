"""The search over stored rows against the oracle: row lengths around the tile
edges, row counts that give a wave one tile or several, and both sides of the line
between one block per row and records merged by a second kernel.  The data are small
integers, so every window sum is exact and ties are common: widths, first starts
and S/N must match (S/N, mean and std to 1e-10: one-pass FP64 moments)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrows,ns", [(1, 1), (5, 31), (7, 991), (7, 992), (7, 993), (9, 1024), (3, 2977),
                                      (6000, 2977), (5500, 1985), (255, 31744), (255, 31745), (256, 31744),
                                      (256, 31745), (3, 126976), (3, 126977)])
@pytest.mark.parametrize("dtype", ["f32", "i32"])
def test_rows_groups_and_ties(nrows, ns, dtype):
    import paper_1601_01165_amd as dd

    rng = np.random.default_rng(nrows + ns)
    x = rng.integers(-3, 4, (nrows, ns)).astype(np.float32 if dtype == "f32" else np.int32)
    x[0] = 2  # constant: S/N 0, width 1, start 0
    got = {k: v.cpu().numpy() for k, v in dd.detect_rows(torch.from_numpy(x).cuda()).items()}
    pick = np.unique(np.concatenate([np.arange(min(nrows, 8)), rng.integers(0, nrows, 40)]))
    want = oracle.detect(x[pick].astype(np.float64), 6)
    assert np.array_equal(got["width"][pick], want["width"])
    assert np.array_equal(got["start"][pick], want["start"])
    for k in ("snr", "mean", "std"):
        assert np.allclose(got[k][pick], want[k], rtol=1e-10, atol=1e-12), k
