"""empty_rows takes what torch.empty takes as a dtype; rows start on 16-byte boundaries."""
import pytest
import torch

import paper_1601_01165_amd as dd


@pytest.mark.parametrize("dtype,want", [(torch.float32, torch.float32), (torch.uint8, torch.uint8), (None, torch.float32),
                                        (float, torch.float64), (int, torch.int64), (bool, torch.bool)])
@pytest.mark.parametrize("n", [1, 4, 15, 16, 17])
def test_empty_rows_dtypes(dtype, want, n):
    t = dd.empty_rows(2, 3, n, dtype, "cpu", zero=True)
    assert t.dtype == want and tuple(t.shape) == (2, 3, n)
    assert t.stride(2) == 1 and t.stride(1) * t.element_size() % 16 == 0 and t.stride(0) == 3 * t.stride(1)
    assert not t.any()
