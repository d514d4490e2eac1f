"""Device memory of a plan's tile tables: what a plan no longer uses is given back, what
its next call needs is kept."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _plan(nc, nd):
    import paper_1601_01165_amd as dd

    return dd.Plan(1270.0 + (np.arange(nc) + 0.5) * 300.0 / nc, 50e-6, np.arange(nd) * 0.25)


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_dropped_tables_are_given_back():
    """A plan of 1024 channels x 2048 DM trials holds the tables of five variants or so (8 MB each) for its
    choice by size; once it is set to one variant, a batch on it drops the others."""
    import paper_1601_01165_amd as dd

    plan = _plan(1024, 2048)
    x = dd.empty_rows(1, 1024, 64 + plan.max_delay, torch.float32, "cuda", zero=True)
    out = dd.empty_rows(1, 2048, 64, torch.float32, "cuda")
    plan.set_variant(plan.variant("f32"))
    before = _free()
    batch = dd.Batch([plan], [x], [out])
    assert _free() - before > 20 * MB
    batch.execute()
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["u8", "f32"])
def test_search_tables_outlive_tuning(dtype):
    """The automatic search keeps the tables of the variants it runs when the tuner of the forward map drops
    what it timed: the next search allocates nothing."""
    import paper_1601_01165_amd as dd

    nc = 256 if dtype == "u8" else 32  # few channels: large float32 calls are searched in place
    plan = _plan(nc, 2048)
    ns = 6000
    x = dd.empty_rows(1, nc, ns + plan.max_delay, torch.uint8 if dtype == "u8" else torch.float32, "cuda", zero=True)
    dd.detect(x, plan, nsamp=ns)
    plan.autotune(1, ns, dtype)
    dd.detect(x, plan, nsamp=ns)  # (torch's allocator holds the outputs and the workspace from here on)
    plan.autotune(1, ns, dtype)
    before = _free()
    dd.detect(x, plan, nsamp=ns)
    assert before - _free() < 1 * MB
