"""Sums of partial rows by a wavefront each and by a workgroup each: both sides of the line between them, ends of a row that share a chunk,
more rows than are in flight."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,m,d,rows_per_run", [(2, 12, 1, 3_000, 5_001, None), (2, 12, 1, 3_000, 4, 3), (3, 4, 1, 4_000, 6_500, None), (3, 4, 1, 4_000, 5_001, None),
                                                    (3, 6, 2, 2_000, 20_003, None), (2, 12, 3, 2_000, 1_027, 4), (2, 4, 1, 900, 40_001, 9), (1, 12, 11, 700, 3_001, 2)])
def test_slabs_against_64_bits(L, n, s, m, d, rows_per_run):
    """Runs are rounded to fp32 once, sums are fp64: as in the other tests of stage 1, 3e-6 of a slab's rms per entry."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(m + d)
    X, w, y = (torch.randn(shape, generator=gen, device="cuda") for shape in ((m, d), (d,), (m,)))
    w /= d ** 0.5
    y += 4.0
    plan = cr.cr_plan_ex(L, n, s, m, d)
    if rows_per_run:
        cr.cr_plan_set_split(plan, cr.CR_SPLIT_ROWS_ONCE, rows_per_run)
    ws = cr.Workspace(plan)
    ws.slab_grads().fill_(float("nan"))
    cr.cr_partial_grads(plan, X, y, w)
    cr.cr_synchronize(plan)
    G = ws.slab_grads().double()
    rb, re_, _, _ = cr.cr_plan_get_segments(plan)
    contribution = (X.double() @ w.double() - y.double())[:, None] * X.double()
    for lo, hi in sorted(set(zip(rb.tolist(), re_.tolist()))):
        ref = contribution[lo:hi].sum(0)
        for q in np.flatnonzero((rb == lo) & (re_ == hi)):
            assert float((G[q] - ref).abs().max() / ref.pow(2).mean().sqrt()) <= 3e-6, (lo, hi, q)
    again = ws.slab_grads().clone()
    cr.cr_partial_grads(plan, X, y, w)
    cr.cr_synchronize(plan)
    assert torch.equal(again, ws.slab_grads())
    del ws
    cr.cr_plan_destroy(plan)
