"""Rows of more than 24 576 columns: one pass with the weights in LDS, two passes, and the rules between them."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

# one pass (48 MB of X and more): the fewest and most chunks per thread of each type and one column on, rows that end in a whole chunk, an
# overlapping one, a chunk of one column; two passes: the same sizes with too few rows, wider rows with 1, 2, 4 and 8 rows per workgroup
CASES = [(24_577, 0, 600), (26_624, 0, 500), (26_625, 0, 480), (30_003, 0, 700), (32_768, 0, 400), (32_769, 0, 400), (34_816, 0, 367), (34_817, 0, 450),
         (24_577, 1, 1_100), (28_672, 1, 900), (28_673, 1, 900), (32_768, 1, 780), (32_777, 1, 800), (36_864, 1, 700), (36_865, 1, 900),
         (24_577, 0, 300), (36_861, 1, 200), (40_000, 0, 13), (40_003, 1, 451), (40_001, 0, 897), (37_002, 1, 1_801), (36_866, 1, 3_601)]


@pytest.mark.parametrize("d,bf16,m,one_pass", [(30_001, 0, 3_000, True), (36_864, 1, 700, True), (30_001, 0, 300, False), (36_865, 1, 900, False)])
def test_what_a_plan_reports_is_the_same_work_when_set(d, bf16, m, one_pass):
    p, q, r = (cr.cr_plan_ex(2, 4, 1, m, d, x_dtype=bf16) for _ in range(3))
    size, info = cr.cr_workspace_bytes(p), cr.cr_plan_info(p)
    cr.cr_plan_set_split(q, info.split_kind, info.split_value)
    assert cr.cr_workspace_bytes(q) == size and all(np.array_equal(a, b) for a, b in zip(cr.cr_plan_get_pieces(p), cr.cr_plan_get_pieces(q)))
    assert (info.split_kind, info.stage1_team_size) == (cr.CR_SPLIT_ROWS_ONCE, 0) and (info.split_value < m) == one_pass
    cr.cr_plan_set_split(r, cr.CR_SPLIT_ROWS_ONCE, m)    # no limit: two passes, long parts
    assert (cr.cr_plan_info(r).num_teams < info.num_teams) == one_pass
    for plan in (p, q, r):
        cr.cr_plan_destroy(plan)


@pytest.mark.parametrize("L,n,s,m,one_pass", [(3, 3, 2, 874, True), (2, 12, 1, 712, False), (2, 12, 1, 2_845, True), (3, 6, 2, 1_423, False), (3, 6, 2, 8_000, True)])
def test_one_pass_where_the_partial_rows_allow_it(L, n, s, m, one_pass):
    """Many slabs cut the parts of one pass into many runs; below some size of X the second pass costs less."""
    p, q = (cr.cr_plan_ex(L, n, s, m, 36_864, x_dtype=1) for _ in range(2))
    cr.cr_workspace_bytes(p)
    info = cr.cr_plan_info(p)
    assert (info.split_value < m) == one_pass
    cr.cr_plan_set_split(q, info.split_kind, info.split_value)
    assert cr.cr_workspace_bytes(q) == cr.cr_workspace_bytes(p) and all(np.array_equal(a, b) for a, b in zip(cr.cr_plan_get_pieces(p), cr.cr_plan_get_pieces(q)))
    for plan in (p, q):
        cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,d,bf16,m", [(3, 3, 2, 30_001, 1, 874), (2, 12, 5, 34_816, 0, 452), (2, 12, 3, 36_864, 1, 1_400)])
def test_runs_that_many_slabs_take(L, n, s, d, bf16, m):
    """Up to 36 workers hold the same rows: their slabs of one pass against those of two, bit for bit where a run makes up the slab, and
    every one of them written."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(d + m)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_(generator=gen)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.randn(m, generator=gen, device="cuda") + 4.0
    slabs = []
    for rows in (None, m):
        plan = cr.cr_plan_ex(L, n, s, m, d, x_dtype=bf16)
        if rows:
            cr.cr_plan_set_split(plan, cr.CR_SPLIT_ROWS_ONCE, rows)
        ws = cr.Workspace(plan)
        assert (ws.info.split_value < m) == (rows is None)
        ws.slab_grads().fill_(float("nan"))
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_synchronize(plan)
        slabs.append(ws.slab_grads().double())
        del ws
        cr.cr_plan_destroy(plan)
    one, two = slabs
    assert float(((one - two).abs().amax(1) / two.pow(2).mean(1).sqrt()).max()) <= 6e-6       # each within 3e-6 of 64 bits


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16,m", CASES)
def test_slabs_against_64_bits(d, bf16, m):
    """The dot product and the residual are fp32 (some 1e-7 of the sum of magnitudes, which is about one here), everything across rows
    fp64: 3e-6 of a slab's rms per entry leaves room for the few rows with a residual much smaller than one."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(d + m)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_(generator=gen)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.randn(m, generator=gen, device="cuda") + 4.0           # residuals away from zero
    for logistic, rows_per_run in ((0, None), (1, None), (0, 1), (0, m)):         # m: two passes for all sizes
        plan = cr.cr_plan_ex(1, 3, 1, m, d, model=logistic, x_dtype=bf16)
        if rows_per_run:
            cr.cr_plan_set_split(plan, cr.CR_SPLIT_ROWS_ONCE, rows_per_run)
        ws = cr.Workspace(plan)
        ws.slab_grads().fill_(float("nan"))
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_synchronize(plan)
        G = ws.slab_grads().double()
        rb, re_, _, _ = cr.cr_plan_get_segments(plan)
        for q in range(len(rb)):
            x = X[int(rb[q]):int(re_[q])].double()
            z = x @ w.double()
            ref = x.T @ ((torch.sigmoid(z) if logistic else z) - y[int(rb[q]):int(re_[q])].double())
            assert float((G[q] - ref).abs().max() / ref.pow(2).mean().sqrt()) <= 3e-6, (d, q)
        again = ws.slab_grads().clone()
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_synchronize(plan)
        assert torch.equal(again, ws.slab_grads())
        del ws
        cr.cr_plan_destroy(plan)
