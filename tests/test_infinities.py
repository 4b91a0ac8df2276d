"""An infinite entry of X reaches its own column of the slabs and no other with the logistic model, since sigmoid(+-inf) is 0 or 1: wherever in
the row it lies, for every shape of stage 1 that forms a row once, under every split that uses them."""
import pytest

import paper_1902_01981_amd as cr

# one column per lane, parts of a wavefront, a wavefront, teams of two to eight; rows that fill their lanes and rows that do not, ends that
# overlap the chunk before; weights in LDS; two passes
SHAPES = [(3, 0), (7, 1), (10, 0), (100, 0), (104, 1), (257, 1), (512, 1), (600, 0), (1_023, 0), (1_024, 1), (1_027, 1), (2_047, 1), (2_048, 0), (3_001, 0),
          (4_096, 0), (4_099, 1), (5_001, 0), (12_289, 0), (16_387, 1), (24_575, 0), (172_033, 1)]


def _check(d, bf16, m, s, split):
    import torch

    gen = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(m, d, generator=gen, device="cuda").to(torch.bfloat16 if bf16 else torch.float32)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.full((m,), 0.25, device="cuda")
    cols = sorted({0, d // 2} | {max(0, d - 1 - i) for i in range(10)})
    for i, c in enumerate(cols):                         # rows far apart, so that other rows are in hand beside them
        X[i * (m // len(cols)), c] = torch.copysign(torch.tensor(float("inf")), w[c].cpu() * (1 if i % 3 else -1))
    plan = cr.cr_plan_ex(1, 3, s, m, d, model=cr.CR_LOGISTIC, x_dtype=bf16)
    if split:
        cr.cr_plan_set_split(plan, *split)
    ws = cr.Workspace(plan)
    cr.cr_partial_grads(plan, X, y, w)
    cr.cr_synchronize(plan)
    rb, re_, _, _ = cr.cr_plan_get_segments(plan)
    for q in range(len(rb)):
        x = X[int(rb[q]):int(re_[q])].double()
        res = torch.sigmoid(x @ w.double()) - 0.25
        got, whole = ws.slab_grads()[q].double(), torch.isfinite(x).all(0)
        assert torch.equal(torch.isfinite(got), whole)
        ref = x.nan_to_num(posinf=0.0, neginf=0.0).T @ res
        assert float(((got - ref)[whole]).abs().max() / ref[whole].pow(2).mean().sqrt()) <= 3e-6      # as for finite data
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16", SHAPES)
@pytest.mark.parametrize("m,split", [(150, None), (1_000, (cr.CR_SPLIT_ROWS_ONCE, 37)), (40, None)])
def test_rows_once(d, bf16, m, split):
    _check(d, bf16, m, 1, split)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16,m", [(30_001, 0, 1_200), (36_861, 1, 1_400)])
def test_weights_in_lds(d, bf16, m):
    _check(d, bf16, m, 1, None)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [1_027, 2_048, 5_001, 12_287])
def test_shared_cells_and_equal_ranges(d):
    _check(d, 0, 600, 1, (cr.CR_SPLIT_SHARED_CELLS, 64))
    _check(d, 0, 600, 0, (cr.CR_SPLIT_EQUAL_RANGES, 31))


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16", [(10, 0), (100, 0), (100, 1), (1_027, 1), (3_001, 0)])
def test_whole_ranges(d, bf16):
    _check(d, bf16, 300, 1, (cr.CR_SPLIT_ROWS_ONCE, cr.CR_ROWS_WHOLE_RANGES))
