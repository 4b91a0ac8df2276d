"""Stage 1 with every row once where a workgroup's part holds several runs and a run several steps with a remainder: the borders at which
the two register sets change hands, a run's sums are put away and the next run's rows are on their way."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr
from _harness import assert_close

# one width per kernel: lanes that share a row (2 to 64), chunks per lane, threads per row, chunks per thread, steps of 4, 2 and 1 rows, with
# and without the next step's rows under way; rows in two passes
WIDTHS = [(3, 0), (8, 0), (13, 0), (30, 0), (64, 0), (100, 0), (255, 0), (400, 0), (700, 0), (1_000, 0), (1_300, 0), (1_999, 0), (2_600, 0), (4_096, 0), (5_001, 0),
          (6_000, 0), (6_500, 0), (8_190, 0), (10_000, 0), (12_000, 0), (14_000, 0), (16_001, 0), (18_000, 0), (20_000, 0), (22_000, 0), (24_575, 0), (30_001, 0),
          (5, 1), (16, 1), (31, 1), (64, 1), (127, 1), (200, 1), (500, 1), (1_027, 1), (1_500, 1), (2_041, 1), (3_000, 1), (3_001, 1), (4_099, 1), (5_001, 1),
          (6_100, 1), (6_143, 1), (8_100, 1), (12_000, 1), (16_000, 1), (20_001, 1), (24_000, 1), (25_002, 1)]


def _size(d, bf16, parts):
    """Rows of a step (at most four per team of threads that share a row) and a number of rows that gives every part seven steps and three
    rows; rows in two passes: sixteen rows under way."""
    p = cr.cr_plan_ex(2, 3, 1, 1_000, d, x_dtype=bf16)
    info = cr.cr_plan_info(p)
    cr.cr_plan_destroy(p)
    step = 4 * info.stage1_teams_per_group if info.stage1_team_size else 16
    if not info.stage1_team_size:
        parts = max(1, 4 * parts // (-(-d // (8 if bf16 else 4)) // 256 + 1))
    elif info.stage1_team_size <= 64 or (bf16 and info.stage1_team_size == 128):
        parts *= 2                                       # two workgroups per compute unit
    return step, parts * (7 * step + 3)


@pytest.mark.parametrize("d,bf16", WIDTHS)
def test_runs_are_as_long_as_the_test_needs(d, bf16):
    """Host: the sizes used below give parts of several steps, and a limit cuts them into runs of an odd number of rows."""
    step, m = _size(d, bf16, 256)
    p = cr.cr_plan_ex(2, 3, 1, m, d, x_dtype=bf16)
    pieces = []
    for value in (2 * step + 1, 10 ** 9):
        cr.cr_plan_set_split(p, cr.CR_SPLIT_ROWS_ONCE, value)
        _, b, e, team = cr.cr_plan_get_pieces(p)
        runs = sorted(set(zip(team.tolist(), b.tolist(), e.tolist())))
        pieces.append(len(runs))
        assert max(e - b for _, b, e in runs) == min(value, max(e - b for _, b, e in runs)) > 2 * step
    assert pieces[0] >= 3 * len(set(team.tolist())) and pieces[0] > 2 * pieces[1]
    cr.cr_plan_destroy(p)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16", WIDTHS)
def test_runs_of_several_steps(d, bf16):
    """Slabs against 64 bits.  What is in fp32 are the dot products, sums of at most four rows and the rounding of partial rows and slabs:
    their errors are independent from row to row and stay near one unit of 2^-24 in the 2-norm; 1e-6 is sixteen of them."""
    import torch

    step, m = _size(d, bf16, torch.cuda.get_device_properties(0).multi_processor_count)
    logistic = d % 2
    gen = torch.Generator(device="cuda").manual_seed(d)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_(generator=gen)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.randn(m, generator=gen, device="cuda")
    y = (y > 0).float() if logistic else y
    ref = None
    for split in ((cr.CR_SPLIT_ROWS_ONCE, 10 ** 9), (cr.CR_SPLIT_ROWS_ONCE, 2 * step + 1), (cr.CR_SPLIT_ROWS_ONCE, cr.CR_ROWS_WHOLE_RANGES)):
        plan = cr.cr_plan_ex(2, 3, 1, m, d, model=logistic, x_dtype=bf16)
        cr.cr_plan_set_split(plan, *split)
        ws = cr.Workspace(plan)
        rb, re_, _, _ = cr.cr_plan_get_segments(plan)
        if ref is None:
            cuts = np.unique(np.concatenate([rb, re_]))
            between = torch.zeros(len(cuts) - 1, d, dtype=torch.float64, device="cuda")
            rows = max(1, (1 << 25) // d)
            for i in range(len(cuts) - 1):
                for lo in range(int(cuts[i]), int(cuts[i + 1]), rows):
                    hi = min(lo + rows, int(cuts[i + 1]))
                    Xd = X[lo:hi].double()
                    z = Xd @ w.double()
                    between[i] += ((torch.sigmoid(z) if logistic else z) - y[lo:hi].double()) @ Xd
            ref = [between[np.searchsorted(cuts, b):np.searchsorted(cuts, e)].sum(0).cpu().numpy() for b, e in zip(rb, re_)]
        ws.slab_grads().fill_(float("nan"))
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_synchronize(plan)
        G = ws.slab_grads().double().cpu().numpy()
        cr.cr_plan_destroy(plan)
        for q, want in enumerate(ref):
            assert_close(G[q], want, 1e-6, 1e-6, ("slab", d, bf16, split, q))
