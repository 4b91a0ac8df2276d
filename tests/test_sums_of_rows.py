"""Stage 1's sums over many rows: fp64 beyond the few rows that a thread adds at a time."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

pytestmark = pytest.mark.gpu

# (d, bf16, m): every kernel family with several hundred rows per accumulator -- lanes that share a row, several chunks per lane, two,
# four and eight wavefronts per row, the widest rows of one pass, rows in two passes
SHAPES = [(8, 0, 8_000_000), (64, 0, 4_000_000), (260, 0, 1_000_000), (1_000, 0, 600_000), (1_100, 0, 128_000), (2_050, 0, 128_000), (6_500, 0, 100_000),
          (10_000, 0, 100_000), (18_000, 0, 60_000), (24_576, 0, 60_000), (30_000, 0, 40_000),
          (16, 1, 8_000_000), (512, 1, 1_000_000), (1_027, 1, 600_000), (3_001, 1, 200_000), (5_001, 1, 200_000), (3_000, 1, 128_000), (8_192, 1, 128_000),
          (20_480, 1, 100_000), (24_576, 1, 100_000), (50_008, 1, 40_000)]


@pytest.mark.parametrize("d,bf16,m", SHAPES)
def test_long_sums_are_not_rounded_on_the_way(d, bf16, m):
    """X = 1, w = 0, y = -c: every entry of a slab is its number of rows times c, a sum whose fp32 rounding errors all point the same way
    while the sum stays within a power of two.  Allowed: four roundings of fp32 sums of at most four rows, one of a partial row, one of
    the slab: six units of 2^-24.  The margin of 1e-9 is for fp64."""
    import torch

    c = float(np.float32(0.1))
    X = torch.ones(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32)
    y = torch.full((m,), -c, device="cuda")
    w = torch.zeros(d, device="cuda")
    for L, n, s in ((1, 3, 1), (1, 4, 0)):
        plan = cr.cr_plan_ex(L, n, s, m, d, x_dtype=bf16)
        ws = cr.Workspace(plan)
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_synchronize(plan)
        G = ws.slab_grads().double().cpu().numpy()
        rb, re_, _, _ = cr.cr_plan_get_segments(plan)
        cr.cr_plan_destroy(plan)
        for q in range(len(rb)):
            want = c * float(re_[q] - rb[q])
            worst = float(np.max(np.abs(G[q] - want))) / want
            assert worst <= 6 * 2.0 ** -24 + 1e-9, (d, bf16, s, q, worst * 2 ** 24)
