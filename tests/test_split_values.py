"""Work splits at the ends of what cr_plan_set_split takes, and what a plan reports about the split it runs (host only)."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr


def _pieces(p):
    return [a.tolist() for a in cr.cr_plan_get_pieces(p)]


# narrow rows (lanes of a wavefront share a row), rows of a whole workgroup, rows in two passes; both types
@pytest.mark.parametrize("d,bf16", [(1, 0), (8, 0), (512, 0), (2_048, 1), (4_096, 0), (3_001, 1), (24_577, 0)])
@pytest.mark.parametrize("value", [2 ** 63 - 1, 2 ** 62 - 1, 2 ** 61, 2 ** 31])
def test_more_rows_than_there_are(d, bf16, value):
    """No limit on rows can be said with any large number: the same split as a limit of all rows, and the value is reported back."""
    kinds = [cr.CR_SPLIT_ROWS_ONCE, cr.CR_SPLIT_ROW_CELLS] + ([cr.CR_SPLIT_SHARED_CELLS] if d == 4_096 else [])
    for kind in kinds:
        p, q = cr.cr_plan_ex(2, 3, 1, 5_000, d, x_dtype=bf16), cr.cr_plan_ex(2, 3, 1, 5_000, d, x_dtype=bf16)
        cr.cr_plan_set_split(p, kind, value)
        cr.cr_plan_set_split(q, kind, 5_000)
        assert _pieces(p) == _pieces(q) and cr.cr_workspace_bytes(p) == cr.cr_workspace_bytes(q)
        assert cr.cr_plan_info(p).split_value == value
        slab, pb, pe, _ = cr.cr_plan_get_pieces(p)
        rb, re_, _, _ = cr.cr_plan_get_segments(p)
        assert np.all(pe > pb) and np.all(pb >= rb[slab]) and np.all(pe <= re_[slab]) and (pe - pb).sum() == cr.cr_plan_info(p).row_visits
        cr.cr_plan_destroy(p)
        cr.cr_plan_destroy(q)
