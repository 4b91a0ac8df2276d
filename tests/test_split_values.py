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


def _runs_as_reported(args, bf16):
    """What the plan reports of its default split can be set, and is then the same work: pieces, kernel, workspace."""
    p, q = cr.cr_plan_ex(*args, x_dtype=bf16), cr.cr_plan_ex(*args, x_dtype=bf16)
    size = cr.cr_workspace_bytes(p)
    a = cr.cr_plan_info(p)
    cr.cr_plan_set_split(q, a.split_kind, a.split_value)
    b = cr.cr_plan_info(q)
    assert cr.cr_workspace_bytes(q) == size
    for field in ("split_kind", "split_value", "num_teams", "num_pieces", "stage1_team_size", "stage1_teams_per_group", "stage1_staged", "unit_slots"):
        assert getattr(a, field) == getattr(b, field), (args, field, getattr(a, field), getattr(b, field))
    assert _pieces(p) == _pieces(q)
    cr.cr_plan_destroy(p)
    cr.cr_plan_destroy(q)
    return a


@pytest.mark.parametrize("L,n,m,d,bf16", [(1, 10, 100_000, 10_000, 0), (2, 4, 1_000_000, 1_024, 0), (3, 3, 600_000, 1_027, 1), (1, 4, 20_000, 30_000, 0)])
def test_no_redundancy_runs_as_reported(L, n, m, d, bf16):
    """s = 0 and 1 GiB or more.  Equal ranges of the row visits are then equal ranges of rows that nobody else holds."""
    info = _runs_as_reported((L, n, 0, m, d), bf16)
    assert info.row_visits == m and info.split_kind == (cr.CR_SPLIT_EQUAL_RANGES if d <= 24_576 else cr.CR_SPLIT_ROWS_ONCE)


@pytest.mark.parametrize("teams", [1, 7, 500, 10 ** 6])
def test_equal_ranges_without_redundancy(teams):
    """The ranges are those of the slab-major row visits, as with redundancy, and every team that has rows is a workgroup."""
    p = cr.cr_plan_ex(2, 3, 0, 3_001, 96)
    cr.cr_plan_set_split(p, cr.CR_SPLIT_EQUAL_RANGES, teams)
    info = cr.cr_plan_info(p)
    slab, pb, pe, team = cr.cr_plan_get_pieces(p)
    rb, re_, _, _ = cr.cr_plan_get_segments(p)
    assert info.num_teams == min(teams, 3_001) and np.all(np.diff(slab) >= 0) and np.all(np.diff(team) >= 0)
    load = np.bincount(team, weights=pe - pb, minlength=info.num_teams)
    assert load.sum() == 3_001 and load.max() - load.min() <= 1
    for q in range(len(rb)):
        idx = np.nonzero(slab == q)[0]
        assert pb[idx[0]] == rb[q] and pe[idx[-1]] == re_[q] and np.array_equal(pb[idx[1:]], pe[idx[:-1]])
    cr.cr_plan_destroy(p)
