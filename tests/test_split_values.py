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


# one range per worker, ranges that overlap without being equal, more ranges than compute units; 1 to 1 870 columns
@pytest.mark.parametrize("L,n,s,m,d,bf16", [(2, 3, 1, 1_200, 100, 0), (1, 10, 4, 253, 900, 0), (3, 4, 1, 328, 1_000, 0), (2, 12, 2, 312, 1_870, 1),
                                             (3, 3, 1, 4_003, 64, 0), (2, 4, 1, 60, 1, 0), (2, 4, 0, 68, 200, 0), (2, 3, 1, 12, 2_500, 0), (2, 4, 1, 8_359, 71, 1),
                                             (2, 4, 1, 60_000, 1_500, 0), (2, 4, 1, 4_000, 50_008, 1), (3, 4, 1, 252_000, 4_096, 0)])
def test_default_runs_as_reported(L, n, s, m, d, bf16):
    info = _runs_as_reported((L, n, s, m, d), bf16)
    assert (info.split_value == cr.CR_ROWS_WHOLE_RANGES) == (info.split_kind == cr.CR_SPLIT_ROWS_ONCE and info.split_value != m)


@pytest.mark.parametrize("L,n,s,m,d,bf16", [(2, 3, 1, 5_000, 64, 0), (3, 4, 1, 9_000, 700, 1), (2, 4, 1, 2_000, 5_000, 0)])
def test_whole_ranges(L, n, s, m, d, bf16):
    """A workgroup per distinct slab range, which it has whole: no partial rows, so the workspace has fewer rows than with parts."""
    p, q = cr.cr_plan_ex(L, n, s, m, d, x_dtype=bf16), cr.cr_plan_ex(L, n, s, m, d, x_dtype=bf16)
    cr.cr_plan_set_split(p, cr.CR_SPLIT_ROWS_ONCE, cr.CR_ROWS_WHOLE_RANGES)
    cr.cr_plan_set_split(q, cr.CR_SPLIT_ROWS_ONCE, m)
    rb, re_, _, _ = cr.cr_plan_get_segments(p)
    slab, pb, pe, team = cr.cr_plan_get_pieces(p)
    ranges = sorted(set(zip(rb.tolist(), re_.tolist())))
    assert cr.cr_plan_info(p).num_teams == len(ranges) and len(slab) == len(rb)
    assert sorted(zip(slab.tolist(), pb.tolist(), pe.tolist())) == sorted(zip(range(len(rb)), rb.tolist(), re_.tolist()))
    assert [ranges[t] for t in team] == list(zip(pb.tolist(), pe.tolist()))
    assert cr.cr_workspace_bytes(p) < cr.cr_workspace_bytes(q)
    cr.cr_plan_destroy(p)
    cr.cr_plan_destroy(q)
    # rows in two passes have no such form: the value then is what any large one is, no limit
    w, v = cr.cr_plan_ex(2, 3, 1, 100, 24_577), cr.cr_plan_ex(2, 3, 1, 100, 24_577)
    cr.cr_plan_set_split(w, cr.CR_SPLIT_ROWS_ONCE, cr.CR_ROWS_WHOLE_RANGES)
    cr.cr_plan_set_split(v, cr.CR_SPLIT_ROWS_ONCE, 100)
    assert _pieces(w) == _pieces(v)
    cr.cr_plan_destroy(w)
    cr.cr_plan_destroy(v)


def test_whole_ranges_of_more_rows_than_a_run_can_have():
    """The kernels count a run's rows in 32 bits: longer ranges are cut into parts as under any large value."""
    p, q = cr.cr_plan_ex(1, 4, 1, 1 << 34, 1), cr.cr_plan_ex(1, 4, 1, 1 << 34, 1)
    cr.cr_plan_set_split(p, cr.CR_SPLIT_ROWS_ONCE, cr.CR_ROWS_WHOLE_RANGES)
    cr.cr_plan_set_split(q, cr.CR_SPLIT_ROWS_ONCE, 1 << 34)
    assert _pieces(p) == _pieces(q) and max(e - b for b, e in zip(*_pieces(p)[1:3])) <= 1 << 30
    cr.cr_plan_destroy(p)
    cr.cr_plan_destroy(q)


@pytest.mark.parametrize("kind", [cr.CR_SPLIT_ROWS_ONCE, cr.CR_SPLIT_ROW_CELLS, cr.CR_SPLIT_SHARED_CELLS])
def test_out_of_host_memory_is_an_error(kind):
    """A split of tens of millions of pieces in a process that may not grow by that much: a status, and the plan can be used on."""
    import os
    import subprocess
    import sys

    code = f"""
import resource
import paper_1902_01981_amd as cr
p = cr.cr_plan_ex(2, 3, 1, 12_000_000, 1_500)
cr.cr_plan_set_split(p, cr.CR_SPLIT_EQUAL_RANGES, 100)
size = int(open('/proc/self/statm').read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (size + (200 << 20), resource.RLIM_INFINITY))
for _ in range(2):
    try:
        cr.cr_plan_set_split(p, {kind}, 1)
        raise SystemExit('the split fits after all')
    except cr.CodedReduceError as e:
        assert e.status == cr.CR_E_NOMEM, e
    assert cr.cr_plan_info(p).num_pieces == 0
cr.cr_plan_set_split(p, cr.CR_SPLIT_ROWS_ONCE, 10_000)
assert cr.cr_plan_info(p).num_pieces > 0 and cr.cr_workspace_bytes(p) > 0
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stderr[-400:])
