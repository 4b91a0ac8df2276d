"""The tables behind the stage-1 splits, replayed on the host: tree_plan.cpp is compiled into a small library, its runs, destinations and
sums are carried out on integer row weights, and every slab must end with exactly the weight of its rows."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_1902_01981_amd as cr

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1902_01981_amd", "csrc")
WRAPPER = r"""
#include "tree_plan.h"
static std::vector<cr::Slab> slabs;
static cr::OnceWork work;
static cr::Split split;
extern "C" void set_slabs(int n, const int64_t *rb, const int64_t *re, const int32_t *node)
{
    slabs.clear();
    for (int i = 0; i < n; ++i) { cr::Slab s{}; s.node = node[i]; s.row_begin = rb[i]; s.row_end = re[i]; s.coef = 1.0; slabs.push_back(s); }
}
extern "C" void equal_parts(int64_t m, int64_t parts, int64_t limit) { cr::once_equal_parts(slabs, m, parts, limit, work); }
extern "C" void equal_parts_copies(int64_t m, int64_t parts, int64_t limit, int64_t most) { cr::once_equal_parts(slabs, m, parts, limit, work, most); }
extern "C" void whole_ranges() { cr::once_whole_ranges(slabs, work); }
extern "C" void equal_ranges(int teams) { cr::split_equal_ranges(slabs, teams, split); cr::once_of_pieces(slabs, split, work); }
extern "C" void queues(int64_t cell_rows, int lanes, int per_group, int slots)
{
    cr::split_shared_queues(slabs, cell_rows, lanes, per_group, slots, split);
    cr::once_of_queues(slabs, split, per_group, work);
}
extern "C" void as_split() { cr::once_as_split(slabs, work, split); }
extern "C" void sizes(int64_t *out)
{
    const int64_t v[] = {(int64_t)work.runs.size(), (int64_t)work.part_run_begin.size() - 1, (int64_t)work.sums.size(), (int64_t)work.dst.size(),
                         work.partials, (int64_t)split.pieces.size(), split.teams};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
extern "C" void tables(int64_t *runs, int32_t *parts, int32_t *sums, int32_t *dst, int64_t *pieces)
{
    for (auto &r : work.runs) { *runs++ = r.row_begin; *runs++ = r.row_end; *runs++ = r.dst_begin; *runs++ = r.dst_end; }
    for (auto b : work.part_run_begin) *parts++ = b;
    for (auto &s : work.sums) { *sums++ = s.row_begin; *sums++ = s.row_end; *sums++ = s.dst_begin; *sums++ = s.dst_end; }
    for (auto d : work.dst) *dst++ = d;
    for (auto &p : split.pieces) { *pieces++ = p.slab; *pieces++ = p.row_begin; *pieces++ = p.row_end; *pieces++ = p.team; }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("tables")
    (d / "w.cpp").write_text(WRAPPER)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "w.cpp"), os.path.join(CSRC, "tree_plan.cpp"), "-o", str(d / "w.so")],
                   check=True)
    return ctypes.CDLL(str(d / "w.so"))


def _ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _load(lib, L, n, s, m):
    p = cr.cr_plan_ex(L, n, s, m, 8)
    rb, re_, _, node = (np.ascontiguousarray(a) for a in cr.cr_plan_get_segments(p))
    cr.cr_plan_destroy(p)
    rb, re_, node = rb.astype(np.int64), re_.astype(np.int64), node.astype(np.int32)
    lib.set_slabs(len(rb), _ptr(rb), _ptr(re_), _ptr(node))
    return rb, re_


def _replay(lib, rb, re_, m):
    """Carries the tables out; returns runs, the parts' bounds and the pieces of the split."""
    size = np.zeros(7, dtype=np.int64)
    lib.sizes(_ptr(size))
    R, P, Q, D, partials, pieces, _ = (int(v) for v in size)
    runs, parts = np.zeros((R, 4), dtype=np.int64), np.zeros(P + 1, dtype=np.int32)
    sums, dst, pc = np.zeros((Q, 4), dtype=np.int32), np.zeros(max(D, 1), dtype=np.int32), np.zeros((max(pieces, 1), 4), dtype=np.int64)
    lib.tables(_ptr(runs), _ptr(parts), _ptr(sums), _ptr(dst), _ptr(pc))
    S = len(rb)
    weight = np.concatenate([[0], np.cumsum((np.arange(m, dtype=np.int64) * 7919) % 10_007 + 1)])
    out, written = np.zeros(S + partials, dtype=np.int64), np.zeros(S + partials, dtype=np.int64)
    assert np.all(np.diff(parts) >= 1) and parts[0] == 0 and parts[-1] == R          # every workgroup has a run to start with
    assert np.all(runs[:, 1] > runs[:, 0]) and np.all(runs[:, 3] > runs[:, 2]) and runs[:, 3].max() <= D
    cuts = np.unique(np.concatenate([rb, re_]))
    for b, e, lo, hi in runs:
        out[dst[lo:hi]] = weight[e] - weight[b]
        written[dst[lo:hi]] += 1
    for b, e, lo, hi in sums:
        assert S <= b < e <= S + partials and np.all(written[b:e] == 1)
        out[dst[lo:hi]] = out[b:e].sum()
        written[dst[lo:hi]] += 1
    assert np.all(written[:S] == 1) and np.all(written <= 1)
    assert np.array_equal(out[:S], weight[re_] - weight[rb])
    return runs, parts, pc[:pieces], cuts


TREES = [(2, 3, 1, 301), (3, 4, 1, 9_001), (2, 12, 2, 4_003), (3, 3, 2, 2_000), (4, 3, 1, 2_222), (1, 10, 4, 777), (1, 6, 0, 500), (2, 5, 0, 1_234), (2, 4, 1, 20),
         (5, 2, 1, 400)]


@pytest.mark.parametrize("L,n,s,m", TREES)
def test_rows_once_tables_replayed(lib, L, n, s, m):
    rb, re_ = _load(lib, L, n, s, m)
    for parts in (1, 7, min(m, 256)):
        for limit in (1, 5, 64, 1 << 40):
            lib.equal_parts(ctypes.c_int64(m), ctypes.c_int64(parts), ctypes.c_int64(limit))
            lib.as_split()
            runs, begin, pieces, cuts = _replay(lib, rb, re_, m)
            assert np.all(runs[:, 1] - runs[:, 0] <= limit) and np.array_equal(runs[1:, 0], runs[:-1, 1]) and runs[0, 0] == 0 and runs[-1, 1] == m
            assert len(begin) - 1 == parts and (pieces[:, 2] - pieces[:, 1]).sum() == (re_ - rb).sum()
    lib.whole_ranges()
    runs, begin, _, _ = _replay(lib, rb, re_, m)
    assert len(runs) == len(begin) - 1 == len(set(zip(rb, re_)))
    if s == 0:
        for teams in (1, 3, 64, m):
            lib.equal_ranges(teams)
            runs, begin, pieces, _ = _replay(lib, rb, re_, m)
            assert len(begin) - 1 == teams and np.array_equal(runs[:, :2], pieces[:, 1:3])


@pytest.mark.parametrize("L,n,s,m", [t for t in TREES if t[2] > 0])
@pytest.mark.parametrize("per_group", [2, 4, 8])
def test_a_workgroup_does_the_cells_it_is_said_to_do(lib, L, n, s, m, per_group):
    """Shared cells: what runs is what the pieces say.  Every workgroup that is named has rows, exactly those of its pieces, each of its
    cells once; where a cell has more holders than a workgroup serves, each of its workgroups forms it."""
    rb, re_ = _load(lib, L, n, s, m)
    for cell_rows in (1, 9, 100, 1 << 30):
        lib.queues(ctypes.c_int64(cell_rows), 8, per_group, 4)
        runs, begin, pieces, _ = _replay(lib, rb, re_, m)
        group = pieces[:, 3] // per_group
        busy = np.unique(group)
        assert len(begin) - 1 == len(busy)
        for part, g in enumerate(busy):
            mine = {(int(b), int(e)) for b, e in pieces[group == g, 1:3]}
            have = [(int(b), int(e)) for b, e in runs[begin[part]:begin[part + 1], :2]]
            assert len(have) == len(mine) and set(have) == mine


@pytest.mark.parametrize("L,n,s,m", TREES)
def test_runs_with_many_slabs_are_handed_on_by_a_sum(lib, L, n, s, m):
    """No run is written to more slabs than allowed, besides its partial row; the same runs, and every slab still complete."""
    rb, re_ = _load(lib, L, n, s, m)
    for parts in (1, 7, min(m, 256)):
        lib.equal_parts(ctypes.c_int64(m), ctypes.c_int64(parts), ctypes.c_int64(1 << 40))
        lib.as_split()
        want, _, pieces, _ = _replay(lib, rb, re_, m)
        for most in (0, 1, 2):
            lib.equal_parts_copies(ctypes.c_int64(m), ctypes.c_int64(parts), ctypes.c_int64(1 << 40), ctypes.c_int64(most))
            lib.as_split()
            runs, _, again, _ = _replay(lib, rb, re_, m)
            assert np.array_equal(runs[:, :2], want[:, :2]) and (runs[:, 3] - runs[:, 2]).max() <= most + 1
            assert sorted(map(tuple, again)) == sorted(map(tuple, pieces))
