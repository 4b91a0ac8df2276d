"""Stage 1 with every row formed once for all slabs that hold it (CR_SPLIT_ROWS_ONCE), at the widths where its kernels change: lanes per
row, chunks per lane, threads per row; the shortest and the widest rows; runs of one row, of a step and whole ones (parts are short here:
test_run_borders.py has runs of several steps)."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr
from cr_inputs import workloads as wl
from _harness import TOL, HipPath, OraclePath, assert_close, gate_for

# (d, bf16): both sides of every border of the variant tables
WIDTHS = [(1, 0), (3, 0), (4, 0), (8, 0), (9, 0), (17, 0), (33, 0), (64, 0), (65, 0), (129, 0), (256, 0), (257, 0), (513, 0), (769, 0), (1024, 0),
          (1025, 0), (2050, 0), (3073, 0), (4099, 0), (5121, 0), (6145, 0), (7168, 0), (7169, 0), (8193, 0), (10_241, 0), (12_290, 0), (14_337, 0),
          (16_385, 0), (18_433, 0), (20_481, 0), (22_529, 0), (24_576, 0),
          (1, 1), (7, 1), (8, 1), (16, 1), (17, 1), (33, 1), (65, 1), (129, 1), (257, 1), (512, 1), (513, 1), (1025, 1), (1537, 1), (2048, 1),
          (2049, 1), (4098, 1), (6145, 1), (8192, 1), (8193, 1), (12_289, 1), (16_385, 1), (20_481, 1), (24_576, 1)]


@pytest.mark.parametrize("value", [1, 19, 10 ** 6])
def test_rows_once_tables(value):
    """Every slab is tiled exactly, no run crosses a slab boundary, the holders of a run share one workgroup, the parts are even."""
    p = cr.cr_plan_ex(3, 3, 1, 4_003, 64)
    cr.cr_plan_set_split(p, cr.CR_SPLIT_ROWS_ONCE, value)
    rb, re_, _, node = cr.cr_plan_get_segments(p)
    slab, pb, pe, team = cr.cr_plan_get_pieces(p)
    info = cr.cr_plan_info(p)
    assert (info.split_kind, info.split_value, info.num_pieces) == (cr.CR_SPLIT_ROWS_ONCE, value, len(slab))
    assert np.all(pe > pb) and (pe - pb).sum() == info.row_visits and np.all(np.diff(team) >= 0)
    cuts = np.unique(np.concatenate([rb, re_]))
    at = np.searchsorted(cuts, pb, side="right")
    assert np.all(pe <= cuts[at])
    for q in range(len(node)):
        idx = np.nonzero(slab == q)[0]
        idx = idx[np.argsort(pb[idx])]
        assert pb[idx[0]] == rb[q] and pe[idx[-1]] == re_[q] and np.array_equal(pb[idx[1:]], pe[idx[:-1]])
    end, by = {}, {}
    for b, e, t in zip(pb, pe, team):
        assert end.setdefault(b, e) == e and by.setdefault(b, t) == t
    rows = np.array([sum(end[b] - b for b in end if by[b] == t) for t in range(info.num_teams)])
    assert rows.max() - rows.min() <= 1 and rows.sum() == 4_003
    cr.cr_plan_destroy(p)
    # rows too wide for one pass: every row once by default too, and what the plan reports can be set
    wide = cr.cr_plan_ex(2, 3, 1, 100, 24_577)
    cr.cr_workspace_bytes(wide)
    info = cr.cr_plan_info(wide)
    assert (info.split_kind, info.stage1_team_size) == (cr.CR_SPLIT_ROWS_ONCE, 0)
    pieces = cr.cr_plan_get_pieces(wide)
    cr.cr_plan_set_split(wide, info.split_kind, info.split_value)
    assert all(np.array_equal(a, b) for a, b in zip(pieces, cr.cr_plan_get_pieces(wide)))
    cr.cr_plan_destroy(wide)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16", WIDTHS)
def test_rows_once_matches_the_oracle(d, bf16):
    """Slabs against the fp64 oracle under the default split and with runs of one row and of up to 13.  What is in fp32 are the dot products and
    sums of at most four rows: inside the parity tests' regression gate (1e-5)."""
    logistic = d % 2 == 0
    m = 12 * 25 + 1 if d > 1024 else 1_801
    cfg = wl.config("cfg3" if logistic else "cfg2", L=2, n=3, s=1, m=m, d=d, model=int(logistic), x_dtype=bf16,
                    w0_std=None if logistic else 1.0, seed=9_000 + d)
    data = wl.make_dataset(cfg)
    orc = OraclePath(2, 3, 1, data["X"], data["y"], int(logistic))
    ref = orc.slab_grads(data["w0"])
    mask = wl.draw_mask(wl.mask_stream(cfg), 2, 3, 1)
    for split in (None, (cr.CR_SPLIT_ROWS_ONCE, 1), (cr.CR_SPLIT_ROWS_ONCE, 13)):
        hip = HipPath(2, 3, 1, data["X"], data["y"], int(logistic), bf16, teams=split)
        assert hip.info.split_kind == cr.CR_SPLIT_ROWS_ONCE
        import torch

        g = hip.gradient(torch.from_numpy(data["w0"]).cuda(), mask)
        G = hip.ws.slab_grads().cpu().numpy()
        for q, want in enumerate(ref):
            assert_close(G[q], want, TOL[bf16], gate_for(), ("slab", split, q))
        assert_close(g, orc.full_gradient(data["w0"]), TOL[bf16], gate_for(hip.info.gamma, 2), ("decoded gradient", split))
        hip.close()


@pytest.mark.gpu
def test_rows_once_streamed_past_the_caches():
    """256 MiB and more: the same kernels with the non-temporal hint.  Rows of 64 to 3000 columns, against the literal row cells (the
    row cells add runs of up to 256 rows in fp32, well under the gate)."""
    import torch

    for d, bf16 in ((64, 0), (1_000, 0), (3_000, 0), (10_000, 0), (1_027, 1), (5_000, 1), (10_000, 1)):
        m = (260 << 20) // (d * (2 if bf16 else 4)) + 77
        X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_()
        y, w = torch.randn(m, device="cuda"), torch.randn(d, device="cuda")
        out = []
        for split in (None, (cr.CR_SPLIT_ROW_CELLS, 256)):
            plan = cr.cr_plan_ex(2, 4, 1, m, d, x_dtype=bf16)
            if split:
                cr.cr_plan_set_split(plan, *split)
            ws = cr.Workspace(plan)
            cr.cr_partial_grads(plan, X, y, w)
            cr.cr_synchronize(plan)
            out.append(ws.slab_grads().double().cpu().numpy())
            cr.cr_plan_destroy(plan)
        for q in range(len(out[0])):
            assert_close(out[0][q], out[1][q], 1e-5, gate_for(), ("slab", d, q))


# rows per workgroup of the first pass 1, 2, 4 and 8 (from 448, 896, 1792 and 3584 rows on 256 compute units) and a ragged last one;
# rows that end in a whole chunk, an overlapping one, a chunk of one column; more rows than are kept in the cache between the passes
WIDE = [(24_577, 0, 13), (24_580, 1, 14), (30_003, 0, 897), (32_768, 1, 451), (24_583, 1, 1_801), (24_578, 0, 3_601)]


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16,m", WIDE)
def test_wide_rows_once(d, bf16, m):
    """Two passes, every row once, against the row cells of every holder separately, which add runs of up to 64 rows in fp32, well under the
    gate (1e-5); `value` 1 and 70 for runs of one row and for parts cut into runs and a remainder."""
    import torch

    for logistic in (0, 1):
        X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_()
        w = torch.randn(d, device="cuda") / d ** 0.5
        y = (torch.rand(m, device="cuda") < 0.5).float()
        out = []
        for split in ((cr.CR_SPLIT_ROW_CELLS, 64), None, (cr.CR_SPLIT_ROWS_ONCE, 1), (cr.CR_SPLIT_ROWS_ONCE, 70)):
            if split and split[1] == 1 and m > 1_000:
                continue
            plan = cr.cr_plan_ex(2, 3, 1, m, d, model=logistic, x_dtype=bf16)
            if split:
                cr.cr_plan_set_split(plan, *split)
            ws = cr.Workspace(plan)
            ws.slab_grads().fill_(float("nan"))
            cr.cr_partial_grads(plan, X, y, w)
            cr.cr_synchronize(plan)
            out.append(ws.slab_grads().double().cpu().numpy())
            cr.cr_plan_destroy(plan)
        for G in out[1:]:
            for q in range(len(G)):
                assert_close(G[q], out[0][q], 1e-5, gate_for(), ("slab", d, q))
