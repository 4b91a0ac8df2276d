"""Rows that several workgroups share: slices of every width, runs that end inside a step, and answers that nobody waits for."""
import ctypes

import pytest

import paper_1902_01981_amd as cr

# the narrowest and widest rows that are shared, both sides of a chunk more per thread, slices of unequal length, odd rows
WIDTHS = [(34_817, 0), (50_001, 0), (60_000, 0), (80_003, 0), (114_688, 0), (36_865, 1), (57_344, 1), (57_347, 1), (80_001, 1), (172_032, 1)]


@pytest.mark.parametrize("d,bf16,m,teams", [(36_865, 1, 40, 10), (36_865, 1, 4_000, 40), (50_008, 1, 4_000, 32), (60_000, 0, 4_000, 24), (114_688, 0, 4_000, 16),
                                            (114_689, 0, 4_000, 4), (172_033, 1, 4_000, 6)])
def test_parts(d, bf16, m, teams):
    """A part per crew, four rows and more; wider rows take two passes, whose parts have the chip's workgroups twice between them."""
    p = cr.cr_plan_ex(2, 4, 1, m, d, x_dtype=bf16)
    cr.cr_workspace_bytes(p)
    assert cr.cr_plan_info(p).num_teams == teams
    cr.cr_plan_destroy(p)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16", WIDTHS)
@pytest.mark.parametrize("m,rows_per_run", [(4, None), (23, None), (61, 3), (79, None), (700, 5)])
def test_nobody_waits(d, bf16, m, rows_per_run):
    """fp32 dot products, everything across rows fp64: 3e-6 of a slab's rms per entry, as for the other wide rows.  With no patience most
    parts of the dot products are worked out again: the same bits."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(d + m)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_(generator=gen)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.randn(m, generator=gen, device="cuda") + 4.0
    slabs = []
    for patience in (None, 0):
        plan = cr.cr_plan_ex(1, 3, 1, m, d, model=cr.CR_LOGISTIC if m == 23 else cr.CR_LINEAR, x_dtype=bf16)
        if rows_per_run:
            cr.cr_plan_set_split(plan, cr.CR_SPLIT_ROWS_ONCE, rows_per_run)
        if patience is not None:
            assert cr.load_library().cr_testing_patience(ctypes.c_void_p(plan), patience) == 0
        ws = cr.Workspace(plan)
        for _ in range(3):                               # launches one after the other: what the last one left is no answer
            ws.slab_grads().fill_(float("nan"))
            cr.cr_partial_grads(plan, X, y, w)
            cr.cr_synchronize(plan)
            slabs.append(ws.slab_grads().clone())
        rb, re_, _, _ = cr.cr_plan_get_segments(plan)
        del ws
        cr.cr_plan_destroy(plan)
    assert all(torch.equal(slabs[0], s) for s in slabs[1:])
    for q in range(len(rb)):
        x = X[int(rb[q]):int(re_[q])].double()
        z = x @ w.double()
        ref = x.T @ ((torch.sigmoid(z) if m == 23 else z) - y[int(rb[q]):int(re_[q])].double())
        assert float((slabs[0][q].double() - ref).abs().max() / ref.pow(2).mean().sqrt()) <= 3e-6


@pytest.mark.gpu
def test_more_steps_than_slots_are_kept_for():
    """16 crews, two rows per step and 1 031 or 1 032 steps: the slots of the first steps are used again."""
    import torch

    m, d, rows = 33_000, 172_032, 2_048
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16).normal_(generator=gen)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.randn(m, generator=gen, device="cuda") + 4.0
    plan = cr.cr_plan_ex(1, 3, 0, m, d, x_dtype=1)
    ws = cr.Workspace(plan)
    rb, re_, _, _ = cr.cr_plan_get_segments(plan)
    ref = torch.zeros(len(rb), d, device="cuda", dtype=torch.float64)
    for q in range(len(rb)):
        for lo in range(int(rb[q]), int(re_[q]), rows):
            x = X[lo:min(lo + rows, int(re_[q]))].double()
            ref[q] += (x @ w.double() - y[lo:lo + len(x)].double()) @ x
    slabs = []
    for patience in (64, 0):
        assert cr.load_library().cr_testing_patience(ctypes.c_void_p(plan), patience) == 0
        ws.slab_grads().fill_(float("nan"))
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_synchronize(plan)
        slabs.append(ws.slab_grads().clone())
    assert torch.equal(*slabs)
    assert float(((slabs[0].double() - ref).abs().amax(1) / ref.pow(2).mean(1).sqrt()).max()) <= 3e-6
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("m,d,bf16", [(4_000, 50_008, 1), (4_000, 60_000, 0)])
def test_what_is_late_costs_little(m, d, bf16):
    """Members that do not wait work out what has not arrived: 1.3 to 1.4 times as long, not as long as a wavefront takes for every slice of every row
    (12 to 17 times)."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(d)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_(generator=gen)
    w, y = torch.randn(d, generator=gen, device="cuda") / d ** 0.5, torch.rand(m, generator=gen, device="cuda")
    plan = cr.cr_plan_ex(2, 4, 1, m, d, model=cr.CR_LOGISTIC, x_dtype=bf16)
    ws = cr.Workspace(plan)
    times = {64: [], 0: []}
    for i in range(30):
        patience = 64 if i % 2 else 0
        assert cr.load_library().cr_testing_patience(ctypes.c_void_p(plan), patience) == 0
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        cr.cr_partial_grads(plan, X, y, w)
        end.record()
        end.synchronize()
        if i >= 10:
            times[patience].append(begin.elapsed_time(end))
    assert sorted(times[0])[5] <= 4.0 * sorted(times[64])[5]
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("bf16", [0, 1])
def test_rows_that_are_not_finite_stay_with_their_slabs(bf16):
    import torch

    m, d = 23, 60_001
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.randn(m, d, generator=gen, device="cuda").to(torch.bfloat16 if bf16 else torch.float32)
    plan = cr.cr_plan_ex(1, 3, 0, m, d, x_dtype=bf16)
    rb, re_, _, _ = cr.cr_plan_get_segments(plan)
    X[int(rb[1]), 7], X[int(re_[1]) - 1, d - 1] = float("inf"), float("nan")     # the first and the last row of the second slab
    ws = cr.Workspace(plan)
    cr.cr_partial_grads(plan, X, torch.zeros(m, device="cuda"), torch.randn(d, generator=gen, device="cuda"))
    cr.cr_synchronize(plan)
    finite = torch.isfinite(ws.slab_grads()).all(1).tolist()
    assert finite == [True, False, True]
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bf16", [(50_001, 0), (60_000, 0), (80_003, 0), (57_347, 1), (50_008, 1), (172_032, 1)])
@pytest.mark.parametrize("patience", [None, 0])
def test_infinities_in_the_last_chunk_of_a_slice(d, bf16, patience):
    """sigmoid(+-inf) is 0 or 1, so that an infinite entry reaches its own column only, wherever the columns are cut into slices: an entry in
    the last chunk of every slice that 2 to 16 workgroups can have, first and last column of the chunk.  The infinite products of a row have one
    sign.  Fewer than 80 rows of these widths are always shared."""
    import torch

    vec = 8 if bf16 else 4
    nq = (d + vec - 1) // vec
    cols = sorted({c for members in range(2, 17) for j in range(1, members + 1) for q in [nq * j // members - 1]
                   for c in (min(q * vec, d - vec), min(q * vec, d - vec) + vec - 1, min(q * vec + vec - 1, d - 1))})
    m = 79
    gen = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(m, d, generator=gen, device="cuda").to(torch.bfloat16 if bf16 else torch.float32)
    w = torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    y = torch.full((m,), 0.25, device="cuda")
    for i, c in enumerate(cols):
        X[i % m, c] = torch.copysign(torch.tensor(float("inf")), w[c].cpu() * (1 if i % m % 3 else -1))
    plan = cr.cr_plan_ex(1, 3, 1, m, d, model=cr.CR_LOGISTIC, x_dtype=bf16)
    if patience is not None:
        assert cr.load_library().cr_testing_patience(ctypes.c_void_p(plan), patience) == 0
    ws = cr.Workspace(plan)
    cr.cr_partial_grads(plan, X, y, w)
    cr.cr_synchronize(plan)
    rb, re_, _, _ = cr.cr_plan_get_segments(plan)
    for q in range(len(rb)):
        lo, hi = int(rb[q]), int(re_[q])
        z = X[lo:hi].double() @ w.double()
        assert not bool(torch.isnan(z).any())
        res = torch.sigmoid(z) - y[lo:hi].double()
        got = ws.slab_grads()[q].double()
        whole = torch.isfinite(X[lo:hi]).all(0)
        assert torch.equal(torch.isfinite(got), whole)
        ref = X[lo:hi].double().nan_to_num(posinf=0.0, neginf=0.0).T @ res
        assert float(((got - ref)[whole]).abs().max() / ref[whole].pow(2).mean().sqrt()) <= 3e-6
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("m,d,bf16", [(61, 50_001, 0), (700, 57_347, 1)])
def test_replays_of_a_captured_launch(m, d, bf16):
    """The number of a launch is kept on the device: replays, with other weights each and calls outside the graph in between, give the bits of
    plain calls."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32).normal_(generator=gen)
    y = torch.randn(m, generator=gen, device="cuda")
    ws_of_seed = [torch.randn(d, generator=gen, device="cuda") / d ** 0.5 for _ in range(4)]
    w, stream = torch.empty(d, device="cuda"), torch.cuda.Stream()
    plan = cr.cr_plan_ex(1, 3, 1, m, d, x_dtype=bf16)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ws = cr.Workspace(plan)
        want = []
        for v in ws_of_seed:
            w.copy_(v)
            cr.cr_partial_grads(plan, X, y, w)
            want.append(ws.slab_grads().clone())
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            cr.cr_partial_grads(plan, X, y, w)
        for i in (0, 1, 2, 3, 1, 0):
            w.copy_(ws_of_seed[i])
            ws.slab_grads().fill_(float("nan"))
            graph.replay()
            stream.synchronize()
            assert torch.equal(ws.slab_grads(), want[i])
            if i % 2:
                cr.cr_partial_grads(plan, X, y, w)
                cr.cr_synchronize(plan)
                assert torch.equal(ws.slab_grads(), want[i])
    del graph, ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
def test_more_launches_than_numbers():
    """A tag has 12 bits for the launch: around the 4 096th launch, with other weights each, nothing of an earlier launch is taken for an answer."""
    import torch

    m, d = 12, 50_001
    gen = torch.Generator(device="cuda").manual_seed(m)
    X, y = torch.randn(m, d, generator=gen, device="cuda"), torch.randn(m, generator=gen, device="cuda")
    w = [torch.randn(d, generator=gen, device="cuda") / d ** 0.5 for _ in range(3)]
    plan = cr.cr_plan_ex(1, 3, 1, m, d)
    ws = cr.Workspace(plan)
    want = []
    for v in w:
        cr.cr_partial_grads(plan, X, y, v)
        want.append(ws.slab_grads().clone())
    for i in range(4_110):
        cr.cr_partial_grads(plan, X, y, w[i % 3])
        if i > 4_080:
            cr.cr_synchronize(plan)
            assert torch.equal(ws.slab_grads(), want[i % 3]), i
    del ws
    cr.cr_plan_destroy(plan)
