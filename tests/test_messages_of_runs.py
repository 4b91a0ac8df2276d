"""After a call of several masks the messages are those that the separate calls would have left, also where a straggler's row keeps what an
earlier mask of the call put there: on every route of the encode, over one batch of masks and two."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

# one launch per mask; a launch each for encode and decode with the nodes side by side, and with a walk (four levels, 462 nodes); one launch
# for up to 16 masks; the wide encode
CASES = [(2, 3, 1, 100, 19), (3, 6, 2, 1_030, 5), (2, 12, 2, 40_001, 4), (4, 3, 1, 83_000, 4), (2, 21, 1, 77, 18), (2, 8, 2, 90_003, 18), (3, 3, 1, 33_001, 5),
         (2, 8, 2, 1_048_580, 3)]


def _masks(rng, steps, groups, n, s):
    masks = np.zeros((steps, groups * n), np.uint8)
    for t in range(steps):
        for g in range(groups):
            masks[t, g * n + rng.choice(n, int(rng.integers(0, s + 1)), replace=False)] = 1
    masks[-1, ::n] = 1 if s else 0                       # stragglers at the end whose rows are an earlier mask's
    masks[-1].reshape(groups, n)[:, s + 1:] = 0
    for g in range(groups):
        extra = np.flatnonzero(masks[-1, g * n:(g + 1) * n])[s:]
        masks[-1, g * n + extra] = 0
    return masks


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,d,steps", CASES)
def test_aggregate_run(L, n, s, d, steps):
    import torch

    N = sum(n ** l for l in range(1, L + 1))
    plan = cr.cr_plan_ex(L, n, s, 2 * N, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    S = cr.cr_plan_info(plan).num_slabs
    gen = torch.Generator(device="cuda").manual_seed(d)
    few = S * d > 1 << 26                                # the same slabs for every mask
    G = torch.randn(1 if few else steps, (S * d + 3) // 4 * 4, generator=gen, device="cuda")
    masks = _masks(np.random.default_rng(d), steps, N // n, n, s)
    M, want, got = ws.messages(), torch.empty(steps, d, device="cuda"), torch.empty(steps, d, device="cuda")
    M.fill_(7.0)
    for t in range(steps):
        cr.cr_load_partial_grads(plan, G[0 if few else t])
        cr.cr_encode_tree(plan, masks[t])
        cr.cr_decode_root(plan, want[t])
    cr.cr_synchronize(plan)
    left = M.clone()
    M.fill_(7.0)
    cr.cr_aggregate_run(plan, G, masks, got, G_step_stride=0 if few else G.shape[1], g_step_stride=d)
    cr.cr_synchronize(plan)
    exact = d < 1_000_000                                # the wide encode of single calls and of runs is the same kernel too
    assert torch.equal(got, want) if exact else torch.allclose(got, want, rtol=1e-5)
    assert torch.equal(M, left)
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,d,steps", [(2, 3, 1, 100, 19), (2, 12, 2, 33_001, 3), (4, 3, 1, 40_004, 3), (2, 21, 1, 77, 18)])
def test_gd_run(L, n, s, d, steps):
    import torch

    N = sum(n ** l for l in range(1, L + 1))
    m = 2 * N
    plan = cr.cr_plan_ex(L, n, s, m, d)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, y, w0 = (torch.randn(shape, generator=gen, device="cuda") for shape in ((m, d), (m,), (d,)))
    masks, lr = _masks(np.random.default_rng(d), steps, N // n, n, s), 0.1 / (m + d)
    M, w, g = ws.messages(), w0.clone(), torch.empty(d, device="cuda")
    M.fill_(7.0)
    for t in range(steps):
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_encode_tree(plan, masks[t])
        cr.cr_decode_root(plan, g)
        cr.cr_gd_update(plan, w, g, lr)
    cr.cr_synchronize(plan)
    left = M.clone()
    M.fill_(7.0)
    w_run, g_run = w0.clone(), torch.empty(d, device="cuda")
    cr.cr_gd_run(plan, X, y, w_run, g_run, masks, lr)
    cr.cr_synchronize(plan)
    assert torch.equal(w, w_run) and torch.equal(g, g_run) and torch.equal(M, left)
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
def test_vectors_among_the_messages():
    """Slabs and decoded vectors of the caller's that lie in the message rows: every message is put down, as by the separate calls."""
    import torch

    n, d, steps = 4, 40, 3
    plan = cr.cr_plan_ex(1, n, 1, 8, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    G = torch.randn(steps, cr.cr_plan_info(plan).num_slabs * d, generator=torch.Generator(device="cuda").manual_seed(d), device="cuda")
    masks = np.zeros((steps, n), np.uint8)
    masks[0, 0] = masks[1, 1] = masks[2, 2] = 1
    M, g = ws.messages(), torch.empty(d, device="cuda")
    left = []
    for run in (False, True):
        M.fill_(7.0)
        if run:                                          # the second row of M is where every mask's gradient goes
            cr.cr_aggregate_run(plan, G, masks, M[1], G_step_stride=G.shape[1], g_step_stride=0)
        else:
            for t in range(steps):
                cr.cr_load_partial_grads(plan, G[t])
                cr.cr_encode_tree(plan, masks[t])
                cr.cr_decode_root(plan, g)
                M[1].copy_(g)
        cr.cr_synchronize(plan)
        torch.cuda.synchronize()
        left.append(M.clone())
    assert torch.equal(left[0], left[1])
    del ws
    cr.cr_plan_destroy(plan)


# where the vector lies among the messages: a first-level row, a row of a worker further down, between two rows
@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,d", [(2, 3, 1, 100), (2, 3, 1, 4_003), (1, 4, 1, 20_000), (2, 12, 2, 33_004)])
@pytest.mark.parametrize("place", ["first", "below", "between"])
def test_models_among_the_messages(L, n, s, d, place):
    """The model of a training run lies where messages are written: the steps start from what the separate calls would find there."""
    import torch

    if L == 1 and place != "first":
        pytest.skip("one level")
    N, steps = sum(n ** l for l in range(1, L + 1)), 3
    plan = cr.cr_plan_ex(L, n, s, 3 * N, d)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, y, w0 = (torch.randn(shape, generator=gen, device="cuda") for shape in ((3 * N, d), (3 * N,), (d,)))
    masks = _masks(np.random.default_rng(d), steps, N // n, n, s)
    at = {"first": d, "below": (N - 2) * d, "between": (N - 2) * d + d // 2 // 4 * 4}[place]
    w, g, left = ws.messages().view(-1)[at:at + d], torch.empty(d, device="cuda"), []
    for run in (False, True):
        ws.messages().fill_(7.0)
        w.copy_(w0)
        if run:
            cr.cr_gd_run(plan, X, y, w, g, masks, 1e-6)
        else:
            for t in range(steps):
                cr.cr_partial_grads(plan, X, y, w)
                cr.cr_encode_tree(plan, masks[t])
                cr.cr_decode_root(plan, g)
                cr.cr_gd_update(plan, w, g, 1e-6)
        cr.cr_synchronize(plan)
        left.append((ws.messages().clone(), g.clone()))
    assert torch.equal(left[0][0], left[1][0]) and torch.equal(left[0][1], left[1][1])
    del ws, w
    cr.cr_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,d", [(2, 3, 1, 100), (2, 3, 1, 4_003), (2, 12, 2, 33_001)])
def test_one_vector_for_two(L, n, s, d):
    """The reference model, the model and the gradient may be one vector: the values are those of a launch each for decode, step and measures."""
    import torch

    N, steps, lr = sum(n ** l for l in range(1, L + 1)), 3, 1e-6
    plan = cr.cr_plan_ex(L, n, s, 3 * N, d)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, y, w0 = (torch.randn(shape, generator=gen, device="cuda") for shape in ((3 * N, d), (3 * N,), (d,)))
    masks = _masks(np.random.default_rng(d), steps, N // n, n, s)
    metrics = torch.empty(steps, 2, device="cuda")
    for g_is_w, star in ((True, None), (False, "w"), (False, "g"), (True, "w")):
        want_w = w0.clone()
        want_g = want_w if g_is_w else torch.empty(d, device="cuda")
        want = []
        for t in range(steps):
            cr.cr_partial_grads(plan, X, y, want_w)
            cr.cr_encode_tree(plan, masks[t])
            cr.cr_decode_root(plan, want_g)
            cr.cr_synchronize(plan)
            before = want_w.double()
            cr.cr_gd_update(plan, want_w, want_g, lr)
            cr.cr_synchronize(plan)
            after = want_w.double()
            ref = {None: None, "w": after, "g": want_g.double()}[star]
            want.append([float((after - before).norm() ** 2 / before.norm() ** 2), -1.0 if ref is None else float((after - ref).norm() ** 2 / ref.norm() ** 2)])
        w = w0.clone()
        g = w if g_is_w else torch.empty(d, device="cuda")
        cr.cr_gd_run(plan, X, y, w, g, masks, lr, {None: None, "w": w, "g": g}[star], metrics)
        cr.cr_synchronize(plan)
        assert torch.equal(w, want_w) and torch.equal(g, want_g), (g_is_w, star)
        # sums of d squares in 64 bits, rounded to fp32 once
        assert np.allclose(metrics.cpu().numpy(), np.array(want), rtol=1e-6, atol=0.0), (g_is_w, star)
    del ws
    cr.cr_plan_destroy(plan)
