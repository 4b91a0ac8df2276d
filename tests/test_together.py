"""Encode, decode and gradient step in one launch, and apart where vectors are longer: cr_gd_run and cr_aggregate_static on both sides
of every rule against the separate calls (the same bits), the convergence measures against 64 bits."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

pytestmark = pytest.mark.gpu

WIDTHS = [1, 3, 4, 31, 33, 1_030, 8_192, 8_195, 32_768, 32_771, 40_001, 81_925]


def _masks(rng, steps, groups, n, s):
    masks = np.zeros((steps, groups * n), dtype=np.uint8)
    for t in range(steps):
        for g in range(groups):
            masks[t, g * n + rng.choice(n, size=int(rng.integers(0, s + 1)), replace=False)] = 1
    return masks


@pytest.mark.parametrize("d", WIDTHS)
# 155 workers whose sub-trees leave a compute unit less LDS than five workgroups need; 462: more than kernel arguments hold
@pytest.mark.parametrize("L,n,s", [(2, 3, 1), (3, 5, 1), (2, 21, 0)])
def test_steps_of_a_run(L, n, s, d):
    import torch

    N = sum(n ** l for l in range(1, L + 1))
    m = 4 * N
    if m * d > 1 << 26:
        m = N
    plan = cr.cr_plan_ex(L, n, s, m, d)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, y, w0, w_star = (torch.randn(shape, generator=gen, device="cuda") for shape in ((m, d), (m,), (d,), (d,)))
    steps, lr = 18, 0.1 / (m + d)                        # more steps than go into one batch of measures
    masks = _masks(np.random.default_rng(d), steps, ws.info.num_groups, n, s)
    w, g = w0.clone(), torch.empty(d, device="cuda")
    want = []
    for t in range(steps):
        before = w.double()
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_encode_tree(plan, masks[t])
        cr.cr_decode_root(plan, g)
        cr.cr_gd_update(plan, w, g, lr)
        want.append([float((w.double() - before).pow(2).sum() / before.pow(2).sum()), float((w.double() - w_star.double()).pow(2).sum() / w_star.double().pow(2).sum())])
    messages = ws.messages().clone()
    for measured in (False, True):
        w_run, g_run = w0.clone(), torch.full((d + 4,), 7.0, device="cuda")
        metrics = torch.full((steps + 1, 2), 7.0, device="cuda") if measured else None
        cr.cr_gd_run(plan, X, y, w_run, g_run, masks, lr, w_star if measured else None, metrics)
        cr.cr_synchronize(plan)
        assert torch.equal(w, w_run) and torch.equal(g, g_run[:d]) and bool((g_run[d:] == 7.0).all())
        assert torch.equal(ws.messages(), messages)
    # sums and quotient in 64 bits, rounded to fp32
    np.testing.assert_allclose(metrics[:steps].cpu().numpy(), np.array(want), rtol=2.0 ** -22)
    assert bool((metrics[steps] == 7.0).all())
    del ws
    cr.cr_plan_destroy(plan)


# two and many distinct coefficients; (3, 6): more than fit; widths at which only some of the calls have the nodes side by side
STATIC = [(*tree, d) for tree in [(2, 12, 2), (3, 6, 2), (3, 4, 1), (2, 8, 2)] for d in WIDTHS]
STATIC += [(2, 12, 5, 81_920), (3, 4, 1, 65_536), (3, 4, 1, 65_537), (4, 2, 1, 81_920), (4, 3, 1, 32_769), (1, 10, 4, 81_920)]


@pytest.mark.parametrize("L,n,s,d", STATIC)
def test_static_aggregation(L, n, s, d):
    import torch

    plan = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
    info = cr.cr_plan_info(plan)
    ws = cr.Workspace(plan)
    G = torch.randn(info.num_slabs, d, device="cuda")
    want, got = torch.empty(d, device="cuda"), torch.full((d + 4,), 7.0, device="cuda")
    for mask in _masks(np.random.default_rng(d), 2, info.num_groups, n, s):
        cr.cr_load_partial_grads(plan, G)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, want)
        cr.cr_aggregate_static(plan, G, mask, got, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(got[:d], want) and bool((got[d:] == 7.0).all())
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.parametrize("L,n,s,d,steps", [(2, 3, 1, 3, 5), (2, 12, 5, 1_003, 19), (2, 3, 1, 32_769, 17), (1, 33, 1, 33_000, 2), (1, 32, 1, 33_001, 3), (3, 4, 1, 40_003, 2),
                                            (4, 2, 1, 40_003, 2), (2, 8, 1, 81_921, 1), (2, 5, 1, 838_861, 1), (2, 4, 1, 1_048_580, 1), (2, 2, 0, 4_194_305, 2)])
def test_runs_of_masks(L, n, s, d, steps):
    """Both sides of the rules for one launch per mask, one for all of them, and two per mask: three calls per mask give the same bits.
    The masks' vectors lie apart, with gaps that stay as they were."""
    import torch

    plan = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    S = ws.info.num_slabs
    stride, apart = (S * d + 3) // 4 * 4 + 8, d + 5
    G = torch.randn(steps * stride, device="cuda")
    g = torch.full((steps, apart), 7.0, device="cuda")
    masks = _masks(np.random.default_rng(d), steps, ws.info.num_groups, n, s)
    want, M = torch.empty(d, device="cuda"), ws.messages()
    M.zero_()
    cr.cr_aggregate_run(plan, G, masks, g, G_step_stride=stride, g_step_stride=apart)
    after = M.clone()
    M.zero_()
    for t in range(steps):
        cr.cr_load_partial_grads(plan, G[t * stride:t * stride + S * d])
        cr.cr_encode_tree(plan, masks[t])
        cr.cr_decode_root(plan, want)
        assert torch.equal(want, g[t, :d]) and bool((g[t, d:] == 7.0).all()), t
    assert torch.equal(M, after)
    again = torch.empty(d, device="cuda")                # the plan is left as the last mask's calls leave it
    cr.cr_aggregate_run(plan, G, masks, g, G_step_stride=stride, g_step_stride=apart)
    cr.cr_decode_root(plan, again)
    assert torch.equal(again, want)
    del ws
    cr.cr_plan_destroy(plan)


# one launch per mask; the nodes side by side and a decode; programs and a decode; all masks in one launch
LAUNCHES = [(2, 12, 5, 32_768, 3, 3, 0), (3, 6, 2, 8_192, 3, 3, 0), (3, 6, 2, 8_193, 3, 3, 3), (6, 2, 1, 32_768, 3, 3, 3), (2, 17, 1, 32_768, 3, 3, 0), (2, 20, 1, 1_003, 3, 3, 3), (2, 24, 1, 1_003, 3, 3, 3), (3, 8, 2, 32_768, 2, 2, 2), (2, 24, 1, 32_769, 3, 1, 0),
            (2, 12, 5, 65_536, 2, 1, 0), (2, 12, 5, 65_537, 2, 2, 2), (2, 8, 2, 65_537, 2, 1, 0), (2, 12, 5, 98_305, 2, 1, 0), (2, 12, 5, 131_073, 2, 2, 2),
            (3, 5, 1, 131_073, 2, 1, 0), (3, 4, 1, 400_001, 2, 1, 0), (2, 17, 1, 235_000, 2, 1, 0), (2, 12, 1, 40_001, 1, 1, 1), (2, 12, 1, 90_001, 1, 1, 0), (2, 12, 5, 81_920, 1, 1, 1),
            (2, 12, 1, 40_001, 17, 2, 1), (4, 2, 1, 40_001, 3, 3, 3), (1, 33, 1, 40_001, 3, 3, 3)]


@pytest.mark.parametrize("L,n,s,d,steps,encodes,decodes", LAUNCHES)
def test_launches_of_a_run(L, n, s, d, steps, encodes, decodes):
    """Which launches a call over several masks takes on both sides of its rules (a launch that does the work of several counts as the
    encode's), with the same bits as three calls per mask: all masks on the same slabs, into the same vector."""
    import torch

    plan = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    G, g, want = torch.randn(ws.info.num_slabs, d, device="cuda"), torch.empty(d, device="cuda"), torch.empty(d, device="cuda")
    masks, M = _masks(np.random.default_rng(d), steps, ws.info.num_groups, n, s), ws.messages()
    M.zero_()
    cr.cr_profile_enable(plan, True)
    cr.cr_aggregate_run(plan, G, masks, g)
    assert (cr.cr_profile_read(plan, cr.CR_K_ENCODE)[1], cr.cr_profile_read(plan, cr.CR_K_DECODE)[1]) == (encodes, decodes)
    cr.cr_profile_enable(plan, False)
    after = M.clone()
    M.zero_()
    for mask in masks:
        cr.cr_load_partial_grads(plan, G)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, want)
    cr.cr_synchronize(plan)
    assert torch.equal(g, want) and torch.equal(M, after)
    del ws
    cr.cr_plan_destroy(plan)
