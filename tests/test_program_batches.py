"""More masks than two batches of programs hold, on the routes that take programs: the host builds the third batch in the pinned half whose
copy to the device has to be done first.  Every mask differs, so that a program of another step shows."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

pytestmark = pytest.mark.gpu


def _masks(rng, steps, groups, n, s):
    masks = np.zeros((steps, groups * n), dtype=np.uint8)
    for t in range(steps):
        for g in range(groups):
            masks[t, g * n + rng.choice(n, size=s, replace=False)] = 1
    masks[5, ::n] = 0                                    # fewer than s stragglers in some groups of one step
    return masks


@pytest.mark.parametrize("L,n,s,d", [(2, 3, 1, 40_003), (2, 21, 1, 1_003)])
def test_training(L, n, s, d):
    """40 steps of cr_gd_run, encode from programs, against the separate calls: the same bits, in one call and in two."""
    import torch

    N = sum(n ** l for l in range(1, L + 1))
    plan = cr.cr_plan_ex(L, n, s, N, d)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, y, w0 = (torch.randn(shape, generator=gen, device="cuda") for shape in ((N, d), (N,), (d,)))
    steps, lr = 40, 0.1 / (N + d)
    masks = _masks(np.random.default_rng(d), steps, ws.info.num_groups, n, s)
    w, g = w0.clone(), torch.empty(d, device="cuda")
    for mask in masks:
        cr.cr_partial_grads(plan, X, y, w)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, g)
        cr.cr_gd_update(plan, w, g, lr)
    for cuts in ((0, 40), (0, 23, 40)):
        w_run, g_run = w0.clone(), torch.empty(d, device="cuda")
        for lo, hi in zip(cuts, cuts[1:]):
            cr.cr_gd_run(plan, X, y, w_run, g_run, masks[lo:hi], lr)
        cr.cr_synchronize(plan)
        assert torch.equal(w_run, w) and torch.equal(g_run, g), cuts
    del ws
    cr.cr_plan_destroy(plan)


@pytest.mark.parametrize("L,n,s,d", [(2, 3, 1, 32_771), (2, 24, 1, 1_003), (2, 24, 1, 3), (3, 6, 2, 73_730)])    # all masks in one launch; launches per mask
@pytest.mark.parametrize("per_step", [False, True])
def test_aggregation(L, n, s, d, per_step):
    import torch

    plan = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    S, steps = ws.info.num_slabs, 37
    masks, stride = _masks(np.random.default_rng(d), steps, ws.info.num_groups, n, s), (S * d + 3) // 4 * 4
    G = torch.randn(steps * stride if per_step else stride, device="cuda")
    want, got, M = torch.empty(steps, d, device="cuda"), torch.full((steps, d), 7.0, device="cuda"), ws.messages()
    M.zero_()
    for t, mask in enumerate(masks):
        cr.cr_load_partial_grads(plan, G[t * stride:] if per_step else G)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, want[t])
    messages = M.clone()
    M.zero_()
    cr.cr_aggregate_run(plan, G, masks, got, G_step_stride=stride if per_step else 0, g_step_stride=d)
    cr.cr_synchronize(plan)
    assert torch.equal(got, want) and torch.equal(M, messages)
    one = torch.empty(d, device="cuda")                  # every mask into the same vector: the last one stays
    cr.cr_aggregate_run(plan, G, masks, one, G_step_stride=stride if per_step else 0)
    cr.cr_synchronize(plan)
    assert torch.equal(one, want[-1]) and torch.equal(M, messages)
    del ws
    cr.cr_plan_destroy(plan)
