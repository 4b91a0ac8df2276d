"""Calls on slab gradients of the caller's rely on nothing that the workspace held before: plans of different trees take turns in one
block, and a block that was overwritten serves the next call.  Trees whose tables fit kernel arguments, whose tables fit with some masks
only, and whose tables never do; encode and decode in one launch, apart, and from programs."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

pytestmark = pytest.mark.gpu

TREES = [(2, 4, 1), (2, 12, 2), (2, 12, 1), (3, 6, 2), (2, 21, 1)]


def _mask(rng, groups, n, s):
    mask = np.zeros(groups * n, dtype=np.uint8)
    for g in range(groups):
        mask[g * n + rng.choice(n, size=s, replace=False)] = 1
    return mask


def _one(plan, G, masks, g):
    """Three calls for the first mask, one for all of them; returns every result."""
    cr.cr_load_partial_grads(plan, G)
    cr.cr_encode_tree(plan, masks[0])
    cr.cr_decode_root(plan, g[0])
    cr.cr_aggregate_run(plan, G, masks, g[1:], g_step_stride=g.shape[1])
    cr.cr_synchronize(plan)
    return g.clone()


@pytest.mark.parametrize("d", [1_003, 32_771, 81_925])
def test_plans_take_turns_in_one_block(d):
    import torch

    rng = np.random.default_rng(d)
    work = []
    for L, n, s in TREES:
        plan = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
        ws = cr.Workspace(plan)
        info = ws.info
        G = torch.randn(info.num_slabs, d, device="cuda")
        masks = np.stack([_mask(rng, info.num_groups, n, s) for _ in range(3)])
        g = torch.empty(4, d, device="cuda")
        work.append((plan, G, masks, g, _one(plan, G, masks, g)))     # alone in a block of its own
        del ws
    size = max(cr.cr_workspace_bytes(w[0]) for w in work)
    block = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
    base = (block.data_ptr() + 255) // 256 * 256
    for plan, *_ in work:
        cr.cr_bind_workspace(plan, base, size, torch.cuda.current_stream().cuda_stream)
    for _ in range(2):
        for plan, G, masks, g, want in work:
            g.fill_(float("nan"))
            assert torch.equal(_one(plan, G, masks, g), want)
            block.fill_(0xff)
    for plan, *_ in work:
        cr.cr_plan_destroy(plan)


def test_more_plans_than_the_library_keeps_tables_for():
    """Each of these trees' tables takes two of the 256 pages: the last plans' travel with the calls.  Destroyed plans give theirs back."""
    import torch

    d = 1_003
    for L, n, s in [(2, 12, 1), (3, 6, 2)]:              # tables that fit the arguments with some masks, and with none
        first = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
        B = cr.cr_plan_get_B(first)
        plans = [first] + [cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY, B=B) for _ in range(139)]
        info = cr.cr_plan_info(first)
        size = cr.cr_workspace_bytes(first)
        block = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        G = torch.randn(info.num_slabs, d, device="cuda")
        rng = np.random.default_rng(n)
        masks = np.stack([_mask(rng, info.num_groups, n, s) for _ in range(5)])
        g = torch.empty(6, d, device="cuda")
        for plan in plans:
            cr.cr_bind_workspace(plan, (block.data_ptr() + 255) // 256 * 256, size, torch.cuda.current_stream().cuda_stream)
        want = _one(first, G, masks, g)
        for plan in plans[1:3] + plans[-3:]:
            block.fill_(0xff)
            g.fill_(float("nan"))
            assert torch.equal(_one(plan, G, masks, g), want)
        for plan in plans:
            cr.cr_plan_destroy(plan)


@pytest.mark.parametrize("L,n,s", [(2, 12, 2), (3, 6, 2)])
def test_a_regression_plan_with_gradients_of_the_callers(L, n, s):
    import torch

    d, m = 1_003, 40 * n ** L
    plan = cr.cr_plan_ex(L, n, s, m, d)
    ws = cr.Workspace(plan)
    info = ws.info
    masks = np.stack([_mask(np.random.default_rng(t), info.num_groups, n, s) for t in range(3)])
    X, y, w = torch.randn(m, d, device="cuda"), torch.randn(m, device="cuda"), torch.randn(d, device="cuda")
    g = torch.empty(4, d, device="cuda")
    cr.cr_partial_grads(plan, X, y, w)                   # the workspace's own slabs first ...
    G = ws.slab_grads().clone()
    cr.cr_encode_tree(plan, masks[0])
    cr.cr_decode_root(plan, g[0])
    cr.cr_synchronize(plan)
    want = g[0].clone()
    ws.buffer.fill_(0xff)
    results = _one(plan, G, masks, g)                    # ... and the same as the caller's, in a block that was overwritten
    assert torch.equal(results[0], want) and torch.equal(results[1], want)
    del ws
    cr.cr_plan_destroy(plan)
