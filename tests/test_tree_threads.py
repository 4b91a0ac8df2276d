"""Workgroups of the tree kernels have as many threads as nodes give work to and the chip holds at once: sizes on both sides of those lines,
against a launch per stage and 64 bits."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

# four chunks per workgroup up to 2 048 columns (and not on small trees), one, two and three workgroups per compute unit (16 chunks: 256 * 64
# columns each), fewer threads than 64, more nodes than teams, 64 chunks from 3 073 columns on or where every node has a wavefront, the
# lines between nodes side by side and a walk, as many nodes as the short arguments hold and one more
CASES = [(2, 12, 2, d) for d in (4, 5, 2_047, 2_048, 2_049, 16_384, 16_385, 32_767)] + [(3, 6, 2, d) for d in (9, 2_048, 2_053, 4_097)] + \
        [(3, 4, 1, 163_840), (3, 4, 1, 163_841), (2, 8, 2, 131_073), (1, 10, 4, 163_843), (3, 6, 2, 40_961), (4, 3, 1, 49_153), (2, 12, 2, 98_305)] + \
        [(1, 48, 1, 70), (1, 49, 1, 70), (1, 20, 1, 70), (1, 32, 1, 70), (3, 3, 1, 5_001), (5, 2, 1, 70)] + \
        [(3, 5, 1, 3_072), (3, 5, 1, 3_073), (4, 2, 1, 300), (2, 3, 1, 2_047), (1, 64, 1, 1_023), (1, 2, 1, 12), (3, 5, 1, 1_031), (5, 2, 1, 6_501), (2, 17, 1, 2_048)]


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s,d", CASES)
def test_one_launch_and_two_give_the_same_bits(L, n, s, d):
    import torch

    N = sum(n ** l for l in range(1, L + 1))
    plan = cr.cr_plan_ex(L, n, s, 3 * N, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    S = cr.cr_plan_info(plan).num_slabs
    rb, re_, coef, worker = cr.cr_plan_get_segments(plan)
    cuts = np.unique(np.concatenate([rb, re_]))
    atoms = torch.randn(len(cuts) - 1, d, generator=gen, device="cuda", dtype=torch.float64)
    lo, hi = np.searchsorted(cuts, rb), np.searchsorted(cuts, re_)
    G = torch.zeros(2, (S * d + 3) // 4 * 4, device="cuda")
    for q in range(S):
        G[:, q * d:(q + 1) * d] = atoms[lo[q]:hi[q]].sum(0).float()
    G[1] *= -2.0
    rng = np.random.default_rng(d)
    masks = np.zeros((2, N), np.uint8)
    for t in range(2):
        for grp in range(N // n):
            masks[t, grp * n + rng.choice(n, s, replace=False)] = 1
    g = torch.full((2, d), float("nan"), device="cuda")
    cr.cr_aggregate_run(plan, G, masks, g, G_step_stride=G.shape[1], g_step_stride=d)
    cr.cr_synchronize(plan)
    messages = ws.messages().clone()
    h = torch.full((d,), float("nan"), device="cuda")
    for t in range(2):
        cr.cr_load_partial_grads(plan, G[t])
        cr.cr_encode_tree(plan, masks[t])
        cr.cr_decode_root(plan, h)
        cr.cr_synchronize(plan)
        assert torch.equal(h, g[t])
        if 4 * N * d <= 90_000_000:
            h.fill_(float("nan"))
            cr.cr_aggregate_static(plan, G[t], masks[t], h, torch.cuda.current_stream().cuda_stream)
            assert torch.equal(h, g[t])
    sends = torch.from_numpy(masks[1] == 0).cuda()
    assert torch.equal(ws.messages()[sends], messages[sends])
    # what is decoded is the sum over all rows; the code amplifies the messages' rounding by gamma per level
    total = atoms.sum(0)
    bound = 2.0 ** -24 * cr.cr_plan_info(plan).gamma ** L * 8
    for t, factor in ((0, 1.0), (1, -2.0)):
        assert float((g[t].double() - factor * total).norm() / total.norm()) <= max(bound, 1e-6)
    del ws
    cr.cr_plan_destroy(plan)
