"""Encode and decode at the edges of their kernels: groups of lanes and of columns that do not fill up, widths on both sides of every
rule, trees of the most nodes that kernel arguments hold and of one more, deep and wide trees, masks with fewer than s stragglers.
The reference is the tree walked in 64 bits with messages rounded to fp32 where they are sent."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

pytestmark = pytest.mark.gpu

# 448 nodes travel as kernel arguments: (n, L) of 420 and 399 nodes and of 462; trees whose sub-tree takes 33 KB and more than 64 KB of LDS;
# groups of 64; one level; eight levels
CASES = [(2, 3, 1, d) for d in (1, 3, 4, 5, 63, 64, 65, 67, 1_023, 1_028)]
CASES += [(1, 2, 0, 100), (1, 64, 1, 130), (1, 10, 4, 1_027), (2, 20, 1, 77), (2, 21, 1, 77), (3, 7, 2, 70), (3, 6, 2, 1_024), (6, 2, 1, 66), (7, 2, 1, 66), (8, 2, 1, 66)]
CASES += [(2, 20, 1, 16_384), (2, 20, 1, 16_385), (3, 5, 4, 65_537), (3, 4, 1, 81_920), (4, 3, 1, 49_152), (4, 3, 1, 49_153), (2, 17, 1, 49_153)]
CASES += [(2, 12, 3, 5_001), (3, 3, 1, 32_768), (3, 3, 1, 32_769), (2, 4, 1, 81_920), (2, 4, 1, 81_921), (2, 8, 2, 81_919), (1, 3, 1, 2_097_151), (1, 3, 1, 2_097_155)]


def _mask(rng, groups, n, s, fewer):
    mask = np.zeros(groups * n, dtype=np.uint8)
    for g in range(groups):
        count = int(rng.integers(0, s + 1)) if fewer else s
        mask[g * n + rng.choice(n, size=count, replace=False)] = 1
    return mask


def _reference(plan, G, mask):
    """(messages, rows of stragglers None; decoded gradient) in 64 bits, every message rounded to fp32."""
    info = cr.cr_plan_info(plan)
    n, N = info.n, info.num_workers
    _, _, coef, worker = cr.cr_plan_get_segments(plan)
    G = G.astype(np.float64)
    own = [coef[worker == k] @ G[worker == k] if (worker == k).any() else np.zeros(G.shape[1]) for k in range(N)]
    row = [cr.cr_plan_decode_row(plan, mask[g * n:(g + 1) * n]) for g in range(N // n)]
    msg = [None] * N
    for k in range(N - 1, -1, -1):                       # children have higher ids: node k's are the group (k + 1)
        if mask[k]:
            continue
        total = own[k]
        for c in range((k + 1) * n, min((k + 2) * n, N)):
            if not mask[c]:
                total = total + row[k + 1][c % n] * msg[c].astype(np.float64)
        msg[k] = total.astype(np.float32)
    return msg, sum(row[0][j] * msg[j].astype(np.float64) for j in range(n) if not mask[j])


def _close(got, ref):
    # both sides round the same 64-bit sums once; a sum next to a tie may fall on either side of it
    assert np.all(np.abs(got - ref) <= 2.0 ** -22 * (np.abs(ref) + np.sqrt(np.mean(np.square(ref))))), np.abs(got - ref).max()


@pytest.mark.parametrize("L,n,s,d", CASES)
def test_messages_and_decode(L, n, s, d):
    import torch

    plan = cr.cr_plan_ex(L, n, s, 6 * sum(n ** l for l in range(1, L + 1)), d, model=cr.CR_AGGREGATE_ONLY)
    info = cr.cr_plan_info(plan)
    ws = cr.Workspace(plan)
    rng = np.random.default_rng(d * 100 + n)
    G = torch.from_numpy(rng.standard_normal((info.num_slabs, d), dtype=np.float32)).cuda()
    g = torch.empty(d + 4, device="cuda")
    for fewer in (False, True):
        mask = _mask(rng, info.num_groups, n, s, fewer)
        M = ws.messages()
        M.fill_(7.0)                                     # stragglers' rows keep what they held
        g.fill_(7.0)
        cr.cr_load_partial_grads(plan, G)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, g)
        cr.cr_synchronize(plan)
        msg, ref = _reference(plan, G.cpu().numpy(), mask)
        M = M.cpu().numpy()
        for k in range(info.num_workers):
            if mask[k]:
                assert np.all(M[k] == 7.0)
            else:
                _close(M[k].astype(np.float64), msg[k].astype(np.float64))
        _close(g[:d].cpu().numpy().astype(np.float64), ref)
        assert bool((g[d:] == 7.0).all())
    cr.cr_plan_destroy(plan)


def test_a_bad_mask_enqueues_nothing():
    import torch

    plan = cr.cr_plan_ex(2, 4, 1, 100, 50, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    G = torch.randn(cr.cr_plan_info(plan).num_slabs, 50, device="cuda")
    g = torch.zeros(50, device="cuda")
    good = np.zeros(20, dtype=np.uint8)
    good[2] = 1
    cr.cr_load_partial_grads(plan, G)
    cr.cr_encode_tree(plan, good)
    before = ws.messages().clone()
    bad = good.copy()
    bad[16:18] = 1
    with pytest.raises(cr.CodedReduceError) as e:
        cr.cr_encode_tree(plan, bad)
    assert e.value.status == cr.CR_E_UNDECODABLE
    cr.cr_decode_root(plan, g)                           # still of the good mask
    cr.cr_synchronize(plan)
    assert torch.equal(ws.messages(), before) and bool((g != 0).any())
    cr.cr_plan_destroy(plan)


@pytest.mark.parametrize("d", [2_097_149, 2_098_179])
def test_gradient_step_in_the_decode_of_long_vectors(d):
    """The gradient step that rides in the decode launch, on both sides of the decode's rule and with columns that two chunks share,
    against the update call."""
    import torch

    m = 6
    plan = cr.cr_plan_ex(1, 2, 0, m, d)
    ws = cr.Workspace(plan)
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, y, w = (torch.randn(shape, generator=gen, device="cuda") for shape in ((m, d), (m,), (d,)))
    g, w_ref = torch.empty(d, device="cuda"), w.clone()
    mask = np.zeros((1, 2), dtype=np.uint8)
    cr.cr_partial_grads(plan, X, y, w_ref)
    cr.cr_encode_tree(plan, mask[0])
    cr.cr_decode_root(plan, g)
    cr.cr_gd_update(plan, w_ref, g, 1e-7)
    g_run = torch.empty_like(g)
    cr.cr_gd_run(plan, X, y, w, g_run, mask, 1e-7)
    torch.cuda.synchronize()
    assert torch.equal(g, g_run) and torch.equal(w, w_ref)
    del ws
    cr.cr_plan_destroy(plan)
