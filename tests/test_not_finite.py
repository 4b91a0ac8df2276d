"""Gradients that are not finite stay where they belong: below a straggler they reach no other node's message and not the decoded
vector.  On every route of the encode: side by side, walked from programs, many masks in one launch, and without an allocation."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1_003, 32_771, 81_925])
@pytest.mark.parametrize("L,n,s,m", [(2, 4, 1, 400), (3, 4, 1, 400), (3, 6, 2, 258), (4, 2, 1, 30), (3, 8, 2, 584)])
def test_below_a_straggler(L, n, s, m, d):
    import torch

    plan = cr.cr_plan_ex(L, n, s, m, d, model=cr.CR_AGGREGATE_ONLY)
    ws = cr.Workspace(plan)
    N, worker = ws.info.num_workers, cr.cr_plan_get_segments(plan)[3]
    mask = np.zeros(N, dtype=np.uint8)
    mask[0::n] = 1                                       # the first child of every parent, which comes before its siblings
    first = [n * (n ** l - 1) // (n - 1) for l in range(L + 1)]      # id of the first node of level l + 1
    below = set()                                        # of the first child of (1, 1), and of (1, 0)
    for l in range(1, L):
        below |= set(range(first[l], first[l] + n ** l)) | (set(range(first[l] + n ** l, first[l] + n ** l + n ** (l - 1))) if l > 1 else set())
    finite = torch.randn(len(worker), d, device="cuda")
    G = finite.clone()
    for q, k in enumerate(worker):
        if int(k) in below or mask[k]:
            G[q] = float("inf") if q % 2 else float("nan")
    g, want, M = torch.empty(3, d, device="cuda"), torch.empty(d, device="cuda"), ws.messages()

    def calls(slabs, out):
        M.zero_()
        cr.cr_load_partial_grads(plan, slabs)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, out)
        return M.clone()

    clean = calls(finite, want)
    assert bool(torch.isfinite(clean).all())
    kept = torch.tensor([k not in below for k in range(N)], device="cuda")
    calls_M = calls(G, g[0])
    M.zero_()
    cr.cr_aggregate_run(plan, G, np.stack([mask, mask]), g[1])
    run_M = M.clone()
    if N * d * 4 < 1 << 26 and N < 500:                  # within the call's limits
        cr.cr_aggregate_static(plan, G, mask, g[2], torch.cuda.current_stream().cuda_stream)
    else:
        g[2] = want
    torch.cuda.synchronize()
    for name, vector, messages in (("calls", g[0], calls_M), ("run", g[1], run_M), ("static", g[2], clean)):
        assert torch.equal(vector, want), name
        assert torch.equal(messages[kept], clean[kept]), name
    del ws
    cr.cr_plan_destroy(plan)
