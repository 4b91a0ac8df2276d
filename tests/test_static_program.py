"""cr_aggregate_static sends its encode program in blocks of kernel arguments: programs of one block and of several, codes with few and
with many distinct coefficients, tables of the widest group, against the three separate calls, whose program travels by copy."""
import numpy as np
import pytest

import paper_1902_01981_amd as cr

# (L, n, s): one short block; two coefficients in all; a coefficient of its own for most terms; several blocks; a group of 64 members
TREES = [(1, 2, 0), (2, 3, 1), (2, 12, 2), (2, 12, 1), (1, 10, 4), (3, 6, 2), (4, 3, 1), (1, 64, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("L,n,s", TREES)
@pytest.mark.parametrize("d", [5, 1_030])
def test_program_blocks(L, n, s, d):
    """The same kernels run on the same tables, so the gradients have the same bits."""
    import torch

    plan = cr.cr_plan_ex(L, n, s, 40 * n ** L, d, model=cr.CR_AGGREGATE_ONLY)
    info = cr.cr_plan_info(plan)
    ws = cr.Workspace(plan)
    rng = np.random.default_rng(L * 1_000 + n * 10 + s)
    G = torch.randn(info.num_slabs, d, device="cuda")
    want, got = torch.empty(d, device="cuda"), torch.empty(d, device="cuda")
    for stragglers in {0, s}:
        mask = np.zeros(info.num_workers, dtype=np.uint8)
        for g in range(info.num_groups):
            mask[g * n + rng.choice(n, size=stragglers, replace=False)] = 1
        ws.messages().zero_()
        cr.cr_load_partial_grads(plan, G)
        cr.cr_encode_tree(plan, mask)
        cr.cr_decode_root(plan, want)
        got.fill_(float("nan"))
        cr.cr_aggregate_static(plan, G, mask, got, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    cr.cr_plan_destroy(plan)
