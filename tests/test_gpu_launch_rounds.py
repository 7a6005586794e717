"""Hop launches of several rounds of workgroups (long implicit lists) against one round of as many as stay resident: how
records are dealt out changes no sum, so the bits are the same."""
import numpy as np
import pytest
import torch

import paper_2207_12000_amd as gp

pytestmark = pytest.mark.gpu


# (rows, columns, type, operator): record counts around two, three and six rounds, with a last round that is not full,
# for groups of 8, 16 and 32 lanes, one and two column slices, weights and none
@pytest.mark.parametrize("n,d,dtype,agg", [(270_001, 24, torch.float32, gp.GP_AGG_SYM), (450_003, 20, torch.bfloat16, gp.GP_AGG_MEAN),
                                           (140_003, 128, torch.float32, gp.GP_AGG_SUM), (150_007, 47, torch.float32, gp.GP_AGG_SYM)])
def test_rounds_change_no_bit(n, d, dtype, agg):
    rng = np.random.default_rng(n)
    src, dst = (rng.integers(0, n, 2 * n).astype(np.int32) for _ in range(2))
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()
    stacks = []
    for blocks in (0, 512):
        gp.gp_set_option("persistent_blocks", blocks)
        try:
            with gp.gp_plan_blocks(src, dst, n, 1 << 19, gp.GP_SYMMETRISE) as plan:
                stacks.append(gp.propagate_tensors(plan, X, agg, 2).view(torch.int16 if dtype == torch.bfloat16 else torch.int32).cpu())
        finally:
            gp.gp_set_option("persistent_blocks", 0)
    assert torch.equal(*stacks)
