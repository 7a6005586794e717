"""Hop launches of several rounds of workgroups (long implicit lists) against one round of as many as stay resident: how
records are dealt out changes no sum, so the bits are the same."""
import json

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


MOST_RESIDENT = 256 * 8  # workgroups of four wavefronts, at most eight wavefronts on a SIMD


def hop_grids(call, path):
    """The workgroups of every hop launch that call() makes."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    p.export_chrome_trace(str(path))
    events = json.loads(path.read_text())["traceEvents"]
    return [e["args"]["grid"][0] for e in events if "gp_hop_segments" in e.get("name", "") and "grid" in e.get("args", {})]


def both_ways(n, pairs, d, dtype, agg, path):
    """The stack with workgroups as the library has them and with 512, and the grids of the first's hop launches."""
    rng = np.random.default_rng(n)
    src, dst = (rng.integers(0, n, pairs).astype(np.int32) for _ in range(2))
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()
    stacks, grids = [], []
    for blocks in (0, 512):
        gp.gp_set_option("persistent_blocks", blocks)
        try:
            with gp.gp_plan_blocks(src, dst, n, 1 << 19, gp.GP_SYMMETRISE) as plan:
                stacks.append(gp.propagate_tensors(plan, X, agg, 2).view(torch.int16 if dtype == torch.bfloat16 else torch.int32).cpu())
                grids.append(hop_grids(lambda: gp.propagate_tensors(plan, X, agg, 2), path))
        finally:
            gp.gp_set_option("persistent_blocks", 0)
    assert torch.equal(*stacks) and len(grids[0]) == 2 and grids[1] == [512, 512]
    return grids[0]


# (rows, columns, type, operator): four rounds and more (eight records per group, of twenty non-zeros) whatever the occupancy,
# with a last round that is not full, for groups of 8, 16 and 32 lanes, weights and none, rows read where they lie and from copies
@pytest.mark.parametrize("n,d,dtype,agg", [(530_001, 24, torch.float32, gp.GP_AGG_SYM), (530_003, 20, torch.bfloat16, gp.GP_AGG_MEAN),
                                           (140_003, 128, torch.float32, gp.GP_AGG_SUM), (270_007, 47, torch.float32, gp.GP_AGG_SYM)])
def test_four_rounds_and_more_are_made(n, d, dtype, agg, tmp_path):
    assert min(both_ways(n, 10 * n, d, dtype, agg, tmp_path / "trace.json")) > MOST_RESIDENT


# records of two to four non-zeros, and rows of 9 to 16 bf16 elements off a dword: one round
@pytest.mark.parametrize("n,mean,d,dtype", [(600_001, 2, 16, torch.float32), (530_001, 4, 24, torch.bfloat16), (300_001, 16, 9, torch.bfloat16)])
def test_short_records_get_one_round(n, mean, d, dtype, tmp_path):
    assert max(both_ways(n, mean * n // 2, d, dtype, gp.GP_AGG_SUM, tmp_path / "trace.json")) <= MOST_RESIDENT
