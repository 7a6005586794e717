"""Plans made on the GPU from lists long enough to be checked and copied beside each other: the host planner's arrays where
pairs give no candidates or the same ones over and over, and its refusal of an id out of range."""
import numpy as np
import pytest

import oracle
import paper_2207_12000_amd as gp
from test_plan_parity import assert_same_plan, check_schedule

pytestmark = pytest.mark.gpu

M = (1 << 18) + 17  # (shorter lists are planned without a second thread)


@pytest.mark.parametrize("kind", ["self pairs", "one pair", "some self pairs", "distinct"])
@pytest.mark.parametrize("flags", [0, gp.GP_SYMMETRISE | gp.GP_ADD_SELF_LOOPS])
def test_the_hosts_plan(kind, flags):
    rng = np.random.default_rng(3)
    n = 50_000
    src, dst = (rng.integers(0, n, M).astype(np.int32) for _ in range(2))
    if kind == "self pairs":
        dst = src.copy()
    if kind == "one pair":
        src[:], dst[:] = 7, n - 1
    if kind == "some self pairs":
        dst = np.where(rng.random(M) < 0.5, src, dst).astype(np.int32)
    with gp.gp_plan_blocks(src, dst, n, 100_000, flags | gp.GP_PLAN_ON_DEVICE) as plan:
        assert_same_plan(plan, oracle.plan_blocks(src, dst, n, 100_000, flags))
        check_schedule(plan, plan.segment_edges)


@pytest.mark.parametrize("at,bad", [(0, -1), (M - 1, 50_000)])
def test_an_id_out_of_range_is_refused(at, bad):
    src = np.arange(M, dtype=np.int32) % 50_000
    dst = src[::-1].copy()
    dst[at] = bad
    with pytest.raises(gp.GpError, match=f"pair {at} = "):
        gp.gp_plan_blocks(src, dst, 50_000, 100_000, gp.GP_SYMMETRISE | gp.GP_PLAN_ON_DEVICE)
