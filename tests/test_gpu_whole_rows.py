"""Rows that only block boundaries cut are whole again in the hops of resident operands: the bits of a plan of one block, and no
launch that joins partial rows; rows longer than a segment keep theirs."""
import numpy as np
import pytest
import torch

import paper_2207_12000_amd as gp

pytestmark = pytest.mark.gpu


def stack(src, dst, n, budget, X, agg, option=None):
    """The stack, a filter of it, the stack made without allocating, and the number of joining launches of the first."""
    if option:
        gp.gp_set_option(*option)
    try:
        with gp.gp_plan_blocks(src, dst, n, budget, gp.GP_ADD_SELF_LOOPS) as plan:
            gp.gp_profile_enable(True)
            out = gp.propagate_tensors(plan, X, agg, 2)
            joins, _ = gp.gp_profile_read("gp_fixup_rows")
            gp.gp_profile_enable(False)
            filt = torch.empty_like(X)
            stream = torch.cuda.current_stream().cuda_stream
            gp.gp_propagate_combine(plan, X.data_ptr(), X.stride(0), X.shape[1], gp.GP_F32, agg, 2, [1.0, 0.5, 0.25], filt.data_ptr(),
                                    filt.stride(0), stream)
            again = torch.empty_like(out)
            gp.gp_propagate_noalloc(plan, X.data_ptr(), X.stride(0), X.shape[1], gp.GP_F32, agg, 2, again.data_ptr(), X.shape[1], stream)
            return out.cpu(), filt.cpu(), again.cpu(), joins, plan.num_partial_rows
    finally:
        if option:
            gp.gp_set_option(option[0], 0)


@pytest.mark.parametrize("budget", [1, 7, 64, 500, 30_000])
@pytest.mark.parametrize("agg", [gp.GP_AGG_SYM, gp.GP_AGG_SUM])
def test_blocks_change_no_bit_where_rows_fit_a_segment(budget, agg):
    rng = np.random.default_rng(5)
    n = 1500 if budget < 500 else 20_000
    dst = np.repeat(rng.permutation(n)[:n // 2], rng.integers(0, 64, n // 2)).astype(np.int32)  # with its loop: 64 at most
    src = rng.integers(0, n, dst.size).astype(np.int32)
    X = torch.randn(n, 37, generator=torch.Generator().manual_seed(1)).cuda()
    one = stack(src, dst, n, 1 << 30, X, agg, ("cache_schedule", 2))
    cut = stack(src, dst, n, budget, X, agg, ("cache_schedule", 2))
    assert cut[4] > 0 and cut[3] == 0 and one[4] == 0
    assert all(torch.equal(a, b) for a, b in zip(one[:3], cut[:3]))
    assert torch.equal(cut[0], cut[2])


def test_a_longer_row_keeps_partial_rows_for_all():
    rng = np.random.default_rng(6)
    n = 2000
    dst = np.concatenate([np.zeros(65), rng.integers(0, n, 9000)]).astype(np.int32)
    src = rng.integers(0, n, dst.size).astype(np.int32)
    src[:65] = np.arange(1, 66)
    X = torch.randn(n, 37, generator=torch.Generator().manual_seed(1)).cuda()
    one, cut = (stack(src, dst, n, b, X, gp.GP_AGG_SYM, ("cache_schedule", 2)) for b in (1 << 30, 500))
    assert one[3] == cut[3] == 2 and torch.equal(cut[0], cut[2])
    assert all(torch.allclose(a, b, rtol=0, atol=64 * 2.0 ** -23 * float(a.abs().max())) for a, b in zip(one[:2], cut[:2]))  # 64 and more terms, regrouped


@pytest.mark.parametrize("option", [("lds_pass", 1), ("cache_schedule", 1), ("hub_pass", 1)])
def test_schedules_with_lists_of_their_own_keep_the_plans_cut(option):
    rng = np.random.default_rng(7)
    n = 4000
    dst = (np.arange(n * 40) // 40).astype(np.int32)
    src = (dst // 400 * 400 + rng.integers(0, 400, dst.size)).astype(np.int32)
    X = torch.randn(n, 64, generator=torch.Generator().manual_seed(1)).cuda()
    one, cut = (stack(src, dst, n, b, X, gp.GP_AGG_SYM, option) for b in (1 << 30, 977))
    assert cut[4] > 0
    assert all(torch.allclose(a, b, rtol=0, atol=41 * 2.0 ** -23 * float(a.abs().max())) for a, b in zip(one[:3], cut[:3]))  # 41 terms, regrouped


@pytest.mark.parametrize("agg", [gp.GP_AGG_SYM, gp.GP_AGG_SUM])
def test_explicit_and_implicit_lists_of_whole_rows_give_the_same_bits(agg):
    rng = np.random.default_rng(8)
    n = 4000
    dst = (np.arange(n * 40) // 40).astype(np.int32)
    src = (dst // 400 * 400 + rng.integers(0, 400, dst.size)).astype(np.int32)
    stream = torch.cuda.current_stream().cuda_stream
    gp.gp_set_option("split_records", 2)
    try:
        stacks = {}
        for schedule in (1, 2):  # explicit, implicit
            gp.gp_set_option("cache_schedule", schedule)
            with gp.gp_plan_blocks(src, dst, n, 977, gp.GP_ADD_SELF_LOOPS) as plan:
                assert plan.num_partial_rows > 0 and (plan.work_lists(64, gp.GP_F32, 4)[0] > 0) == (schedule == 1)
                for d in (64, 96):
                    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).cuda()
                    out, first = torch.empty(3, n, d, device="cuda"), torch.empty(3, n, d, device="cuda")
                    if d != 64:  # before a call has made explicit lists for this width: implicit ones
                        gp.gp_propagate_noalloc(plan, X.data_ptr(), d, d, gp.GP_F32, agg, 2, first.data_ptr(), d, stream)
                    gp.gp_profile_enable(True)
                    gp.gp_propagate(plan, X.data_ptr(), d, d, gp.GP_F32, agg, 2, out.data_ptr(), d, stream)
                    joins, _ = gp.gp_profile_read("gp_fixup_rows")
                    gp.gp_profile_enable(False)
                    assert joins == 0
                    assert d == 64 or torch.equal(first, out)
                    stacks[schedule, d] = out.cpu()
        assert torch.equal(stacks[1, 64], stacks[2, 64]) and torch.equal(stacks[1, 96], stacks[2, 96])
    finally:
        gp.gp_set_option("split_records", 0)
        gp.gp_set_option("cache_schedule", 0)
