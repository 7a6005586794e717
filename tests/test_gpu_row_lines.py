"""Hops that read X and the slabs between from rows on 128-byte lines of their own, against hops that read them where they
lie (no room for the copies): the same sums in the same order, so the same bits."""
import numpy as np
import pytest
import torch

import paper_2207_12000_amd as gp

pytestmark = pytest.mark.gpu

BITS = {torch.float32: torch.int32, torch.bfloat16: torch.int16}


def graph(n, hub):
    """Mean degree 24; node 3 has `hub` neighbours, so that rows of partial sums are among those handed on."""
    rng = np.random.default_rng(n)
    src, dst = rng.integers(0, n, 12 * n), rng.integers(0, n, 12 * n)
    return np.concatenate([src, np.full(hub, 3)]).astype(np.int32), np.concatenate([dst, rng.permutation(n)[:hub]]).astype(np.int32)


def both(n, run):
    """run(plan) with and without room for copies; the plan of the second has none left by the first."""
    out = []
    for room in (0, 1):
        gp.gp_set_option("list_bytes", room)
        try:
            with gp.gp_plan_blocks(*graph(n, n // 10), n, 1 << 17, gp.GP_SYMMETRISE) as plan:
                out.append(run(plan).cpu())
        finally:
            gp.gp_set_option("list_bytes", 0)
    assert out[0].isfinite().all() and torch.equal(*(o.view(BITS[o.dtype]) for o in out))


# widths on either side of a line, off 16, 8 and 4 bytes; one wide enough for column slices, one of several vectors a lane
@pytest.mark.parametrize("n,d,dtype,agg,K", [(40_000, 33, "float32", gp.GP_AGG_SYM, 3), (40_000, 63, "float32", gp.GP_AGG_SUM, 2),
                                             (60_000, 66, "float32", gp.GP_AGG_MEAN, 1), (20_000, 150, "float32", gp.GP_AGG_SYM, 2),
                                             (20_000, 47, "bfloat16", gp.GP_AGG_MEAN, 3), (9_000, 301, "bfloat16", gp.GP_AGG_SYM, 2),
                                             (60_000, 126, "bfloat16", gp.GP_AGG_SUM, 2), (7_000, 599, "bfloat16", gp.GP_AGG_SUM, 1)])
@pytest.mark.parametrize("where", ["tensor", "in place", "padded"])
def test_hop_stack(n, d, dtype, agg, K, where):
    dtype = getattr(torch, dtype)
    ld = d + (d % 2 * 2 if where == "padded" else 0)  # an odd stride stays odd
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()

    def run(plan):
        stack = torch.zeros(K + 1, n, ld, dtype=dtype, device="cuda")
        src = X
        if where == "in place":
            stack[0, :, :d] = X
            src = stack
        code = gp.GP_F32 if dtype == torch.float32 else gp.GP_BF16
        for _ in range(2):  # a plan's first call, and one on what that left
            gp.gp_propagate(plan, src.data_ptr(), src.stride(-2), d, code, agg, K, stack.data_ptr(), ld,
                            torch.cuda.current_stream().cuda_stream)
        assert torch.equal(stack[0, :, :d], X) and not stack[:, :, d:].any()  # nothing is written past a row
        return stack

    both(n, run)


@pytest.mark.parametrize("n,d,dtype", [(40_000, 20, "float32"), (40_000, 63, "float32"), (20_000, 47, "bfloat16"), (60_000, 100, "bfloat16")])
def test_filter(n, d, dtype):
    dtype = getattr(torch, dtype)
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()

    def run(plan):
        out = torch.empty_like(X)
        gp.gp_propagate_combine(plan, X.data_ptr(), d, d, gp.GP_F32 if dtype == torch.float32 else gp.GP_BF16, gp.GP_AGG_SYM, 3,
                                [0.5, 0.25, 0.125, 0.125], out.data_ptr(), d, torch.cuda.current_stream().cuda_stream)
        return out

    both(n, run)


@pytest.mark.parametrize("n,d", [(1, 5), (3, 47), (37_123, 47), (1000, 4), (5, 1023)])
@pytest.mark.parametrize("ld_in,ld_out", [(0, 0), (3, 1), (1, 8)])
def test_slot_0_of_ragged_rows(n, d, ld_in, ld_out):
    X = torch.randn(n, d + ld_in, device="cuda")
    out = torch.zeros(n, d + ld_out, device="cuda")
    with gp.gp_plan_blocks(np.zeros(0, np.int32), np.zeros(0, np.int32), n, 10, gp.GP_ADD_SELF_LOOPS) as plan:
        gp.gp_propagate(plan, X.data_ptr(), d + ld_in, d, gp.GP_F32, gp.GP_AGG_SUM, 0, out.data_ptr(), d + ld_out,
                        torch.cuda.current_stream().cuda_stream)
    assert torch.equal(out[:, :d], X[:, :d]) and not out[:, d:].any()
