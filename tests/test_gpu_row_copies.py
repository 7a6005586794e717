"""Which hops read X and the slabs between from copies with rows on 128-byte lines of their own, counted by the launches that
copy, and that their bits are those of hops that read rows where they lie; what the slabs take."""
import numpy as np
import pytest
import torch

import paper_2207_12000_amd as gp
from test_gpu_row_lines import BITS, graph

pytestmark = pytest.mark.gpu


def both(n, run, copied):
    """run(plan) with and without room for copies; the plan of the second has none left by the first.  copied: whether the
    first reads a copy of X (one launch more)."""
    out, copies = [], []
    for room in (0, 1):
        gp.gp_set_option("list_bytes", room)
        gp.gp_profile_enable(True)
        try:
            with gp.gp_plan_blocks(*graph(n, n // 10), n, 1 << 17, gp.GP_SYMMETRISE) as plan:
                out.append(run(plan).cpu())
                copies.append(gp.gp_profile_read("gp_copy_rows")[0])
        finally:
            gp.gp_profile_enable(False)
            gp.gp_set_option("list_bytes", 0)
    assert out[0].isfinite().all() and torch.equal(*(o.view(BITS[o.dtype]) for o in out))
    assert copies[0] - copies[1] == copied


def hop_stack(n, d, dtype, agg, K, where, copied, ld=None):
    dtype = getattr(torch, dtype)
    ld = ld or d + (d % 2 * 2 if where == "padded" else 0)  # an odd stride stays odd
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()

    def run(plan):
        stack = torch.zeros(K + 1, n, ld, dtype=dtype, device="cuda")
        src = X
        if where == "in place":
            stack[0, :, :d] = X
            src = stack
        code = gp.GP_F32 if dtype == torch.float32 else gp.GP_BF16
        for _ in range(2):  # a plan's first call, which makes no slabs (unless it gains a ms by them), and the next
            gp.gp_propagate(plan, src.data_ptr(), src.stride(-2), d, code, agg, K, stack.data_ptr(), ld,
                            torch.cuda.current_stream().cuda_stream)
        assert torch.equal(stack[0, :, :d], X) and not stack[:, :, d:].any()  # nothing is written past a row
        return stack

    both(n, run, copied)


# widths on either side of a line, off 16, 8 and 4 bytes; rows that several to a line hold; one wide enough for column
# slices, one of several vectors a lane; one hop and more
@pytest.mark.parametrize("n,d,dtype,agg,K", [(300_000, 15, "float32", gp.GP_AGG_SUM, 3), (40_000, 47, "float32", gp.GP_AGG_SYM, 3),
                                             (40_000, 63, "float32", gp.GP_AGG_SUM, 2), (70_000, 58, "float32", gp.GP_AGG_MEAN, 1),
                                             (40_000, 159, "float32", gp.GP_AGG_SYM, 2), (280_000, 15, "bfloat16", gp.GP_AGG_SUM, 2),
                                             (20_000, 47, "bfloat16", gp.GP_AGG_MEAN, 3), (9_000, 301, "bfloat16", gp.GP_AGG_SYM, 2),
                                             (70_000, 126, "bfloat16", gp.GP_AGG_SUM, 2), (7_000, 599, "bfloat16", gp.GP_AGG_SUM, 1)])
@pytest.mark.parametrize("where", ["tensor", "in place", "padded"])
def test_hop_stack(n, d, dtype, agg, K, where):
    hop_stack(n, d, dtype, agg, K, where, True)


# rows of a few elements, which a copy would only spread out; slabs that an L2 holds most of until they are wider; rows that
# touch no fewer lines; small matrices
@pytest.mark.parametrize("n,d,dtype", [(600_000, 1, "bfloat16"), (400_000, 3, "bfloat16"), (360_000, 3, "float32"), (250_000, 5, "float32"),
                                       (60_000, 9, "bfloat16"), (131_000, 10, "float32"), (160_000, 7, "float32"), (1_200_000, 7, "bfloat16"), (40_000, 33, "float32"), (20_000, 47, "float32"), (60_000, 100, "bfloat16")])
def test_rows_that_are_read_where_they_lie(n, d, dtype):
    hop_stack(n, d, dtype, gp.GP_AGG_SUM, 2, "tensor", False)


# rows that save lines by leaving slots that are wider than they are: from four elements on, in the shortest vectors too
@pytest.mark.parametrize("n,d,dtype,ld,K,copied", [(600_000, 2, "float32", 5, 2, False), (600_000, 3, "float32", 5, 2, False),
                                                   (600_000, 4, "float32", 5, 2, True), (2_800_000, 3, "bfloat16", 10, 2, False),
                                                   (700_000, 7, "bfloat16", 7, 6, True)])
def test_narrow_rows_in_wider_slots(n, d, dtype, ld, K, copied):
    hop_stack(n, d, dtype, gp.GP_AGG_SUM, K, "tensor", copied, ld)


@pytest.mark.parametrize("n,d,dtype,copied", [(80_000, 20, "float32", False), (40_000, 63, "float32", True), (20_000, 47, "bfloat16", True),
                                              (60_000, 100, "bfloat16", False), (10_000, 20, "float32", False)])
def test_filter(n, d, dtype, copied):
    """Slabs as wide as there is room for, and X from a copy, or as its rows lie on lines already."""
    dtype = getattr(torch, dtype)
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()
    ld = -(-d * X.element_size() // 128) * 128 // X.element_size()
    on_lines = torch.zeros(n, ld, dtype=dtype, device="cuda")
    on_lines[:, :d] = X

    def run(plan):
        out = torch.empty(2, n, d, dtype=dtype, device="cuda")
        for x, o, copies in ((X, out[0], copied), (on_lines, out[1], False)):
            before = gp.gp_profile_read("gp_copy_rows")[0]
            gp.gp_propagate_combine(plan, x.data_ptr(), x.stride(0), d, gp.GP_F32 if dtype == torch.float32 else gp.GP_BF16, gp.GP_AGG_SYM, 3,
                                    [0.5, 0.25, 0.125, 0.125], o.data_ptr(), d, torch.cuda.current_stream().cuda_stream)
            assert gp.gp_profile_read("gp_copy_rows")[0] - before == copies
        assert torch.equal(*(o.view(BITS[o.dtype]) for o in out))
        return out

    both(n, run, False)  # (the slabs that a filter needs take the copy in any case)


def test_slabs_of_a_plan_used_at_growing_widths_stay_bounded():
    n, widths = 100_000, range(41, 127, 5)
    src = np.random.default_rng(1).integers(0, n, 32 * n).astype(np.int32)
    dst = np.repeat(np.arange(n, dtype=np.int32), 32)  # rows of 32: no partial rows, whose buffer grows too
    X, out = torch.zeros(n, 128, device="cuda"), torch.empty(4 * n * 128, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    gp.gp_set_option("cache_schedule", 2)
    gp.gp_profile_enable(True)
    try:
        with gp.gp_plan_blocks(src, dst, n, 1 << 23, 0) as plan:
            def call(d, K):
                """Bytes of device memory that the call took."""
                free = torch.cuda.mem_get_info()[0]
                gp.gp_propagate(plan, X.data_ptr(), d, d, gp.GP_F32, gp.GP_AGG_SUM, K, out.data_ptr(), d, stream)
                torch.cuda.synchronize()
                return free - torch.cuda.mem_get_info()[0]

            assert plan.num_partial_rows == 0
            call(32, 3)  # plan and lists; rows on lines as they are
            assert gp.gp_profile_read("gp_copy_rows")[0] == 1
            slab = n * 256
            assert 0.9 * slab < call(63, 1) < 1.5 * slab  # one slab for one hop (memory comes in pages of 2 MiB)
            assert 0.9 * slab < call(63, 3) < 1.5 * slab  # the other
            copies = gp.gp_profile_read("gp_copy_rows")[0]
            taken = sum(call(d, 3) for d in widths)
            assert gp.gp_profile_read("gp_copy_rows")[0] - copies > len(widths) + 8
            assert taken <= 2 * 2 * n * 512  # at most twice the widest row's two slabs (2.6 times, each as large as its call needs)
    finally:
        gp.gp_profile_enable(False)
        gp.gp_set_option("cache_schedule", 0)
