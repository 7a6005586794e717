"""Records of a plan whose blocks are walked by several threads (fewer blocks than threads): every block's records longest
first, and in list order among equals, as one thread makes them."""
import numpy as np
import pytest

import paper_2207_12000_amd as gp
from test_plan_parity import check_schedule


def expected_order(plan, L):
    """(start, length, row) of every record: the list cut at row starts, block starts and every L non-zeros after them."""
    rowptr, boff = plan.rowptr, plan.block_off
    starts = []
    for p in range(plan.num_blocks):
        lo, hi, last = boff[p], boff[p + 1], p == plan.num_blocks - 1
        cut = np.unique(np.concatenate([[lo], rowptr[:-1][(rowptr[:-1] >= lo) & (rowptr[:-1] < hi)]]))
        cut = cut[cut < hi]
        end = np.append(cut[1:], hi)
        pieces = np.concatenate([np.arange(a, z, L) for a, z in zip(cut, end)]) if cut.size else np.empty(0, np.int64)
        row = np.searchsorted(rowptr, pieces, side="right") - 1
        length = np.minimum(np.minimum(rowptr[row + 1], hi) - pieces, L)
        deg = np.diff(rowptr)
        empty = np.flatnonzero((deg == 0) & (((rowptr[:-1] >= lo) & (rowptr[:-1] < hi)) | (last & (rowptr[:-1] >= plan.nnz))))
        row, length = np.concatenate([row, empty]), np.concatenate([length, np.zeros(empty.size, np.int64)])
        pieces = np.concatenate([pieces, rowptr[empty]])
        order = np.lexsort((pieces, row, -length))
        starts.append(np.stack([pieces[order], length[order], row[order]]))
    return np.concatenate(starts, axis=1)


@pytest.mark.parametrize("blocks", [1, 2, 7])
@pytest.mark.parametrize("kind", ["skewed", "one row", "mostly empty"])
def test_records_of_parts_are_those_of_one_walk(kind, blocks):
    rng = np.random.default_rng(blocks)
    n, m = 140_000, 90_000  # (a thread is given 16,384 rows and more)
    src = rng.integers(0, n, m)
    dst = (n * rng.random(m) ** 4).astype(np.int64)  # rows of thousands and of none
    if kind == "one row":                             # a block is one part's, the other parts have nothing
        src, dst, n = np.arange(n), np.zeros(n, np.int64), n + 1
    if kind == "mostly empty":
        dst = dst % 11 + n - 11
        n += 40_000
    with gp.gp_plan_blocks(src.astype(np.int32), dst.astype(np.int32), n, -(-m // blocks), 0) as plan:
        L = plan.segment_edges
        check_schedule(plan, L)
        seg = plan.segments
        start = seg["start_lo"].astype(np.int64) | (seg["start_hi"].astype(np.int64) << 32)
        assert np.array_equal(np.stack([start, seg["len"], seg["row"]]).astype(np.int64), expected_order(plan, L))
