"""Row clusters against label propagation written out plainly: every row takes the most frequent label of its sources,
ties to the smallest, all rows at once, until fewer than one row in 2000 changes or ten times."""
import numpy as np
import pytest

import oracle
import paper_2207_12000_amd as gp


def plain_clusters(rowptr, col, n):
    lab = np.arange(n)
    for _ in range(10):
        nxt = lab.copy()
        for i in range(n):
            if rowptr[i + 1] > rowptr[i]:
                l, c = np.unique(lab[col[rowptr[i]:rowptr[i + 1]]], return_counts=True)
                nxt[i] = l[np.argmax(c)]        # the first of the largest counts: the smallest label
        changed = int((nxt != lab).sum())
        lab = nxt
        if changed * 2000 < n:
            break
    return np.unique(lab, return_inverse=True)[1]


@pytest.mark.parametrize("kind", ["sparse", "directed", "communities", "pairs", "hub"])
def test_labels_are_those_of_plain_propagation(kind):
    rng = np.random.default_rng(11)
    n, flags = 700, gp.GP_SYMMETRISE
    if kind == "sparse":                      # empty rows, rows of one and two sources, ties
        src, dst = rng.integers(0, n, 500), rng.integers(0, n, 500)
    elif kind == "directed":
        src, dst, flags = rng.integers(0, n, 3000), rng.integers(0, n, 3000), 0
    elif kind == "communities":               # majorities of exactly half, and just over it
        src = rng.integers(0, n, 6000)
        dst = np.where(rng.random(6000) < 0.6, src // 70 * 70 + rng.integers(0, 70, 6000), rng.integers(0, n, 6000))
    elif kind == "pairs":
        src, dst = np.arange(0, n, 2), np.arange(1, n, 2)
    else:
        src, dst = np.zeros(n - 1, dtype=np.int64), np.arange(1, n)
    op = oracle.plan_blocks(src.astype(np.int32), dst.astype(np.int32), n, 1 << 20, flags)
    with gp.gp_plan_blocks(src.astype(np.int32), dst.astype(np.int32), n, 1 << 20, flags) as plan:
        label = plan.row_clusters()[0]
    assert np.array_equal(label, plain_clusters(op.rowptr, op.col, n))
