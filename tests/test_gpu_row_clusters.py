"""Row clusters made on the GPU (the first call on a plan that is there) against those the host makes: labels and figures
equal, over row lengths on either side of what a lane, a wavefront's table and a workgroup's table take."""
import numpy as np
import pytest

import gp_synth
import paper_2207_12000_amd as gp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu_or_skip):
    yield


def star_rows(lengths, n, rng):
    """One row of each length, from distinct sources; directed, so no other row is touched."""
    src = np.concatenate([rng.permutation(n)[:l] for l in lengths])
    return src, np.repeat(np.arange(len(lengths)), lengths)


def graph(kind):
    rng = np.random.default_rng(19)
    if kind == "lengths":                     # short, mid and big rows at their edges; many empty ones
        n = 20_000
        src, dst = star_rows([1, 2, 63, 64, 65, 127, 511, 512, 513, 1024, 8191, 8192, 8193, 16_385, 19_000], n, rng)
        more = rng.integers(0, n, (2, 3000))  # some rows whose labels move on
        return n, np.concatenate([src, more[0]]), np.concatenate([dst, more[1]]), 0
    if kind == "table":                       # a workgroup's table, filled to three quarters, and past it
        n = 20_000
        src, dst = star_rows([12_287, 12_288, 12_289, 16_383, 16_384], n, rng)
        more = rng.integers(0, n, (2, 3000))
        return n, np.concatenate([src, more[0]]), np.concatenate([dst, more[1]]), 0
    if kind == "huge":                        # rows that count in memory, more than go side by side; labels that do and do not repeat
        n, lengths = 700_001, [700_001, 300_000] + [13_000] * 300
        src, dst = star_rows(lengths, n, rng)
        more = rng.integers(0, n, (2, 2 * n))
        return n, np.concatenate([src, more[0]]), np.concatenate([dst, more[1]]), 0
    if kind == "ties":                        # pairs, squares: every label as often as the next
        i = np.arange(0, 4000, 4)
        return 4001, np.concatenate([i, i + 1, i + 2, i + 3]), np.concatenate([i + 1, i + 2, i + 3, i]), gp.GP_SYMMETRISE
    if kind == "communities":                 # rows of some 120 sources, two thirds inside
        n, m = 6_000, 360_000
        src = rng.integers(0, n, m)
        dst = np.where(rng.random(m) < 0.67, src // 300 * 300 + rng.integers(0, 300, m), rng.integers(0, n, m))
        return n, src, dst, gp.GP_SYMMETRISE
    if kind == "one":
        return 1, np.zeros(1, np.int64), np.zeros(1, np.int64), gp.GP_ADD_SELF_LOOPS
    if kind == "power law":                   # one giant cluster from the second round on
        w = gp_synth.make_workload(2, scale=0.3, with_features=False)
        return w.n, w.src, w.dst, w.flags
    n = int(rng.integers(20, 900))            # "sparse": rows of no, one and two sources
    return n, rng.integers(0, n, n // 2), rng.integers(0, n, n // 2), gp.GP_SYMMETRISE


@pytest.mark.parametrize("planner", [0, gp.GP_PLAN_ON_DEVICE])
@pytest.mark.parametrize("kind", ["lengths", "ties", "communities", "one", "power law", "sparse", "table", "huge"])
def test_the_gpus_clusters_are_the_hosts(kind, planner):
    import torch
    n, src, dst, flags = graph(kind)
    src, dst = src.astype(np.int32), dst.astype(np.int32)
    with gp.gp_plan_blocks(src, dst, n, 1 << 20, flags) as host, gp.gp_plan_blocks(src, dst, n, 1 << 20, flags | planner) as plan:
        want = host.row_clusters()            # no call has been made: the host's
        x = torch.ones((n, 4), device="cuda")
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
            gp.propagate_tensors(plan, x, gp.GP_AGG_SUM, 1)
            torch.cuda.synchronize()
        assert any("gp_weigh_clusters" in e.key for e in prof.key_averages()) == (host.nnz > 0)
        got = plan.row_clusters()
    assert np.array_equal(got[0], want[0]) and got[1:] == want[1:]


def test_a_row_of_many_sources_takes_time_in_proportion():
    """Labels that never repeat in a row, and that all change in every round: a cycle, and one row of `length` sources."""
    import torch

    def microseconds(length):
        n = 400_000
        rows = np.arange(n, dtype=np.int32)
        src = np.concatenate([np.roll(rows, 1), np.random.default_rng(3).permutation(n)[:length].astype(np.int32)])
        dst = np.concatenate([rows, np.zeros(length, np.int32)])
        with gp.gp_plan_blocks(src, dst, n, 1 << 20, 0) as plan:
            x = torch.ones((n, 4), device="cuda")
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
                gp.propagate_tensors(plan, x, gp.GP_AGG_SUM, 1)
                torch.cuda.synchronize()
        return sum(e.device_time_total for e in prof.key_averages() if "gp_label" in e.key)

    microseconds(10)
    assert microseconds(320_000) < 32 * microseconds(20_000)  # 16 times the sources
