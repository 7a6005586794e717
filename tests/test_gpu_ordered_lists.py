"""Implicit lists on ids in walking order, an XCD taking runs of 32 records: sizes around a run and around the runs
that the XCDs share, against the fp64 oracle at 1e-5 * (A^^k |X|); and calls that may not build the ordered list."""
import re

import numpy as np
import pytest

import gp_synth
import oracle
import paper_2207_12000_amd as gp

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _defaults(gpu_or_skip):
    yield
    for name in ("column_slices", "segment_edges", "cache_schedule", "hub_pass", "lds_pass", "split_records", "list_bytes"):
        gp.gp_set_option(name, 0)


def graph(n, m, seed):
    rng = np.random.default_rng(seed)
    return rng.integers(0, n, m).astype(np.int32), (rng.integers(0, n, m) ** 2 // max(1, n)).astype(np.int32)


def hops(plan, x, agg, K):
    import torch
    out = gp.propagate_tensors(plan, x, agg, K)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 257, 1025, 4099])   # rows = records where no row is cut
@pytest.mark.parametrize("slices", [1, 4, 8])
@pytest.mark.parametrize("agg", [gp.GP_AGG_SYM, gp.GP_AGG_MEAN])
def test_runs_of_records_match_the_oracle(n, slices, agg):
    import torch
    gp.gp_set_option("column_slices", slices)
    gp.gp_set_option("cache_schedule", 2)          # no clusters: implicit lists
    gp.gp_set_option("segment_edges", 16)          # hubs are cut: more records than rows
    src, dst = graph(n, 6 * n, n)
    d, K, budget = 40, 2, max(64, 3 * n)
    X = gp_synth.features(n, d, "normal", gp_synth.rng_for(7, n))
    op = oracle.plan_blocks(src, dst, n, budget, gp.GP_SYMMETRISE)
    with gp.gp_plan_blocks(src, dst, n, budget, gp.GP_SYMMETRISE) as plan:
        got = hops(plan, torch.from_numpy(X).cuda(), agg, K).cpu().numpy().astype(np.float64)
    Xw = X.astype(np.float64)
    want, bound = oracle.propagate(op, Xw, agg, K), oracle.bound_stack(op, Xw, agg, K)
    for k in range(K + 1):
        assert np.all(np.abs(got[k] - want[k]) <= 1e-5 * bound[k] + 1e-30), f"hop {k}"


def test_captured_calls_that_find_no_ordered_list():
    """A plan whose calls so far took the LDS pass has no ordered list; a captured call of another width may not make
    one and runs on the plan's own order, with the same bits."""
    import torch
    w = gp_synth.make_workload(2, scale=0.2, d=36)
    gp.gp_set_option("hub_pass", 1)
    n, K, budget = w.n, 2, max(20_000, w.m // 3)
    op = oracle.plan_blocks(w.src, w.dst, n, budget, w.flags)
    with gp.gp_plan_blocks(w.src, w.dst, n, budget, w.flags) as plan:
        first = kernels(lambda: hops(plan, torch.from_numpy(w.X).cuda(), gp.GP_AGG_SYM, K))
        assert sum("gp_hop_cluster_lds" in k for k in first) == K and not any("gp_order_columns" in k for k in first)
        x = torch.from_numpy(np.ascontiguousarray(w.X[:, :3])).cuda()
        out = torch.zeros((K + 1, n, 3), device="cuda:0")
        g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=side):
            gp.gp_propagate(plan, x.data_ptr(), 3, 3, gp.GP_F32, gp.GP_AGG_SYM, K, out.data_ptr(), 3,
                            torch.cuda.current_stream().cuda_stream)
        for rep in range(3):
            X = gp_synth.features(n, 3, "normal", gp_synth.rng_for(5, rep))
            x.copy_(torch.from_numpy(X))
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            eager = {}
            made = kernels(lambda: eager.update(out=hops(plan, x, gp.GP_AGG_SYM, K)))
            assert any("gp_order_columns" in k for k in made) == (rep == 0)  # the captured call had made none
            assert torch.equal(out, eager["out"])
            got, Xw = out.cpu().numpy().astype(np.float64), X.astype(np.float64)
            want, bound = oracle.propagate(op, Xw, gp.GP_AGG_SYM, K), oracle.bound_stack(op, Xw, gp.GP_AGG_SYM, K)
            for k in range(K + 1):
                assert np.all(np.abs(got[k] - want[k]) <= 1e-5 * bound[k] + 1e-30), f"hop {k}"


@pytest.mark.parametrize("d", [7, 40, 128])
def test_rows_of_few_and_many_partial_rows(d):
    """Rows cut into 2 .. 18 segments: the fix-up's partial rows in flight (four and four more) and its remainders, and the
    filter sum, which takes the very rows of the stack: at most one rounding per term of sum_k |c_k| |A^^k X|."""
    import torch
    gp.gp_set_option("cache_schedule", 2)
    gp.gp_set_option("segment_edges", 8)
    n, K, coeff = 400, 3, [0.5, -0.25, 2.0, 0.125]
    lengths = [9, 16, 17, 24, 25, 32, 33, 40, 41, 64, 65, 72, 73, 129, 137, 140]
    rng = np.random.default_rng(d)
    src = np.repeat(np.arange(len(lengths)), lengths).astype(np.int32)
    dst = np.concatenate([rng.choice(np.arange(20, n), c, replace=False) for c in lengths]).astype(np.int32)
    X = gp_synth.features(n, d, "normal", gp_synth.rng_for(3, d))
    op = oracle.plan_blocks(src, dst, n, 1 << 20, gp.GP_SYMMETRISE)
    with gp.gp_plan_blocks(src, dst, n, 1 << 20, gp.GP_SYMMETRISE) as plan:
        x = torch.from_numpy(X).cuda()
        stack = hops(plan, x, gp.GP_AGG_SYM, K).cpu().numpy().astype(np.float64)
        out = torch.empty_like(x)
        gp.gp_propagate_combine(plan, x.data_ptr(), d, d, gp.GP_F32, gp.GP_AGG_SYM, K, coeff, out.data_ptr(), d,
                                torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    Xw = X.astype(np.float64)
    want, bound = oracle.propagate(op, Xw, gp.GP_AGG_SYM, K), oracle.bound_stack(op, Xw, gp.GP_AGG_SYM, K)
    for k in range(K + 1):
        assert np.all(np.abs(stack[k] - want[k]) <= 1e-5 * bound[k] + 1e-30), f"hop {k}"
    total = sum(abs(c) * np.abs(s) for c, s in zip(coeff, stack))
    exact = sum(c * s for c, s in zip(coeff, stack))
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - exact) <= (K + 1) * 2.0 ** -24 * 1.01 * total + 1e-30)


@pytest.mark.parametrize("dtype,d,pad", [(gp.GP_F32, 64, 0), (gp.GP_F32, 47, 2), (gp.GP_F32, 1100, 1), (gp.GP_BF16, 72, 0), (gp.GP_BF16, 601, 1),
                                         (gp.GP_BF16, 600, 1)])
def test_first_hop_writes_the_filters_two_terms(dtype, d, pad):
    """c0 X + c1 A^ X in one hop, X's rows aligned less well than the output's (the fix-up then takes X's vectors and
    column passes): fp32 sums to 1e-5 of the magnitudes, and one rounding of the result for bf16 storage."""
    import torch
    gp.gp_set_option("cache_schedule", 2)
    gp.gp_set_option("segment_edges", 8)
    n, c0, c1 = 300, 0.75, -1.5
    src, dst = graph(n, 4000, d)
    X = torch.randn(n, d + pad, generator=torch.Generator().manual_seed(d)).to(torch.float32 if dtype == gp.GP_F32 else torch.bfloat16)
    x = X.cuda()
    out = torch.full((n, d), float("nan"), dtype=x.dtype, device="cuda")
    Xw = X[:, :d].double().numpy()
    op = oracle.plan_blocks(src, dst, n, 900, gp.GP_SYMMETRISE)
    with gp.gp_plan_blocks(src, dst, n, 900, gp.GP_SYMMETRISE) as plan:
        assert plan.num_partial_rows > 0
        gp.gp_propagate_combine(plan, x.data_ptr(), d + pad, d, dtype, gp.GP_AGG_SYM, 1, [c0, c1], out.data_ptr(), d,
                                torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    hop = oracle.propagate(op, Xw, gp.GP_AGG_SYM, 1)[1]
    want = c0 * Xw + c1 * hop
    err = np.abs(out.double().cpu().numpy() - want)
    sums = 1e-5 * (c0 * np.abs(Xw) + abs(c1) * oracle.bound_stack(op, Xw, gp.GP_AGG_SYM, 1)[1])
    assert np.all(err <= sums + (2.0 ** -8 * np.abs(want) + sums * 2.0 ** -8 if dtype == gp.GP_BF16 else 0.0) + 1e-30)


def noalloc(plan, x, agg, K):
    import torch
    n, d = x.shape
    out = torch.empty((K + 1, n, d), device="cuda:0")
    gp.gp_propagate_noalloc(plan, x.data_ptr(), d, d, gp.GP_F32, agg, K, out.data_ptr(), d, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return out


def kernels(call):
    """The names of the kernels that a call launches, in order."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
    return [e.name for e in p.events() if "gp::" in e.name]


def weights_read(names):
    """How the hop launches among them get their weights (the kernel's last parameter): 1 = from the n-vector, by column
    id, 2 = one per non-zero."""
    return [int(m.group(1)) for m in (re.search(r"gp_hop_segments<.*?, (\d)>", x) for x in names) if m]


@pytest.mark.parametrize("earlier", ["hubs in LDS", "split records", "no hops", "sum's list after sym", "mean's lists after sym"])
def test_calls_that_may_not_allocate_have_weights_per_nonzero(earlier):
    """After any allocating call of the sym operator, whatever its own hops ran on, a call that may not allocate finds
    weights for the list that it walks."""
    import torch
    K, communities = 2, earlier in ("split records", "mean's lists after sym")
    w = gp_synth.make_workload(4, scale=0.01, d=52) if communities else gp_synth.make_workload(2, scale=0.2, d=36)
    gp.gp_set_option("hub_pass", 1)
    if communities:
        gp.gp_set_option("lds_pass", 2)
        gp.gp_set_option("cache_schedule", 1)
        gp.gp_set_option("split_records", 1 if earlier == "split records" else 2)
    op = oracle.plan_blocks(w.src, w.dst, w.n, w.m, w.flags)
    X = np.ascontiguousarray(w.X[:, :52 if communities else 3])
    x = torch.from_numpy(X).cuda()
    with gp.gp_plan_blocks(w.src, w.dst, w.n, w.m, w.flags) as plan:
        wide = torch.randn(w.n, 1100 if communities else 36, device="cuda")
        if earlier == "no hops":
            hops(plan, wide, gp.GP_AGG_SYM, 0)
        elif earlier == "split records":
            assert len(weights_read(kernels(lambda: hops(plan, x, gp.GP_AGG_SYM, K)))) == 2 * K   # cold records, hot records
        elif earlier == "mean's lists after sym":
            hops(plan, wide, gp.GP_AGG_SYM, 1)       # several column passes: implicit lists
            hops(plan, x, gp.GP_AGG_MEAN, 1)         # explicit lists
        else:
            assert sum("gp_hop_cluster_lds" in k for k in kernels(lambda: hops(plan, wide, gp.GP_AGG_SYM, K))) == K
            if earlier == "sum's list after sym":
                assert any("gp_order_columns" in k for k in kernels(lambda: hops(plan, x, gp.GP_AGG_SUM, 1)))
        assert weights_read(kernels(lambda: noalloc(plan, x, gp.GP_AGG_SYM, K))) == [2] * K
        got = noalloc(plan, x, gp.GP_AGG_SYM, K).cpu().numpy().astype(np.float64)
    Xw = X.astype(np.float64)
    want, bound = oracle.propagate(op, Xw, gp.GP_AGG_SYM, K), oracle.bound_stack(op, Xw, gp.GP_AGG_SYM, K)
    for k in range(K + 1):
        assert np.all(np.abs(got[k] - want[k]) <= 1e-5 * bound[k] + 1e-30), f"hop {k}"


@pytest.mark.parametrize("agg", [gp.GP_AGG_SYM, gp.GP_AGG_MEAN])
@pytest.mark.parametrize("room", ["none", "weights"])
def test_calls_without_room_run_on_the_plans_order_and_the_next_call_asks_again(agg, room):
    """Device memory is short while the first calls run: they do without the copy in walking order (and without
    weights per non-zero), with the same bits; the copy is made by the first call that finds room, and only by it."""
    import torch
    K = 3
    w = gp_synth.make_workload(2, scale=0.2, d=40)
    gp.gp_set_option("cache_schedule", 2)
    x = torch.from_numpy(w.X).cuda()
    op = oracle.plan_blocks(w.src, w.dst, w.n, w.m, w.flags)
    sym = agg == gp.GP_AGG_SYM
    with gp.gp_plan_blocks(w.src, w.dst, w.n, w.m, w.flags) as plan:
        gp.gp_set_option("list_bytes", 1 if room == "none" else 4 * plan.nnz)
        out = {}

        def call(name):
            names = kernels(lambda: out.update({name: hops(plan, x, agg, K)}))
            return [sum(part in k for k in names) for part in ("gp_order_columns", "gp_fill_edge_weights")], weights_read(names)

        for i in range(2):
            made, read = call(f"short{i}")
            assert made == [0, int(sym and room == "weights" and i == 0)]
            assert read == [(1 if room == "none" else 2) if sym else 0] * K
        gp.gp_set_option("list_bytes", 0)
        assert call("room") == ([1, int(sym)], [2 if sym else 0] * K)
        assert call("again") == ([0, 0], [2 if sym else 0] * K)
    for name in ("short1", "room", "again"):
        assert torch.equal(out[name], out["short0"]), name
    got, Xw = out["short0"].cpu().numpy().astype(np.float64), w.X.astype(np.float64)
    want, bound = oracle.propagate(op, Xw, agg, K), oracle.bound_stack(op, Xw, agg, K)
    for k in range(K + 1):
        assert np.all(np.abs(got[k] - want[k]) <= 1e-5 * bound[k] + 1e-30), f"hop {k}"


@pytest.mark.parametrize("dtype,d,K", [(gp.GP_F32, 52, 1), (gp.GP_F32, 52, 3), (gp.GP_F32, 7, 1), (gp.GP_BF16, 72, 1)])
def test_first_hop_on_explicit_lists_writes_the_filters_two_terms(dtype, d, K):
    """The same sums from the per-XCD lists of a community graph: fp32 to 1e-5 of the magnitudes, and one rounding of
    the result for bf16 storage."""
    import torch
    gp.gp_set_option("cache_schedule", 1)
    gp.gp_set_option("lds_pass", 2)
    gp.gp_set_option("segment_edges", 16)
    w = gp_synth.make_workload(4, scale=0.01, d=d)
    coeff = [0.75, -1.5, 0.5, 0.25][:K + 1]
    X = torch.from_numpy(w.X).to(torch.float32 if dtype == gp.GP_F32 else torch.bfloat16)
    x, out = X.cuda(), torch.full((w.n, d), float("nan"), dtype=X.dtype, device="cuda")
    Xw = X.double().numpy()
    op = oracle.plan_blocks(w.src, w.dst, w.n, w.m // 3, w.flags)
    with gp.gp_plan_blocks(w.src, w.dst, w.n, w.m // 3, w.flags) as plan:
        assert plan.num_partial_rows > 0

        def call():
            gp.gp_propagate_combine(plan, x.data_ptr(), d, d, dtype, gp.GP_AGG_SYM, K, coeff, out.data_ptr(), d,
                                    torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()

        names = kernels(call)
        assert len(weights_read(names)) == K and not any("gp_order_columns" in k or "gp_hop_cluster_lds" in k for k in names)
    want = sum(c * h for c, h in zip(coeff, oracle.propagate(op, Xw, gp.GP_AGG_SYM, K)))
    err = np.abs(out.double().cpu().numpy() - want)
    sums = 1e-5 * sum(abs(c) * b for c, b in zip(coeff, oracle.bound_stack(op, Xw, gp.GP_AGG_SYM, K)))
    assert np.all(err <= sums + (2.0 ** -8 * (np.abs(want) + sums) if dtype == gp.GP_BF16 else 0.0) + 1e-30)
