"""GPU parity of gp_lc_forward (Appendix A, LC version of GPRGNN) against the fp64
oracle, element by element.

Tolerance.  Every layer is an fp32 dot product of length in_l accumulated in some
order, so its error is at most gamma_{in_l} = in_l * u (u = 2^-24, first order)
times sum |a||w|; later layers pass that on through |W| (ReLU is 1-Lipschitz) and
add their own.  With the scaling by gamma_k and the K+1-term sum the total is at most
(sum_l in_l + T + K + 2) * u * bound, bound = sum_k |gamma_k| |X_k| |W_1| ... |W_T|;
the tests allow 1.5 times that for the higher-order terms.  (Where an fp32 product is taken as six bf16 products, at
most u of each term is left out and the two partial sums are added once more: 2 u more for such a layer, whose
sums have more than 16 terms, so that half of in_l covers it.)
"""
import numpy as np
import pytest

import gp_synth
import oracle
from oracle import lc
import paper_2207_12000_amd as gp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu_or_skip):
    yield


def tolerance(d, widths, K):
    return 1.5 * (d + sum(widths[:-1]) + len(widths) + K + 2) * 2.0 ** -24


def make_weights(rng, d, widths):
    dims = [d] + list(widths)
    return [(rng.normal(size=(dims[t], dims[t + 1])) / np.sqrt(dims[t])).astype(np.float32) for t in range(len(widths))]


def run(stack_np, ids, gamma, Ws, bf16=False, ldo_pad=0):
    """stack_np: float32 (or uint16 bf16 bits) array (K+1, n, d).  Returns the GPU result."""
    import torch
    if bf16:
        stack = torch.from_numpy(stack_np.view(np.int16)).view(torch.bfloat16).cuda()
    else:
        stack = torch.from_numpy(stack_np).cuda()
    batch = None if ids is None else torch.from_numpy(np.asarray(ids, dtype=np.int32)).cuda()
    Wd = [torch.from_numpy(W).cuda() for W in Ws]
    B = stack.shape[1] if ids is None else len(ids)
    C = Ws[-1].shape[1]
    buf = torch.full((B, C + ldo_pad), -7.0, device="cuda")
    out = gp.lc_forward_tensors(stack, batch, gamma, Wd, out=buf[:, :C])
    torch.cuda.synchronize()
    if ldo_pad:
        assert torch.all(buf[:, C:] == -7.0)              # nothing written past the row
    return out.cpu().numpy().astype(np.float64)


def check(stack_np, ids, gamma, Ws, bf16=False, **kw):
    got = run(stack_np, ids, gamma, Ws, bf16=bf16, **kw)
    wide = gp_synth.bf16_bits_to_f32(stack_np) if bf16 else stack_np
    rows = np.arange(wide.shape[1]) if ids is None else ids
    want = lc.lc_forward(wide, rows, gamma, Ws)
    bound = lc.lc_bound(wide, rows, gamma, Ws)
    tol = tolerance(wide.shape[2], [W.shape[1] for W in Ws], len(gamma) - 1)
    err = np.abs(got - want)
    assert got.shape == want.shape
    assert np.all(err <= tol * bound + 1e-30), f"worst ratio {np.max(err / (bound + 1e-300)):.3g} (allowed {tol:.3g})"
    return got


CASES = [
    # d, widths, K, n, B
    (128, [256, 256, 256, 40], 3, 3000, 209),     # the paper's shape: hidden 256, four layers, 40 classes
    (100, [256, 41], 3, 2000, 4096),              # d not a multiple of 8, duplicates in the batch
    (602, [256, 256, 41], 2, 700, 130),           # three feature panels
    (7, [5], 2, 50, 33),                          # one layer: a linear model on the filtered features
    (64, [192, 172], 5, 500, 64),                 # layers that end inside a wave's columns
    (33, [37, 130, 3], 1, 300, 1),                # odd widths, a single row
    (16, [64] * 7 + [10], 0, 200, 77),            # K = 0, eight layers
    (256, [128, 128], 4, 400, 191),
]


@pytest.mark.parametrize("d,widths,K,n,B", CASES)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("tile_rows", [32, 64])
def test_parity(d, widths, K, n, B, bf16, tile_rows):
    """Both work-item heights that can be asked for (64 stands for 48, the tallest there is, where fp32 products are
    taken as six bf16 products); the library's own choice, 16 rows among them, is in the tests at the end."""
    rng = np.random.default_rng(1000 + d + B)
    stack = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    if bf16:
        stack = gp_synth.f32_to_bf16_bits(stack)
    ids = rng.integers(0, n, B)
    gamma = rng.normal(size=K + 1)
    gp.gp_set_option("lc_tile_rows", tile_rows)
    try:
        check(stack, ids, gamma, make_weights(rng, d, widths), bf16=bf16, ldo_pad=3 if B < 100 else 0)
    finally:
        gp.gp_set_option("lc_tile_rows", 0)


def test_all_rows_and_determinism():
    rng = np.random.default_rng(7)
    stack = rng.normal(size=(3, 1000, 48)).astype(np.float32)
    Ws = make_weights(rng, 48, [96, 12])
    a = check(stack, None, [0.5, 0.3, 0.2], Ws)
    b = run(stack, None, [0.5, 0.3, 0.2], Ws)
    assert np.array_equal(a, b)


def test_rows_outside_the_graph_give_zero_rows():
    rng = np.random.default_rng(8)
    stack = rng.normal(size=(2, 100, 20)).astype(np.float32)
    Ws = make_weights(rng, 20, [32, 6])
    ids = np.array([5, -1, 100, 99, 2 ** 31 - 1, 0], dtype=np.int64)
    got = run(stack, ids, [1.0, 1.0], Ws)
    assert np.all(got[[1, 2, 4]] == 0.0)
    want = lc.lc_forward(stack, ids[[0, 3, 5]], [1.0, 1.0], Ws)
    assert np.allclose(got[[0, 3, 5]], want, rtol=1e-4, atol=1e-5)


def test_unaligned_operands():
    """A stack whose rows are not 16-byte aligned (ld = d + 1, base off by one
    element) takes the element-wise gather."""
    import torch
    rng = np.random.default_rng(9)
    K, n, d, ld = 2, 150, 30, 31
    flat = torch.zeros((K + 1) * n * ld + 1, device="cuda")
    stack_np = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    view = flat[1:].view(K + 1, n, ld)
    view[:, :, :d] = torch.from_numpy(stack_np).cuda()
    Ws = make_weights(rng, d, [64, 8])
    Wd = [torch.from_numpy(W).cuda() for W in Ws]
    ids = rng.integers(0, n, 70)
    batch = torch.from_numpy(ids.astype(np.int32)).cuda()
    out = torch.empty((70, 8), device="cuda")
    gamma = [0.2, 0.5, 0.3]
    gp.gp_lc_forward(view.data_ptr(), ld, gp.GP_F32, n, d, K, batch.data_ptr(), 70, gamma,
                     [W.data_ptr() for W in Wd], [64, 8], out.data_ptr(), 8, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    want = lc.lc_forward(stack_np, ids, gamma, Ws)
    bound = lc.lc_bound(stack_np, ids, gamma, Ws)
    assert np.all(np.abs(out.cpu().numpy() - want) <= tolerance(d, [64, 8], K) * bound + 1e-30)


def test_large_batch_goes_through_in_pieces():
    """16 hops x 256 output columns: the per-hop results of 40,000 rows exceed the
    library's buffer, so the batch is processed in several pieces."""
    rng = np.random.default_rng(10)
    K, n, d = 15, 3000, 16
    stack = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    Ws = make_weights(rng, d, [256])
    ids = rng.integers(0, n, 40000)
    check(stack, ids, rng.normal(size=K + 1), Ws)


def test_on_the_propagated_stack_of_config_2():
    """The consumer on the real thing: config 2's hop stack as gp_propagate leaves it
    in HBM, one mini-batch of 4096 rows (the paper's batch size) and all rows, with
    the paper's model shape (hidden 256, four layers, 40 classes) and PPR-initialised
    gamma.  The oracle runs on the GPU's own stored stack."""
    import torch
    w = gp_synth.make_workload(2)
    rng = np.random.default_rng(2)
    Ws = make_weights(rng, w.d, [256, 256, 256, 40])
    gamma = oracle.ppr_coefficients(0.1, w.K)
    with gp.gp_plan_blocks(w.src, w.dst, w.n, w.block_budget_edges, w.flags) as lp:
        stack = gp.propagate_tensors(lp, torch.from_numpy(w.X).cuda(), w.agg, w.K)
    Wd = [torch.from_numpy(W).cuda() for W in Ws]
    stack_np = stack.cpu().numpy()
    tol = tolerance(w.d, [256, 256, 256, 40], w.K)
    for ids in (rng.permutation(w.n)[:4096], None):
        batch = None if ids is None else torch.from_numpy(ids.astype(np.int32)).cuda()
        out = gp.lc_forward_tensors(stack, batch, gamma, Wd)
        torch.cuda.synchronize()
        rows = np.arange(w.n) if ids is None else ids
        want = lc.lc_forward(stack_np, rows, gamma, Ws)
        bound = lc.lc_bound(stack_np, rows, gamma, Ws)
        err = np.abs(out.cpu().numpy() - want)
        assert np.all(err <= tol * bound + 1e-30), f"worst ratio {np.max(err / (bound + 1e-300)):.3g} (allowed {tol:.3g})"


def test_random_shapes():
    """Forty seeded random shapes: feature widths 1 .. 300 (one or two panels), one to
    four layers of widths 1 .. 256, 1 .. 5 hops, 1 .. 300 rows, work-item heights asked for and
    chosen, batch lists with out-of-range entries mixed in."""
    rng = np.random.default_rng(4242)
    try:
        for case in range(40):
            d = int(rng.integers(1, 301))
            T = int(rng.integers(1, 5))
            widths = [int(rng.integers(1, 257)) for _ in range(T)]
            K = int(rng.integers(0, 5))
            n = int(rng.integers(1, 400))
            B = int(rng.integers(1, 301))
            stack = rng.normal(size=(K + 1, n, d)).astype(np.float32)
            ids = rng.integers(0, n, B)
            gamma = rng.normal(size=K + 1)
            Ws = make_weights(rng, d, widths)
            gp.gp_set_option("lc_tile_rows", int(rng.choice([0, 32, 64])))
            print(f"case {case}: d {d} widths {widths} K {K} n {n} B {B}", flush=True)
            check(stack, ids, gamma, Ws)
    finally:
        gp.gp_set_option("lc_tile_rows", 0)


def test_replays_in_a_hip_graph():
    """After one eager call (which sizes the library's buffer) the call allocates
    nothing and can be captured; every replay must reproduce the eager bits."""
    import torch
    rng = np.random.default_rng(11)
    K, n, d = 3, 2000, 64
    stack = torch.from_numpy(rng.normal(size=(K + 1, n, d)).astype(np.float32)).cuda()
    Ws = [torch.from_numpy(W).cuda() for W in make_weights(rng, d, [128, 128, 16])]
    batch = torch.from_numpy(rng.integers(0, n, 500).astype(np.int32)).cuda()
    gamma = [0.4, 0.3, 0.2, 0.1]
    eager = gp.lc_forward_tensors(stack, batch, gamma, Ws).clone()
    torch.cuda.synchronize()
    out = torch.zeros_like(eager)
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):                           # the binding takes torch's current stream
        gp.lc_forward_tensors(stack, batch, gamma, Ws, out=out)
    for _ in range(3):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        gp.lc_forward_tensors(stack, batch, gamma, Ws)               # eager work between the replays
        torch.cuda.synchronize()


BRANCH_CASES = [
    # d, widths, K, depth, comb, B
    (128, [256, 256, 256], 3, [0, 1, 2, 3], gp.GP_COMB_CONCAT, 300),   # the paper's form: hop k runs k layers, concat pooling
    (128, [256, 256, 256], 3, [0, 1, 2, 3], gp.GP_COMB_MAX, 300),      # max pooling
    (64, [40, 40], 2, [1, 2, 2], gp.GP_COMB_SUM, 100),
    (30, [17, 33, 5], 4, [3, 0, 1, 2, 3], gp.GP_COMB_CONCAT, 77),      # widths 5, 17, 33, 5 side by side
    (20, [64], 5, [1, 0, 0, 0, 0, 1], gp.GP_COMB_MAX, 10),
    (48, [96, 12], 2, [0, 2, 0], gp.GP_COMB_SUM, 5000),                # one branch: written directly
]


@pytest.mark.parametrize("d,widths,K,depth,comb,B", BRANCH_CASES)
@pytest.mark.parametrize("bf16", [False, True])
def test_branches_parity(d, widths, K, depth, comb, B, bf16):
    import torch
    rng = np.random.default_rng(2000 + d + B)
    n = 1500
    stack_np = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    if bf16:
        stack_np = gp_synth.f32_to_bf16_bits(stack_np)
        stack = torch.from_numpy(stack_np.view(np.int16)).view(torch.bfloat16).cuda()
    else:
        stack = torch.from_numpy(stack_np).cuda()
    wide = gp_synth.bf16_bits_to_f32(stack_np) if bf16 else stack_np
    ids = rng.integers(0, n, B)
    gamma = rng.normal(size=K + 1) if comb == gp.GP_COMB_SUM else np.ones(K + 1)
    Ws = make_weights(rng, d, widths)
    out = gp.lc_forward_tensors(stack, torch.from_numpy(ids.astype(np.int32)).cuda(), gamma,
                                [torch.from_numpy(W).cuda() for W in Ws], depth=depth, comb=comb)
    torch.cuda.synchronize()
    want = lc.lc_forward_branches(wide, ids, gamma, Ws, depth, comb)
    bound = lc.lc_bound_branches(wide, ids, gamma, Ws, depth, comb)
    err = np.abs(out.cpu().numpy().astype(np.float64) - want)
    tol = tolerance(d, widths, K)
    assert out.shape == want.shape
    assert np.all(err <= tol * bound + 1e-30), f"worst ratio {np.max(err / (bound + 1e-300)):.3g} (allowed {tol:.3g})"


@pytest.mark.parametrize("B,C,pad", [(1, 1, 0), (5, 40, 0), (1000, 41, 3), (333, 172, 0), (64, 256, 5), (7, 1000, 0)])
def test_softmax_rows(B, C, pad):
    """fp32 arithmetic: the rounded difference h - max (|h - max| < 64 here) costs up to
    64 * 2^-24 relative in exp, in the numerator and in every term of the denominator,
    the C-term sum C * 2^-24, exp itself and the division a few ulp."""
    import torch
    rng = np.random.default_rng(3000 + B + C)
    H = (rng.normal(size=(B, C)) * 6).astype(np.float32)
    buf = torch.full((B, C + pad), 9.0, device="cuda")
    buf[:, :C] = torch.from_numpy(H).cuda()
    gp.gp_lc_softmax(buf.data_ptr(), B, C, C + pad, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = buf[:, :C].cpu().numpy().astype(np.float64)
    want = lc.softmax_rows(H)
    assert np.all(np.abs(got - want) <= (C + 160) * 2.0 ** -24 * want + 1e-37)
    if pad:
        assert torch.all(buf[:, C:] == 9.0)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d,widths,B", [(31, [256, 40], 47), (300, [130, 70], 49), (64, [65], 16), (32, [129, 256], 97)])
def test_infinities_and_nans(d, widths, B, bf16):
    """Sums that an infinity, a NaN or a number beyond the largest bf16 one takes part in are plain fp32
    arithmetic's: the same infinities and NaNs as the oracle, and the other elements within tolerance."""
    rng = np.random.default_rng(77 + d)
    n, K = 120, 1
    stack = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    stack[0, 3, 1] = np.inf
    stack[1, 5, 0] = -np.inf
    stack[0, 7, d - 1] = np.nan
    if bf16:
        stack = gp_synth.f32_to_bf16_bits(stack)
        stack[0, 7, d - 1] = 0x7FC0
    else:
        stack[0, 9, 2] = np.float32(3.4e38)  # rounds to infinity in bf16
    Ws = make_weights(rng, d, widths)
    Ws[0][2] *= np.float32(1e-3)
    ids = np.concatenate([[3, 5, 7, 9, 0], rng.integers(10, n, B - 5)])
    gamma = [0.5, 0.25]
    got = run(stack, ids, gamma, Ws, bf16=bf16)
    wide = gp_synth.bf16_bits_to_f32(stack) if bf16 else stack
    with np.errstate(all="ignore"):
        want = lc.lc_forward(wide, ids, gamma, Ws)
        bound = lc.lc_bound(wide, ids, gamma, Ws)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want)) and not np.all(np.isfinite(want))
    ok = np.isfinite(want)
    assert np.all(np.abs(got - want)[ok] <= tolerance(d, widths, K) * bound[ok] + 1e-30)


@pytest.mark.parametrize("d,widths,B,bf16", [(100, [256, 172, 41], 333, False), (270, [70, 130], 5000, True), (48, [40], 17, False),
                                             (128, [256, 256, 256, 40], 9000, False),
                                             (90, [131, 77, 40], 3000, False)])
def test_captured_call_that_writes_its_result_directly(d, widths, B, bf16):
    """A concatenating call under graph capture splits its weights where it uses them (no shared slot), or needs none
    split (the last model): every replay gives the eager call's bits, with other calls of the library in between."""
    import torch
    rng = np.random.default_rng(5 + d)
    n, K, T = 700, 2, len(widths)
    stack = torch.from_numpy(rng.normal(size=(K + 1, n, d)).astype(np.float32)).cuda()
    if bf16:
        stack = stack.bfloat16()
    Wd = [torch.from_numpy(W).cuda() for W in make_weights(rng, d, widths)]
    batch = torch.from_numpy(rng.integers(0, n, B).astype(np.int32)).cuda()
    depth, gamma = [T, 1, T], [1.0, 0.5, 0.25]

    def call(out=None):
        return gp.lc_forward_tensors(stack, batch, gamma, Wd, out=out, depth=depth, comb=gp.GP_COMB_CONCAT)

    eager = call()
    out = torch.empty_like(eager)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        call(out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out)
    for _ in range(3):
        out.fill_(-3.0)
        graph.replay()
        gp.lc_forward_tensors(stack, batch[:9], gamma, Wd)
        torch.cuda.synchronize()
        assert torch.equal(out, eager)


def test_calls_on_many_streams():
    """Direct calls on more streams than the library has slots for split weights, interleaved without waiting: each
    gives what it gives alone.  (A model and a batch large enough that the weights are split beforehand.)"""
    import torch
    rng = np.random.default_rng(21)
    n, d = 9000, 96
    stack = torch.from_numpy(rng.normal(size=(1, n, d)).astype(np.float32)).cuda()
    models = [[torch.from_numpy(W).cuda() for W in make_weights(rng, d, [256, 256, 256, 64])] for _ in range(5)]
    want = [gp.lc_forward_tensors(stack, None, [1.0], m) for m in models]
    outs = [torch.empty_like(want[0]) for _ in range(40)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(20)]
    for k in range(40):
        with torch.cuda.stream(streams[k % 20]):
            gp.lc_forward_tensors(stack, None, [1.0], models[k % 5], out=outs[k])
    torch.cuda.synchronize()
    for k in range(40):
        assert torch.equal(outs[k], want[k % 5]), k


def test_one_handle_that_is_a_stream_of_its_own_in_every_thread():
    """hipStreamPerThread (handle 2) names another stream in each thread: direct calls of two threads on it, with
    different weights and nothing that orders them, each give what they give alone."""
    import threading
    import torch
    per_thread = 2
    rng = np.random.default_rng(31)
    n, d = 30000, 96
    stack = torch.from_numpy(rng.normal(size=(1, n, d)).astype(np.float32)).cuda()
    models = [[torch.from_numpy(W).cuda() for W in make_weights(rng, d, [256, 200, 64])] for _ in range(2)]
    want = [gp.lc_forward_tensors(stack, None, [1.0], m) for m in models]
    outs = [[torch.empty_like(want[0]) for _ in range(12)] for _ in models]
    torch.cuda.synchronize()
    start, failures = threading.Barrier(2), []

    def work(k):
        try:
            torch.cuda.set_device(0)
            start.wait(30)
            for out in outs[k]:
                gp.lc_forward_tensors(stack, None, [1.0], models[k], out=out, stream=per_thread)
            torch.cuda.synchronize()   # before the thread ends and its stream with it
        except Exception as e:  # noqa: BLE001
            failures.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not failures, failures
    for k in range(2):
        for j, out in enumerate(outs[k]):
            assert torch.equal(out, want[k]), (k, j)


def test_direct_calls_beside_a_capture():
    """Direct calls allocate nothing: on streams the library has not seen, while another stream is captured in the mode
    that forbids allocations to everybody, they work and the capture survives them."""
    import torch
    rng = np.random.default_rng(41)
    n, d = 30000, 64
    stack = torch.from_numpy(rng.normal(size=(1, n, d)).astype(np.float32)).cuda()
    Ws = [torch.from_numpy(W).cuda() for W in make_weights(rng, d, [256, 200, 40])]
    want = gp.lc_forward_tensors(stack, None, [1.0], Ws)
    outs = [torch.empty_like(want) for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in outs]
    counter = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode="global"):
        counter.add_(1.0)
        for out, s in zip(outs, streams):
            gp.lc_forward_tensors(stack, None, [1.0], Ws, out=out, stream=s.cuda_stream)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.all(counter == k + 1.0)
    for out in outs:
        assert torch.equal(out, want)


@pytest.mark.parametrize("d,widths,K", [(5300, [256], 0), (5600, [256], 0), (5600, [250, 40], 1)])
def test_weights_that_fill_the_room_for_split_ones(d, widths, K):
    """The largest weights that are split beforehand, and larger ones, which are split where they are used."""
    rng = np.random.default_rng(51 + d)
    stack = rng.normal(size=(K + 1, 150, d)).astype(np.float32)
    check(stack, rng.integers(0, 150, 3000), rng.normal(size=K + 1), make_weights(rng, d, widths))


def test_captured_sum_after_a_call_with_fewer_features():
    """The library's buffer depends on rows and output columns alone: a summing call on more features and more
    layers than the eager calls before it can be captured, and its replays are right after eager calls on still more."""
    import torch
    rng = np.random.default_rng(61)
    n, K, C, B = 300, 1, 40, 2000
    batch = torch.from_numpy(rng.integers(0, n, B).astype(np.int32)).cuda()
    gamma = [0.75, 0.5]

    def model(d, widths):
        stack = torch.from_numpy(rng.normal(size=(K + 1, n, d)).astype(np.float32)).cuda()
        return stack, [torch.from_numpy(W).cuda() for W in make_weights(rng, d, widths)]

    small, wide, wider = model(32, [C]), model(3000, [256, 256, C]), model(5000, [256, C])
    out = torch.full((B, C), -1.0, device="cuda")
    gp.lc_forward_tensors(small[0], batch, gamma, small[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gp.lc_forward_tensors(wide[0], batch, gamma, wide[1], out=out)
    want = gp.lc_forward_tensors(wide[0], batch, gamma, wide[1])
    for _ in range(3):
        gp.lc_forward_tensors(wider[0], batch, gamma, wider[1])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        out.fill_(-1.0)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("x_exp,w_exps", [
    (-118, [100, 0]),      # features whose last bits lie below the normal range
    (-124, [110, 4]),
    (-90, [-20, 100]),     # the first layer's activations are as small
    (60, [-122, 30]),      # weights as small
    (0, [-118, 118]),
    (112, [-112, 0]),      # features, activations, weights around and beyond the largest that is split
    (20, [95, -110]),
    (-100, [113, -20]),
    (120, [-120, 4]),
])
def test_operands_of_any_magnitude(x_exp, w_exps, bf16):
    """Powers of two on features and weights, down to subnormal numbers and up to the largest: plain fp32 arithmetic's
    tolerance holds at every magnitude (results and intermediates are normal numbers)."""
    rng = np.random.default_rng(71)
    d, widths, B, K = 96, [256, 40], 60, 1
    stack = rng.normal(size=(K + 1, 80, d)).astype(np.float32) * np.float32(2.0 ** x_exp)
    if bf16:
        stack = gp_synth.f32_to_bf16_bits(stack)
    Ws = [(W * 2.0 ** e).astype(np.float32) for W, e in zip(make_weights(rng, d, widths), w_exps)]
    check(stack, rng.integers(0, 80, B), [0.5, 0.25], Ws, bf16=bf16)


def test_small_operands_beside_large_ones():
    """Half of the features are tiny and meet large weights, the other half the other way round: both halves count alike."""
    rng = np.random.default_rng(72)
    d, widths, B, K = 128, [256, 40], 60, 0
    stack = rng.normal(size=(K + 1, 80, d)).astype(np.float32)
    Ws = make_weights(rng, d, widths)
    stack[:, :, ::2] *= np.float32(2.0 ** -120)
    Ws[0][::2] *= np.float32(2.0 ** 60)
    Ws[0][1::2] *= np.float32(2.0 ** -60)
    check(stack, rng.integers(0, 80, B), [1.0], Ws)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [1, 2, 15, 16, 17, 257, 272])
def test_short_sums_are_plain_fp32(d, bf16):
    """A first layer (or its last panel) of few terms, numbers just above a power of two, where the parts that six bf16
    products leave out are largest.  The second layer picks single columns, which changes nothing, so the result is
    the first layer's: one term is a product rounded once, and n terms keep n roundings."""
    rng = np.random.default_rng(81 + d)
    n, N, C = 100, 256, 64
    stack = (1.0 + rng.uniform(0.0, 2.0 ** -7, size=(1, n, d))).astype(np.float32)
    if bf16:
        stack = gp_synth.f32_to_bf16_bits(stack)
    W1 = (1.0 + rng.uniform(0.0, 2.0 ** -7, size=(d, N))).astype(np.float32)
    W2 = np.zeros((N, C), np.float32)
    cols = rng.permutation(N)[:C]
    W2[cols, np.arange(C)] = 1.0
    got = run(stack, np.arange(n), [1.0], [W1, W2], bf16=bf16)
    wide = (gp_synth.bf16_bits_to_f32(stack) if bf16 else stack)[0].astype(np.float64)
    want = wide @ W1.astype(np.float64)[:, cols]
    assert np.all(np.abs(got - want) <= d * 2.0 ** -24 * (1 + 1e-6) * want)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d,widths", [(40, [256, 200, 41]), (300, [100, 250, 64]), (128, [256, 256, 40]), (128, [256, 40]), (60, [130, 40])])
def test_a_row_does_not_depend_on_the_rows_beside_it(d, widths, bf16):
    """Rows with an infinity, a NaN or a very large number change nothing in the other rows, bit for bit; nor do the
    number of rows in the batch and the height of the work items."""
    rng = np.random.default_rng(91 + d)
    n, K, B = 400, 1, 333
    stack = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    Ws = make_weights(rng, d, widths)
    gamma = [0.5, 0.25]
    odd = stack.copy()
    odd[0, 1, 3], odd[1, 1, 7], odd[0, 2, 5], odd[1, 3, 0], odd[0, 3, 1] = np.inf, -np.inf, np.nan, 3e38, -2e35
    odd[1, 4] *= np.float32(1e30)     # finite sums beyond those that may be split
    if bf16:
        stack, odd = gp_synth.f32_to_bf16_bits(stack), gp_synth.f32_to_bf16_bits(odd)
        odd[0, 2, 5] = 0x7FC0
    ids = rng.integers(5, n, B)
    plain = run(stack, ids, gamma, Ws, bf16=bf16)
    mixed = ids.copy()
    at = rng.permutation(B)[:40]
    mixed[at] = 1 + np.arange(40) % 4
    rest = np.setdiff1d(np.arange(B), at)
    with np.errstate(all="ignore"):
        got = run(odd, mixed, gamma, Ws, bf16=bf16)
    assert not np.all(np.isfinite(got[at])) and np.array_equal(got[rest], plain[rest])
    assert np.array_equal(run(stack, ids[:7], gamma, Ws, bf16=bf16), plain[:7])
    assert np.array_equal(run(stack, np.tile(ids, 20), gamma, Ws, bf16=bf16)[-B:], plain)
    for rows in (32, 64):
        gp.gp_set_option("lc_tile_rows", rows)
        try:
            assert np.array_equal(run(stack, ids, gamma, Ws, bf16=bf16), plain)
        finally:
            gp.gp_set_option("lc_tile_rows", 0)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d,widths,K,B", [
    (39, [128], 3, 700), (40, [128], 3, 700),                # the last model on the fp32 instruction, the first in six products
    (124, [40], 1, 90), (128, [40], 1, 90), (127, [64, 64], 1, 40),
    (128, [128, 40], 0, 512 * 16), (128, [128, 40], 0, 512 * 32), (128, [128, 40], 0, 512 * 32 + 1),  # weights split where they are used
    (128, [256, 250], 1, 100), (129, [256, 250], 1, 100), (160, [256, 40], 3, 64 * 16), (160, [256, 40], 3, 64 * 16 + 1),  # .. or beforehand
    (192, [256] * 4, 0, 60), (193, [256] * 4, 0, 60), (224, [256, 256], 0, 6000), (225, [256, 256], 0, 6000),
    (100, [131, 77, 40], 0, 50), (64, [253, 66, 129], 1, 50),  # .. lanes whose last columns lie beyond the layer
    (150, [64, 40], 0, 2048 * 32), (150, [64, 40], 0, 2048 * 32 + 1), (257, [64, 40], 0, 512 * 32 + 1),
    (600, [64, 16], 3, 40), (600, [64, 16], 0, 16),          # 16 rows to an item, three panels
    (100, [256, 172, 41], 3, 1), (256, [65] * 7 + [10], 0, 17), (270, [70, 130], 2, 600),
])
def test_edges_of_the_rules(d, widths, K, B, bf16):
    """Both sides of every line at which another kernel, or another way for the weights, is taken, with the work items'
    height left to the library: 16 rows in the small batches."""
    rng = np.random.default_rng(101 + d + B)
    n = 300
    stack = rng.normal(size=(K + 1, n, d)).astype(np.float32)
    if bf16:
        stack = gp_synth.f32_to_bf16_bits(stack)
    check(stack, rng.integers(0, n, B), rng.normal(size=K + 1), make_weights(rng, d, widths), bf16=bf16, ldo_pad=1)
