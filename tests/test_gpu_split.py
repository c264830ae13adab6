"""Split items (fp32 dot products as bf16 part products) where they can go
wrong, in the tiled and the series-lane layout: the shortest and longest rows
they take, lengths that leave one column in the last tile or block, 1 to 65
kernels of a dilation, every kernel length, kernels of many widths in one item,
exact sums, series scaled to the ends of the fp32 range, rows beside a row of
NaN and infinities, calls of all sizes and captured calls."""
import sys

import numpy as np
import pytest

from _util import assert_mpv_parity, assert_parity, full_dilations_set, kernel_set, many_widths_set

pytestmark = pytest.mark.gpu


def _log(msg):
    print("[gpu-split] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_2601_17091_amd as rk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rk.library()
    return torch, rk


def _run(env, ks, X, split=True, **kw):
    """Features of X; split: whether the plan has to have split items (None:
    either)."""
    torch, rk = env
    plan = rk.Plan(ks, X.shape[1], **kw)
    assert split is None or (plan.info()["split_items"] > 0) == split
    F = plan.transform(torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    return F.cpu().numpy()


def _check(F, ref, mpv, what):
    (assert_mpv_parity if mpv else assert_parity)(F, ref, what)


# 129: the shortest; 193, 257: one column in a last tile, a last block; 1,021:
# odd; 3,200: the last with two rows per workgroup; 6,463 / 6,464 / 6,465 and
# 9,983 / 9,984 / 9,985: around the rows that take the next workgroup shape;
# 20,255: near the longest; 20,300: too long (fp32 items)
@pytest.mark.parametrize("L", [129, 193, 257, 1021, 3200, 6463, 6464, 6465, 9983, 9984, 9985, 20255, 20300])
def test_row_lengths(env, oracle, L):
    _, rk = env
    K = 2500 if L < 4000 else 4000   # enough that split items pay at this length
    ks = rk.generate_kernels(3000 + L, K, L)
    rng = np.random.default_rng(L)
    X = rng.standard_normal((5 if L < 4000 else 2, L)).cumsum(1)
    X = ((X - X.mean(1, keepdims=True)) / X.std(1, keepdims=True)).astype(np.float32)
    ref = oracle.transform(X, ks)
    for mpv in (False, True):
        _log("L=%d mpv=%s" % (L, mpv))
        _check(_run(env, ks, X, split=L < 20300, mpv=mpv), ref, mpv, "L=%d" % L)


@pytest.mark.parametrize("L,kw", [(41, {}), (41, dict(series=True)), (131, {}), (321, {}), (321, dict(clamped=True))])
def test_lengths_and_paddings(env, oracle, L, kw):
    """Items of several lengths, even ones among them, of three and four
    widths (an item masks two or four), and of kernels with one output."""
    ks = many_widths_set(L, L)
    X = np.random.default_rng(17 + L).standard_normal((4, L)).astype(np.float32)
    _log("lengths and paddings L=%d %s, %d kernels" % (L, kw, len(ks["length"])))
    ref = oracle.transform(X, ks)
    for mpv in (False, True):
        _check(_run(env, ks, X, mpv=mpv, **kw), ref, mpv, "paddings")


@pytest.mark.parametrize("L", [41, 321])
def test_exact_sums(env, oracle, L):
    """Integer series, weights and biases: every partial sum is exact, so PPV
    and MAX equal the oracle's, with many sums that cancel to zero."""
    ks = many_widths_set(L, L)
    rng = np.random.default_rng(L)
    ks["weights"] = np.where(ks["weights"] != 0, rng.integers(-2, 3, ks["weights"].shape), 0).astype(np.float32)
    ks["bias"] = rng.choice([-2, -1, 1, 2], len(ks["bias"])).astype(np.float32)
    X = rng.integers(-3, 4, (5, L)).astype(np.float32)
    X[1], X[2], X[3] = 0.0, np.float32(-0.0), 1.5
    _log("exact sums L=%d" % L)
    ref = oracle.transform(X, ks)
    for kw in ([dict(series=True), {}] if L <= 128 else [{}]):
        F = _run(env, ks, X, **kw)
        np.testing.assert_array_equal(F[:, 0::2], ref["cnt"].astype(np.float32) / ref["O"][None].astype(np.float32))
        np.testing.assert_array_equal(F[:, 1::2], ref["F"][:, 1::2])


@pytest.mark.parametrize("count", [1, 2, 15, 31, 32, 33, 65])
def test_kernels_per_dilation(env, oracle, count):
    """A dilation's kernels fill one item, one less, one more, and two (a
    handful is left to fp32 items)."""
    ks = full_dilations_set(400, count, count)
    X = np.random.default_rng(count).standard_normal((3, 400)).astype(np.float32)
    _log("%d kernels of each length at a dilation" % count)
    _check(_run(env, ks, X, split=count >= 15), oracle.transform(X, ks), False, "count=%d" % count)


@pytest.mark.parametrize("e", [-80, -40, 40, 110])
def test_power_of_two_scaling(env, e):
    """Scaling the series and the biases by 2^e scales every part, product
    and sum exactly (all parts stay normal at 2^-80): PPV is unchanged and
    MAX scales bit for bit, up to sums near the fp32 maximum."""
    _, rk = env
    ks = rk.generate_kernels(77, 1500, 300)
    rng = np.random.default_rng(5)
    X = rng.standard_normal((3, 300)).astype(np.float32)
    a = _run(env, ks, X)
    ks2 = dict(ks, bias=np.ldexp(ks["bias"], e).astype(np.float32))
    _log("scaled by 2^%d" % e)
    b = _run(env, ks2, np.ldexp(X, e).astype(np.float32))
    np.testing.assert_array_equal(a[:, 0::2], b[:, 0::2])
    np.testing.assert_array_equal(np.ldexp(a[:, 1::2].astype(np.float64), e), b[:, 1::2].astype(np.float64))


def test_neighbour_rows_do_not_mix(env):
    """Rows of NaN and of infinities leave the features of the rows staged
    beside them as they are alone."""
    torch, rk = env
    for L in (150, 500):
        ks = rk.generate_kernels(78, 1500, L)
        rng = np.random.default_rng(6)
        X = rng.standard_normal((7, L)).astype(np.float32)
        want = _run(env, ks, X)
        Y = X.copy()
        Y[1], Y[4], Y[6] = np.nan, np.inf, -np.inf
        _log("rows of NaN and infinity, L=%d" % L)
        got = _run(env, ks, Y)
        keep = [0, 2, 3, 5]
        np.testing.assert_array_equal(got[keep], want[keep])


@pytest.mark.parametrize("L,bias", [(500, True), (9985, True), (9985, False)])
def test_captured_call(env, L, bias):
    """A call under graph capture, in a layout whose fp32 items run beside the
    split items (without biases: fp32 and Toeplitz items alone), and an eager
    call of the same plan on another stream before the capture ends: both give
    what an eager call gives, at every replay."""
    torch, rk = env
    ks = rk.generate_kernels(81, 1500 if L < 9985 else 6000, L)
    if not bias:
        ks["bias"][:] = 0.0
    plan = rk.Plan(ks, L, clamped=True)
    info = plan.info()
    assert (info["split_items"] > 0) == bias
    assert info["toeplitz_items"] > 0 or L == 500
    X = torch.randn((6, L), device="cuda")
    want = plan.transform(X)
    F, F2 = torch.zeros_like(want), torch.zeros_like(want)
    other, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    _log("captured call L=%d" % L)
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        plan.transform_into(X, F)
        plan.transform_into(X, F2, stream=other)
    torch.cuda.synchronize()
    assert torch.equal(F2, want)
    for _ in range(3):
        F.fill_(-1)
        F2 = plan.transform(X)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(F, want) and torch.equal(F2, want)


@pytest.mark.parametrize("L,n", [(11, 65), (16, 31), (63, 97), (64, 64), (65, 130), (127, 33), (128, 193)])
def test_series_lane_layout(env, oracle, L, n):
    """Short series, 32 to a tile: series counts around the 32 of a tile and
    the 64 of a workgroup, odd and even numbers of positions; the tiled layout
    of the same kernels gives the same PPV and MAX bit for bit."""
    _, rk = env
    K = 1500
    ks = rk.generate_kernels(4000 + L, K, L)
    rng = np.random.default_rng(L)
    X = rng.standard_normal((n, L)).astype(np.float32)
    ref = oracle.transform(X, ks)
    for mpv in (False, True):
        _log("series-lane L=%d n=%d mpv=%s" % (L, n, mpv))
        F = _run(env, ks, X, mpv=mpv, series=True)
        _check(F, ref, mpv, "series L=%d" % L)
        T = _run(env, ks, X, mpv=mpv, tiled=True)
        nf = 3 if mpv else 2
        np.testing.assert_array_equal(F[:, 0::nf], T[:, 0::nf])
        np.testing.assert_array_equal(F[:, 1::nf], T[:, 1::nf])


@pytest.mark.parametrize("L,d,kw", [(100, 1 << 24, dict(series=True)), (100, 1 << 24, dict(tiled=True)),
                                    (100, 1 << 16, dict(series=True)), (500, 1 << 16, {}), (500, 1 << 28, {})])
def test_far_taps(env, oracle, L, d, kw):
    """Dilations far beyond the series, with paddings to match: the outer taps
    of every output read padding."""
    rng = np.random.default_rng(L)
    n = 64
    ks = kernel_set([3] * n, [d] * n, [d] * n, rng.uniform(-1, 1, n), [rng.standard_normal(3) for _ in range(n)])
    X = rng.standard_normal((70, L)).astype(np.float32)
    _log("far taps L=%d d=%d %s" % (L, d, kw))
    _check(_run(env, ks, X, split=None, **kw), oracle.transform(X, ks), False, "far taps")


@pytest.mark.parametrize("L,kw", [(100, dict(series=True)), (100, dict(tiled=True)), (400, {})])
def test_tiny_samples(env, L, kw):
    """Samples of about 2^-120 under kernels without bias: scaling by a power
    of two is exact but for sums that round at 2^-149 (2^-29 of 2^-120), which
    can turn a later rounding: at most one unit in the last place of each of
    11 partial sums, below 16 x 2^-120.  (Samples cut to bf16 parts would be
    off by 2^-14.)"""
    _, rk = env
    ks = rk.generate_kernels(83, 1500, L)
    ks["bias"][:] = 0.0
    rng = np.random.default_rng(83)
    X = rng.standard_normal((4, L)).astype(np.float32)
    _log("tiny samples L=%d %s" % (L, kw))
    a, b = (_run(env, ks, Y, split=False, **kw) for Y in (X, np.ldexp(X, -120).astype(np.float32)))
    back = np.ldexp(b[:, 1::2].astype(np.float64), 120)
    np.testing.assert_allclose(back, a[:, 1::2], rtol=0, atol=11 * 2.0 ** -20)


# 300: a few items per workgroup, dealt to its wavefronts in parts, and over
# all XCDs in the short calls; 2,000: the long call's fp32 items run beside the
# split items, the short calls' in their launch; 11,000: one workgroup per CU;
# 64: series-lane, half the series of a workgroup at a time
@pytest.mark.parametrize("L,K,n,mpv", [(300, 600, 3000, False), (300, 2000, 700, True), (2000, 1000, 500, False),
                                       (2000, 5000, 150, True), (11000, 600, 40, False), (64, 400, 4200, False),
                                       (128, 600, 4200, False)])
def test_rows_do_not_depend_on_the_call(env, oracle, L, K, n, mpv):
    torch, rk = env
    ks = rk.generate_kernels(900 + L, K, L)
    rng = np.random.default_rng(L + K)
    X = rng.standard_normal((n, L)).cumsum(1).astype(np.float32)
    X /= np.abs(X).max(1, keepdims=True)
    plan = rk.Plan(ks, L, mpv=mpv)
    assert plan.info()["split_items"] > 0
    _log("rows of calls of any size L=%d K=%d n=%d mpv=%s" % (L, K, n, mpv))
    Xd = torch.from_numpy(X).cuda()
    F = plan.transform(Xd)
    for lo, hi in ((0, 1), (1, 4), (5, 22), (n - 3, n)):
        assert torch.equal(plan.transform(Xd[lo:hi].contiguous()), F[lo:hi]), (lo, hi)
    rows = [0, n // 2, n - 1]
    _check(F[rows].cpu().numpy(), oracle.transform(X[rows], ks), mpv, "rows of a long call")
