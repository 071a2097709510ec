"""Which convolution kernel takes a call, at the lines between them.

The weight gradient works in tiles of 4 or of 8 channels (by the number of
workgroups), with vector loads at w stride 1 or 2 or element by element; every form
sums in the same order, so each is compared bit for bit with chains formed here.
"""
import time

import numpy as np
import pytest

from test_gpu_conv_edges import _chains

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return torch


@pytest.mark.parametrize("xs,co,K,strides,relu", [
    ((1, 29, 3, 4, 8), 31, 3, (1, 1, 1), True),     # 576 workgroups of 4 x 4 channels: tiles of 8; vector loads
    ((2, 30, 3, 5, 16), 32, 3, (2, 1, 2), False),   # the same at w stride 2
    ((1, 31, 4, 5, 7), 29, 3, (1, 2, 3), True),     # element by element
    ((3, 90, 2, 3, 8), 92, 1, (1, 1, 1), True),     # 1x1x1, tiles of 8
    ((2, 90, 2, 3, 5), 91, 1, (1, 1, 1), False),
    ((5, 3, 1, 1, 4), 2, 1, (1, 1, 1), True),       # tiles of 4, fewer outputs than chains
    ((1, 6, 5, 7, 9), 9, 3, (1, 1, 1), False),
])
def test_weight_gradient_forms(xs, co, K, strides, relu):
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(8)
    N, ci, p = xs[0], xs[1], K // 2
    x = rng.standard_normal(xs).astype(np.float32)
    out = [(n + 2 * p - K) // s + 1 for n, s in zip(xs[2:], strides)]
    y, dy = (rng.standard_normal((N, co, *out)).astype(np.float32) for _ in range(2))
    g = (np.where(y > 0, dy, np.float32(0)) if relu else dy).transpose(1, 0, 2, 3, 4).reshape(co, -1)
    xp = np.pad(x, [(0, 0), (0, 0)] + [(p, p)] * 3)
    dw = np.empty((co, ci, K, K, K), np.float32)
    for kd, kh, kw in np.ndindex(K, K, K):
        at = [slice(k, k + (n - 1) * s + 1, s) for k, n, s in zip((kd, kh, kw), out, strides)]
        v = xp[(slice(None), slice(None), *at)].transpose(1, 0, 2, 3, 4).reshape(ci, -1)
        dw[:, :, kd, kh, kw] = _chains([t.copy() for t in np.broadcast_arrays(g[:, None], v[None])])
    db = _chains((g, None))
    X, Y, DY, Wt = (torch.tensor(a, device="cuda") for a in (x, y, dy, dw))
    DW, DB = torch.empty_like(Wt), torch.empty(co, device="cuda")
    B.fwi_conv3d_backward(None, B.conv_shape(*xs, co, K, strides), X, Wt, Y, DY, relu, None, DW, DB)
    assert np.array_equal(DW.cpu().numpy(), dw) and np.array_equal(DB.cpu().numpy(), db)


@pytest.mark.parametrize("xs,co", [((4, 3, 24, 32, 32), 5), ((2, 48, 8, 8, 8), 48)])
def test_weight_gradient_takes_as_long_on_every_route(xs, co):
    """Eager, captured, and on a stream after many others have been used: the same
    launch, so about the same time (twice is allowed)."""
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    sh = B.conv_shape(*xs, co, 3, (1, 1, 1))
    X = torch.randn(xs, device="cuda")
    DY = torch.randn(xs[0], co, *xs[2:], device="cuda")
    W = torch.empty(co, xs[1], 3, 3, 3, device="cuda")
    DW = torch.empty_like(W)

    def call(stream):
        B.fwi_conv3d_backward(stream, sh, X, W, DY, DY, True, None, DW, None)

    def best(f):
        f()
        torch.cuda.synchronize()
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            for _ in range(20):
                f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    eager = best(lambda: call(None))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(None)
    assert best(graph.replay) < 2 * eager
    streams = [torch.cuda.Stream() for _ in range(12)]
    a = torch.ones(4096, dtype=torch.float64, device="cuda")
    o = torch.empty(1, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for s in streams[:-1]:
        B.fwi_dot(s.cuda_stream, a.numel(), a, a, None, o)
        torch.cuda.synchronize()
    assert best(lambda: call(streams[-1].cuda_stream)) < 2 * eager


@pytest.mark.parametrize("K", [1, 3])
def test_more_positions_than_32_bits_count(K):
    """One sample and channel of 1291^3 = 2^31 + 4.2e6 positions: forward, data, weight
    and bias gradients.  Small whole numbers, so that every sum is exact in FP32 (the
    largest partial sums, of 2^31 terms of both signs, stay below 2^24)."""
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    n, p = 1291, K // 2
    gen = torch.Generator(device="cuda").manual_seed(3)

    def signs():
        return torch.randint(-1, 2, (n, n, n), generator=gen, device="cuda", dtype=torch.int8).float()

    X, DY = signs(), signs()
    W = torch.randint(-3, 4, (1, 1, K, K, K), generator=gen, device="cuda").float()
    b = torch.ones(1, device="cuda")
    Y, DX = torch.full_like(X, 7.0), torch.full_like(X, 7.0)
    DW, DB = torch.empty_like(W), torch.empty(1, device="cuda")
    sh = B.conv_shape(1, 1, n, n, n, 1, K, (1, 1, 1))
    B.fwi_conv3d_forward(None, sh, X, W, b, True, Y)
    torch.cuda.synchronize()
    print("forward done", flush=True)
    B.fwi_conv3d_backward(None, sh, X, W, Y, DY, True, DX, DW, DB)
    torch.cuda.synchronize()
    print("backward done", flush=True)
    taps = list(np.ndindex(K, K, K))
    dw, db = torch.zeros(len(taps), dtype=torch.float64, device="cuda"), 0.0

    def padded(t, a, e):            # planes [a - p, e + p) of t, zeros around
        out = torch.zeros(e - a + 2 * p, n + 2 * p, n + 2 * p, device="cuda")
        lo, hi = max(a - p, 0), min(e + p, n)
        out[lo - a + p:hi - a + p, p:p + n, p:p + n] = t[lo:hi]
        return out

    def shifted(t, k, m):
        return t[k[0]:k[0] + m, k[1]:k[1] + n, k[2]:k[2] + n]

    for a in range(0, n, 64):
        e = min(a + 64, n)
        xp, m = padded(X, a, e), e - a
        g = torch.where(Y[a:e] > 0, DY[a:e], torch.zeros((), device="cuda"))
        y = torch.ones(m, n, n, device="cuda")
        for i, k in enumerate(taps):
            y += W[0, 0][k] * shifted(xp, k, m)
            dw[i] += (g * shifted(xp, k, m)).sum(dtype=torch.float64)
        assert torch.equal(Y[a:e], y.relu())
        db += float(g.sum(dtype=torch.float64))
    for a in range(0, n, 64):
        e = min(a + 64, n)
        lo, hi = max(a - p, 0), min(e + p, n)
        G = torch.zeros(e - a + 2 * p, n + 2 * p, n + 2 * p, device="cuda")
        G[lo - a + p:hi - a + p, p:p + n, p:p + n] = torch.where(Y[lo:hi] > 0, DY[lo:hi], torch.zeros((), device="cuda"))
        dx = torch.zeros(e - a, n, n, device="cuda")
        for k in taps:
            dx += W[0, 0][k] * shifted(G, tuple(2 * p - q for q in k), e - a)
        assert torch.equal(DX[a:e], dx)
    assert torch.equal(DW.double().flatten(), dw) and float(DB) == db


def _taps(n, k, s, K):
    """Outputs along an axis that have tap k, and their places in the input."""
    o = np.arange((n + 2 * (K // 2) - K) // s + 1)
    i = o * s + k - K // 2
    keep = (i >= 0) & (i < n)
    return o[keep], i[keep]


def _conv_both(x, w, b, g, strides):
    """y = b + w * x and dx = w^T * g in FP64, tap by tap: a place outside contributes
    nothing, whatever the weight."""
    K = w.shape[2]
    out = [(n + 2 * (K // 2) - K) // s + 1 for n, s in zip(x.shape[2:], strides)]
    y = np.broadcast_to(b[None, :, None, None, None], (x.shape[0], w.shape[0], *out)).copy()
    dx = np.zeros(x.shape)
    with np.errstate(all="ignore"):
        for k in np.ndindex(K, K, K):
            o, i = zip(*(_taps(n, q, s, K) for n, q, s in zip(x.shape[2:], k, strides)))
            oi, ii = (slice(None), slice(None), *np.ix_(*o)), (slice(None), slice(None), *np.ix_(*i))
            wk = w[:, :, k[0], k[1], k[2]]
            # products before sums: an infinite weight times 0 is no number, times a value infinite
            y[oi] = y[oi] + (wk[None, :, :, None, None, None] * x[ii][:, None]).sum(2)
            dx[ii] = dx[ii] + (wk[None, :, :, None, None, None] * g[oi][:, :, None]).sum(1)
    return y, dx


@pytest.mark.parametrize("xs,co,K,strides", [
    ((2, 3, 5, 6, 7), 4, 3, (1, 1, 1)),
    ((1, 9, 6, 5, 9), 20, 3, (2, 1, 2)),
    ((2, 3, 4, 3, 5), 17, 1, (2, 1, 1)),
])
def test_a_weight_that_is_no_number_stays_with_its_tap(xs, co, K, strides):
    """Infinite and undefined weights of border taps: results that do not have the tap
    are what they are without it (FP32 within 1e-5 of the largest finite)."""
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(5)
    x, w = rng.standard_normal(xs), rng.standard_normal((co, xs[1], K, K, K))
    x, w, b = (a.astype(np.float32).astype(np.float64) for a in (x, w, rng.standard_normal(co)))
    w[0, 1, 0, 0, 0] = np.inf
    w[co - 1, 0, K - 1, K // 2, 0] = -np.inf
    w[1, 2, K // 2, 0, K - 1] = np.nan
    out = [(n + 2 * (K // 2) - K) // s + 1 for n, s in zip(xs[2:], strides)]
    g = rng.standard_normal((xs[0], co, *out)).astype(np.float32).astype(np.float64)
    y, dx = _conv_both(x, w, b, g, strides)
    X, W, b_, G = (torch.tensor(a, dtype=torch.float32, device="cuda") for a in (x, w, b, g))
    Y, DX, DW = torch.empty_like(G), torch.empty_like(X), torch.empty_like(W)
    sh = B.conv_shape(*xs, co, K, strides)
    B.fwi_conv3d_forward(None, sh, X, W, b_, False, Y)
    B.fwi_conv3d_backward(None, sh, X, W, G, G, False, DX, DW, None)
    for got, ref in ((Y, y), (DX, dx)):
        got, fin = got.cpu().numpy(), np.isfinite(ref)
        assert fin.any() and not fin.all()
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        assert np.abs(got[fin] - ref[fin]).max() <= 1e-5 * np.abs(ref[fin]).max()


@pytest.mark.parametrize("xs,co,K,strides", [
    ((2, 1, 7, 9, 11), 16, 3, (1, 1, 1)),       # few input channels: 16 taps a step
    ((1, 3, 33, 32, 31), 19, 3, (1, 1, 1)),     # as many positions as make that the faster one
    ((1, 3, 5, 7, 9), 19, 3, (2, 1, 2)),        # and as few as do not
    ((3, 16, 3, 5, 7), 16, 1, (1, 1, 1)),       # 1x1x1
    ((1, 17, 3, 5, 7), 33, 1, (1, 2, 1)),
])
@pytest.mark.parametrize("fp32", [0, 1])
def test_bf16_narrow_layers(xs, co, K, strides, fp32):
    """Against the FP64 oracle on the rounded operands, within one BF16 unit (FP32
    output: the accumulation's 1e-5 of the largest)."""
    torch = _torch()
    import oracle.convnet as C
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(6)
    x = rng.standard_normal(xs).astype(np.float32)
    w = (rng.standard_normal((co, xs[1], K, K, K)) / np.sqrt(xs[1] * K ** 3)).astype(np.float32)
    b = rng.standard_normal(co).astype(np.float32)
    ref = C.conv3d_forward(C.bf16_round(x), C.bf16_round(w), b.astype(np.float64), strides, True)
    X, W, b_ = (torch.tensor(a, device="cuda") for a in (x, w, b))
    Y = torch.empty(ref.shape, dtype=torch.float32 if fp32 else torch.bfloat16, device="cuda")
    B.fwi_conv3d_forward_bf16(None, B.conv_shape(*xs, co, K, strides), X.bfloat16(), W.bfloat16(), b_, True, fp32, Y)
    got = Y.float().cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= (0 if fp32 else 2.0 ** -7) * np.abs(ref) + 1e-5 * np.abs(ref).max())


def test_bf16_layer_of_one_channel_is_quick():
    """8 samples of 64x16x16, one channel to 16, stride (2, 1, 1): 9 us a call with the
    kernel for few channels, 35 us without it."""
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    sh = B.conv_shape(8, 1, 64, 16, 16, 16, 3, (2, 1, 1))
    X = torch.randn(8, 1, 64, 16, 16, device="cuda").bfloat16()
    W = torch.randn(16, 1, 3, 3, 3, device="cuda").bfloat16()
    Y = torch.empty(8, 16, 32, 16, 16, device="cuda", dtype=torch.bfloat16)
    t = []
    for _ in range(10):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(100):
            B.fwi_conv3d_forward_bf16(None, sh, X, W, None, True, 0, Y)
        torch.cuda.synchronize()
        t.append((time.perf_counter() - t0) / 100)
    assert min(t[1:]) < 20e-6


@pytest.mark.parametrize("xs,co,K,strides", [
    # a thread per result: one to two channels and many positions, one channel and few,
    # one position; K = 1
    ((3, 1, 45, 44, 46), 1, 3, (1, 1, 1)),
    ((2, 2, 51, 53, 55), 1, 3, (1, 1, 1)),
    ((2, 1, 9, 7, 5), 20, 3, (2, 1, 2)),
    ((4, 3, 1, 1, 1), 2, 3, (1, 1, 1)),
    ((2, 4, 7, 9, 11), 1, 1, (1, 2, 1)),
    ((2, 1, 7, 9, 11), 2, 1, (1, 1, 1)),
    # 32 rows a wave in both directions: 65,536 positions, or half as many and more than
    # 32 rows; channels that are no multiple of 32, a last tile that is not full
    ((2, 35, 26, 27, 25), 37, 3, (1, 1, 1)),
    ((3, 18, 29, 28, 27), 20, 1, (1, 1, 1)),
    # a position short of 65,536 (16 rows a wave)
    ((1, 18, 63, 32, 32), 17, 1, (1, 1, 1)),
])
def test_fp32_forms(xs, co, K, strides):
    """Forward and data gradient against FP64 sums (1e-5 of the largest magnitude)."""
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(11)
    x = rng.standard_normal(xs).astype(np.float32)
    w = (rng.standard_normal((co, xs[1], K, K, K)) / np.sqrt(xs[1] * K ** 3)).astype(np.float32)
    b = rng.standard_normal(co).astype(np.float32)
    X, W, b_ = (torch.tensor(a, device="cuda") for a in (x, w, b))
    out = [(n + 2 * (K // 2) - K) // s + 1 for n, s in zip(xs[2:], strides)]
    Y = torch.empty(xs[0], co, *out, device="cuda")
    DY = torch.tensor(rng.standard_normal(Y.shape).astype(np.float32), device="cuda")
    DX, DW = torch.empty_like(X), torch.empty_like(W)
    sh = B.conv_shape(*xs, co, K, strides)
    B.fwi_conv3d_forward(None, sh, X, W, b_, True, Y)
    B.fwi_conv3d_backward(None, sh, X, W, Y, DY, True, DX, DW, None)
    got = Y.cpu().numpy()
    # the mask is the library's own output's: a value within rounding of 0 may fall either way
    g = np.where(got > 0, DY.cpu().numpy(), 0).astype(np.float64)
    y, dx = np.empty(got.shape), np.zeros(xs)
    for n in range(xs[0]):
        y[n] = b[:, None, None, None]
        for k in np.ndindex(K, K, K):
            o, i = zip(*(_taps(m, q, s, K) for m, q, s in zip(xs[2:], k, strides)))
            oi, ii = (slice(None), *np.ix_(*o)), (slice(None), *np.ix_(*i))
            wk = w[:, :, k[0], k[1], k[2]].astype(np.float64)
            y[n][oi] += np.tensordot(wk, x[n][ii].astype(np.float64), 1)
            dx[n][ii] += np.tensordot(wk.T, g[n][oi], 1)
    for a, ref in ((got, np.maximum(y, 0)), (DX.cpu().numpy(), dx)):
        assert np.abs(a - ref).max() <= 1e-5 * np.abs(ref).max()
