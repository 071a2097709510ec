"""The matrix-core convolutions where their tiles and loads end.

Channel counts around 16, 32 and their multiples, position counts around 32,
extents that allow vector loads and that do not, strides that leave taps without
outputs, and enough positions for one, two and four waves a tile.  Against the
FP64 oracle: FP32 within 1e-5 of the largest magnitude (FP32 sums of up to 2000
products), the BF16 output within one BF16 unit.
"""
import numpy as np
import pytest

import oracle.convnet as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("xs,co,K,strides,relu", [
    ((1, 1, 1, 1, 1), 1, 1, (1, 1, 1), False),
    ((1, 1, 3, 3, 3), 1, 3, (2, 2, 2), True),
    ((2, 31, 4, 4, 8), 33, 3, (1, 1, 1), True),       # vector loads of both operands
    ((1, 33, 5, 6, 12), 17, 3, (2, 1, 1), True),
    ((2, 32, 6, 7, 5), 64, 3, (1, 2, 3), False),      # scalar loads, w stride 3
    ((3, 16, 2, 4, 16), 16, 1, (1, 1, 1), True),
    ((2, 40, 3, 8, 4), 2, 1, (2, 2, 1), False),
    ((4, 3, 24, 32, 32), 5, 3, (1, 1, 1), True),      # a wave per tile
    ((2, 5, 16, 32, 36), 7, 3, (1, 1, 1), False),     # two
])
def test_conv_edges(xs, co, K, strides, relu):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(3)
    x = rng.standard_normal(xs).astype(np.float32)
    w = (rng.standard_normal((co, xs[1], K, K, K)) / np.sqrt(xs[1] * K ** 3)).astype(np.float32)
    b = rng.standard_normal(co).astype(np.float32)
    y_o = C.conv3d_forward(x.astype(np.float64), w.astype(np.float64), b.astype(np.float64), strides, relu)
    dy = rng.standard_normal(y_o.shape).astype(np.float32)
    X, Wt, Bt, DY = (torch.tensor(a, device="cuda") for a in (x, w, b, dy))
    sh = B.conv_shape(*xs, co, K, strides)
    Y = torch.empty(y_o.shape, dtype=torch.float32, device="cuda")
    B.fwi_conv3d_forward(None, sh, X, Wt, Bt, relu, Y)
    got = Y.cpu().numpy().astype(np.float64)
    # the mask is the library's own output's: a value within rounding of 0 may fall either way
    dx_o, dw_o, db_o = C.conv3d_backward(x.astype(np.float64), w.astype(np.float64), got, dy.astype(np.float64),
                                         strides, relu)
    DX, DW, DB = torch.empty_like(X), torch.empty_like(Wt), torch.empty_like(Bt)
    B.fwi_conv3d_backward(None, sh, X, Wt, Y, DY, relu, DX, DW, DB)
    for a, ref in ((got, y_o), (DX.cpu().numpy(), dx_o), (DW.cpu().numpy(), dw_o), (DB.cpu().numpy(), db_o)):
        assert np.abs(a - ref).max() <= 1e-5 * max(np.abs(ref).max(), 1e-30)
    # the same from pointers that are not on 16 bytes
    if relu:
        pad = [torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t) for t in (X, Y, DY)]
        DW2 = torch.empty_like(Wt)
        B.fwi_conv3d_backward(None, sh, pad[0], Wt, pad[1], pad[2], relu, None, DW2, None)
        assert np.abs(DW2.cpu().numpy() - dw_o).max() <= 1e-5 * max(np.abs(dw_o).max(), 1e-30)
    Xb, Wb = X.bfloat16(), Wt.bfloat16()
    ref = C.conv3d_forward(C.bf16_round(x), C.bf16_round(w), b.astype(np.float64), strides, relu)
    Yb = torch.empty(ref.shape, dtype=torch.bfloat16, device="cuda")
    B.fwi_conv3d_forward_bf16(None, sh, Xb, Wb, Bt, relu, 0, Yb)
    got = Yb.float().cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-5 * np.abs(ref).max())


def _chains(terms):
    """256 chains over the last axis (outputs through the batch) of (a, b) products, one
    multiply-add after another in FP32, then the tree; b None: sums of a."""
    a, b = terms
    n = -(-a.shape[-1] // 256) * 256
    pad = [(0, 0)] * (a.ndim - 1) + [(0, n - a.shape[-1])]
    a = np.pad(a, pad).astype(np.float64).reshape(*a.shape[:-1], -1, 256)
    b = np.ones_like(a) if b is None else np.pad(b, pad).astype(np.float64).reshape(a.shape)
    acc = np.zeros((*a.shape[:-2], 256), np.float32)
    for k in range(a.shape[-2]):     # the product is exact in FP64, the sum's rounding there far below FP32's
        acc = (a[..., k, :] * b[..., k, :] + acc).astype(np.float32)
    while acc.shape[-1] > 1:
        h = acc.shape[-1] // 2
        acc = acc[..., :h] + acc[..., h:]
    return acc[..., 0]


@pytest.mark.parametrize("xs,co,strides", [
    ((2, 5, 4, 6, 8), 7, (1, 1, 1)),       # vector loads
    ((3, 3, 5, 8, 16), 18, (2, 1, 2)),     # vector loads, w stride 2
    ((2, 17, 4, 6, 9), 3, (1, 2, 2)),      # scalar loads; outputs that a chunk of 16 shares across samples
])
def test_weight_gradient_order(xs, co, strides):
    """The order of the sums is part of the result: bit for bit against the chains
    above, over several workgroups a tile and (captured) in one."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(4)
    N, ci, K = xs[0], xs[1], 3
    x = rng.standard_normal(xs).astype(np.float32)
    out = [(n - 1) // s + 1 for n, s in zip(xs[2:], strides)]
    y, dy = (rng.standard_normal((N, co, *out)).astype(np.float32) for _ in range(2))
    g = np.where(y > 0, dy, np.float32(0)).transpose(1, 0, 2, 3, 4).reshape(co, -1)
    xp = np.pad(x, [(0, 0), (0, 0), (1, 1), (1, 1), (1, 1)])
    dw = np.empty((co, ci, K, K, K), np.float32)
    for kd in range(K):
        for kh in range(K):
            for kw in range(K):
                at = [slice(k, k + (n - 1) * s + 1, s) for k, n, s in zip((kd, kh, kw), out, strides)]
                v = xp[(slice(None), slice(None), *at)].transpose(1, 0, 2, 3, 4).reshape(ci, -1)
                dw[:, :, kd, kh, kw] = _chains([t.copy() for t in np.broadcast_arrays(g[:, None], v[None])])
    db = _chains((g, None))
    sh = B.conv_shape(*xs, co, K, strides)
    X, Y, DY, Wt = (torch.tensor(a, device="cuda") for a in (x, y, dy, dw))
    DW, DB = torch.empty_like(Wt), torch.empty(co, device="cuda")
    B.fwi_conv3d_backward(None, sh, X, Wt, Y, DY, True, None, DW, DB)
    assert np.array_equal(DW.cpu().numpy(), dw) and np.array_equal(DB.cpu().numpy(), db)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.fwi_conv3d_backward(None, sh, X, Wt, Y, DY, True, None, DW, DB)
    for _ in range(3):
        DW.zero_()
        DB.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(DW.cpu().numpy(), dw) and np.array_equal(DB.cpu().numpy(), db)
