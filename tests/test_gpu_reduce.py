"""Reductions over many workgroups: edges of their parts, streams and capture.

The result is a fixed tree over parts that depend on n alone, so eager launches
(many workgroups), launches on streams and launches in a captured graph (one
workgroup) give the same bits; against an exactly rounded sum the error of the
terms stays below the roundings of a term in its part (n / 65,536 of them), the
two trees and the products: 1e-14 of the sum of magnitudes.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 2048, 2049, 278_851, 2048 * 256 + 1, 1_000_003])
def test_dot_and_absmax(n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1504_08340_amd import binding as B
    rng = np.random.default_rng(n)
    a, b, w = rng.standard_normal((3, n))
    ta, tb, tw = (torch.tensor(v, device="cuda") for v in (a, b, w))
    out = torch.zeros(4, dtype=torch.float64, device="cuda")
    B.fwi_dot(None, n, ta, tb, tw, out[0:1])
    B.fwi_dot(None, n, ta, tb, None, out[1:2])
    B.fwi_absmax(None, n, ta, out[2:3])
    eager = out.clone()
    got = eager.cpu().numpy()
    for v, terms in ((got[0], a * b * w), (got[1], a * b)):
        assert abs(v - math.fsum(terms)) <= 1e-14 * np.abs(terms).sum()
    assert got[2] == np.abs(a).max()
    # two streams at once, each with its own results
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [torch.zeros(20, dtype=torch.float64, device="cuda") for _ in streams]
    torch.cuda.synchronize()
    for k in range(20):
        for st, o in zip(streams, outs):
            B.fwi_dot(st.cuda_stream, n, ta, tb, tw, o[k:k + 1])
    torch.cuda.synchronize()
    for o in outs:
        assert torch.equal(o, eager[0].expand(20))
    # captured, replayed beside eager launches
    g = torch.cuda.CUDAGraph()
    cap = torch.zeros(2, dtype=torch.float64, device="cuda")
    with torch.cuda.graph(g):
        B.fwi_dot(None, n, ta, tb, tw, cap[0:1])
        B.fwi_absmax(None, n, ta, cap[1:2])
    for _ in range(3):
        cap.fill_(-1.0)
        g.replay()
        B.fwi_dot(None, n, ta, tb, tw, out[3:4])
        torch.cuda.synchronize()
        assert cap[0] == eager[0] and cap[1] == eager[2] and out[3] == eager[0]


# The regularization's gradient by tiles of 4x4x2 bricks: one brick, one tile,
# a brick more along every axis, several tiles with one short of full.
@pytest.mark.parametrize("ne", [(1, 1, 1), (4, 4, 2), (5, 5, 3), (9, 3, 4), (3, 8, 7)])
def test_regularization_gradient_at_tile_edges(ne):
    """Sums of at most 72 terms with cancelling signs, FP64: 1e-12 of the largest."""
    import torch
    import paper_1504_08340_amd as P
    import workloads as W
    from oracle.regularize import Regularizer
    wl = W.tiny(ne_int=ne, nsteps=2, seed=9)
    r = Regularizer(wl.prob)
    S = P.Solver(wl.prob, wl.src_node, wl.src_dir, wl.rec_node)
    f = wl.lam / np.abs(wl.lam).max()
    v, g = S.tensor(np.zeros(1)), S.tensor(np.zeros(f.size))
    for kind, eps in ((P.FWI_REG_TIKHONOV, 0.0), (P.FWI_REG_TV, 1e-3)):
        P.fwi_regularization(S.plan, None, kind, eps, S.tensor(f), v, g)
        vo, go = r.tikhonov(f) if kind == P.FWI_REG_TIKHONOV else r.total_variation(f, eps)
        assert abs(float(v[0]) - vo) <= 1e-12 * abs(vo)
        assert np.abs(g.cpu().numpy() - go).max() <= 1e-12 * np.abs(go).max()
    torch.cuda.synchronize()
    S.close()
