"""Reductions without a slot (captured, on the per-thread default stream): one
workgroup, a wave a part.  The same bits as many workgroups give, and no slower than
one workgroup that streams the operands.
"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
PER_THREAD = 2          # hipStreamPerThread


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return torch


# one part; two; as many as waves, and one more; every part, and parts of two strides
@pytest.mark.parametrize("n", [7, 2048, 2049, 2048 * 16, 2048 * 16 + 1, 2048 * 256, 2048 * 300 + 5])
def test_every_route_gives_the_same_bits(n):
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(n)
    a, b, w = (torch.randn(n, generator=gen, dtype=torch.float64, device="cuda") for _ in range(3))
    y, t = a.float(), b.float()

    def calls(stream, o, l, g):
        B.fwi_dot(stream, n, a, b, w, o[0:1])
        B.fwi_dot(stream, n, a, b, None, o[1:2])
        B.fwi_absmax(stream, n, a, o[2:3])
        B.fwi_mse(stream, n, y, t, l, g)

    outs = [(torch.zeros(3, dtype=torch.float64, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros_like(y))
            for _ in range(3)]
    calls(None, *outs[0])
    torch.cuda.synchronize()
    calls(PER_THREAD, *outs[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(None, *outs[2])
    for _ in range(3):
        for v in outs[2]:
            v.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        for k in (1, 2):
            assert all(torch.equal(p, q) for p, q in zip(outs[0], outs[k]))
    r = (y.double() - t.double())
    assert abs(float(outs[0][1]) - float((r * r).sum()) / (2 * n)) <= 1e-6 * float(outs[0][1])


@pytest.mark.parametrize("ne", [(2, 3, 2), (9, 7, 5)])
def test_regularization_value_on_every_route(ne):
    torch = _torch()
    import paper_1504_08340_amd as P
    import workloads as W
    wl = W.tiny(ne_int=ne, nsteps=2, seed=9)
    S = P.Solver(wl.prob, wl.src_node, wl.src_dir, wl.rec_node)
    f, v = S.tensor(wl.lam / np.abs(wl.lam).max()), S.tensor(np.zeros(3))
    for kind in (P.FWI_REG_TIKHONOV, P.FWI_REG_TV):
        P.fwi_regularization(S.plan, None, kind, 1e-3, f, v[0:1], None)
        torch.cuda.synchronize()
        P.fwi_regularization(S.plan, PER_THREAD, kind, 1e-3, f, v[1:2], None)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            P.fwi_regularization(S.plan, None, kind, 1e-3, f, v[2:3], None)
        graph.replay()
        torch.cuda.synchronize()
        assert float(v[0]) > 0 and v[0] == v[1] == v[2]
    S.close()


def test_one_workgroup_streams():
    """An inner product of 10^6 entries with weights, 24 MB: 0.32 ms in one workgroup of
    1,024 threads, 1.30 ms in one of 256 that waits for each part."""
    torch = _torch()
    from paper_1504_08340_amd import binding as B
    n = 1_000_000
    a, b, w = torch.randn(3, n, dtype=torch.float64, device="cuda")
    o = torch.empty(1, dtype=torch.float64, device="cuda")
    best = 1.0
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(10):
            B.fwi_dot(PER_THREAD, n, a, b, w, o)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 10)
    assert best < 0.6e-3


def test_slots_are_given_back():
    """A program that has used 150 streams gets its next reductions as fast as the first
    (64 slots; one workgroup takes more than 50 times as long), and the same bits."""
    torch = _torch()
    import ctypes
    from paper_1504_08340_amd import binding as B
    n = 4_000_000
    a = torch.randn(n, dtype=torch.float64, device="cuda")
    o = torch.zeros(160, dtype=torch.float64, device="cuda")
    streams = []
    for _ in range(150):
        s = ctypes.c_void_p()
        assert B._lib.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        streams.append(s.value)

    def best(stream, k):
        t = []
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            B.fwi_dot(stream, n, a, a, None, o[k:k + 1])
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    first = best(streams[0], 0)
    for k, s in enumerate(streams):
        B.fwi_dot(s, n, a, a, None, o[k:k + 1])
    torch.cuda.synchronize()
    late = [best(streams[k], k) for k in (149, 0, 70, 149)]
    assert max(late) < 5 * first, (first, late)
    # two at once on streams that share no slot now
    for _ in range(20):
        for k in range(60, 150):
            B.fwi_dot(streams[k], n // 8, a, a, None, o[k:k + 1])
        torch.cuda.synchronize()
        assert bool((o[60:150] == o[60]).all())
    for s in streams:
        assert B._lib.hipStreamDestroy(ctypes.c_void_p(s)) == 0
