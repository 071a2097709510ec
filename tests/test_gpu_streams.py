"""Calls of one thread on one plan over two streams.

A misfit returns without waiting; a model check (which every solve makes) on
another stream must not touch what the misfit still needs, nor read its sums.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_misfit_beside_model_checks():
    """Misfits queued on one stream while checks run on another: every J has the
    bits of a J formed alone, and every check those of a check made alone."""
    import torch
    import paper_1504_08340_amd as P
    import workloads as W
    wl = W.tiny(ne_int=(16, 16, 8), nsteps=200, seed=2)      # 18,513 material nodes: 73 partial values a quantity
    S = P.Solver(wl.prob, wl.src_node, wl.src_dir, wl.rec_node)
    rho, lam, mu = (S.tensor(a) for a in (wl.rho, wl.lam, wl.mu))
    g = torch.Generator(device="cuda").manual_seed(1)
    tr, obs = (torch.randn(S.trace_shape, generator=g, dtype=torch.float64, device="cuda") for _ in range(2))
    res = torch.empty_like(tr)
    J = torch.zeros(401, dtype=torch.float64, device="cuda")
    P.fwi_misfit(S.plan, None, tr, obs, res, J[400:])
    alone = P.fwi_check_model(S.plan, None, rho, lam, mu)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for k in range(20):
        for i in range(20 * k, 20 * k + 20):
            P.fwi_misfit(S.plan, a.cuda_stream, tr, obs, res, J[i:i + 1])
        for _ in range(4):                                   # each waits for its own stream only
            assert P.fwi_check_model(S.plan, b.cuda_stream, rho, lam, mu) == alone
    torch.cuda.synchronize()
    assert float(J[400]) > 0 and bool((J == J[400]).all()), int((J != J[400]).sum())
    S.close()
