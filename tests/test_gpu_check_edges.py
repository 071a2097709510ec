"""The model check in one workgroup (up to 4,096 material nodes) and in many."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ne", [(1, 1, 1), (7, 7, 8), (8, 7, 8), (13, 11, 7), (33, 32, 32)])
def test_check_values(ne):
    """27, 3825, 4335, 9315 and 283,075 nodes; minima and maxima placed at the ends, exact but
    for the roots."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1504_08340_amd as P
    import workloads as W
    wl = W.tiny(ne_int=ne, nsteps=2, seed=4)
    S = P.Solver(wl.prob, wl.src_node, wl.src_dir, wl.rec_node)
    rng = np.random.default_rng(1)
    n = wl.lam.size
    for last in (0, n - 1):
        rho, lam, mu = (1.0 + rng.uniform(size=n) for _ in range(3))
        rho[last], mu[last] = 0.5, 0.25
        lam[n - 1 - last] = 9.0
        try:
            info = P.fwi_check_model(S.plan, None, *(S.tensor(a) for a in (rho, lam, mu)))
        except P.FwiError as e:      # the step of the mesh's own model need not fit this one
            assert e.status == -5
            continue
        assert info[:3] == [rho.min(), mu.min(), (3 * lam + 2 * mu).min()]
        assert abs(info[3] - np.sqrt((lam + 2 * mu) / rho).max()) <= 1e-15 * info[3]
    with pytest.raises(P.FwiError) as e:
        mu[n - 1] = -1.0
        P.fwi_check_model(S.plan, None, *(S.tensor(a) for a in (rho, lam, mu)))
    assert e.value.status == -1
    S.close()
