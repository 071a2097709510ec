"""The stage's element launch at the edges of its tiles, against the oracle.

Tiles hold 5x4x2 bricks: meshes of one brick, of exactly one tile, of one brick
more, and of PML layers thinner and thicker than a tile, so that every part
(interior, gradient, S-rows, u-rows) meets full and ragged tiles along each
axis.  Bounds: FP64 a few hundred roundings (1e-13 for one operator
application, 1e-9 for a gradient of a few steps); FP32 1e-4 for gradients.
"""
import numpy as np
import pytest

import workloads as W
from helpers import nodal_from_state, rel_l2, state_from_nodal

pytestmark = pytest.mark.gpu

MESHES = [((1, 1, 1), 1, 1), ((5, 4, 2), 1, 2), ((6, 5, 3), 2, 3), ((4, 9, 1), 5, 1), ((11, 3, 5), 3, 5)]


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1504_08340_amd as pkg
    return pkg


@pytest.mark.parametrize("ne,ps,pb", MESHES)
def test_operator_and_gradient_at_tile_edges(P, ne, ps, pb):
    from oracle.assemble import System
    from oracle.solve import Stepper
    wl = W.tiny(ne_int=ne, npml_side=ps, npml_bottom=pb, nsteps=8, nsrc=2, seed=11)
    s = System(wl.prob, wl.rho, wl.lam, wl.mu)
    rng = np.random.default_rng(2)
    x1, x2 = rng.standard_normal(s.n_state), rng.standard_normal(s.n_state)
    h = rng.standard_normal(s.n_hist)
    x0 = np.zeros(s.n_state)
    x0[s.hist] = h
    S = P.Solver(wl.prob, wl.src_node, wl.src_dir, wl.rec_node)
    m = [S.tensor(a) for a in (wl.rho, wl.lam, wl.mu, wl.wavelet)]
    X = [S.tensor(np.repeat(nodal_from_state(s, v)[None], wl.nsrc, 0)) for v in (x0, x1, x2)]
    ghat = np.zeros(s.n_state)
    ghat[s.hist] = s.G[s.hist, :].T @ h
    for which, ref in ((0, s.Minv * -(s.G @ h + s.K @ x1 + s.C @ x2)),
                       (1, s.Minv * -(ghat + s.K.T @ x1 + s.C.T @ x2))):
        out = S.apply_operator(which, *m[:3], *X).cpu().numpy()
        for k in range(wl.nsrc):
            assert np.abs(state_from_nodal(s, out[k]) - ref).max() <= 1e-13 * np.abs(ref).max()
    for full in (False, True):
        st = Stepper(s, wl.src_node, wl.src_dir, wl.rec_node, full_gradient=full)
        tr, states = st.forward(wl.wavelet, store=True)
        gl_o, gm_o, _ = st.adjoint_gradient(wl.wavelet, 0.5 * tr, states)
        for precision, tol in ((P.FWI_FP64, 1e-9), (P.FWI_FP32, 1e-4)):
            T = P.Solver(wl.prob, wl.src_node, wl.src_dir, wl.rec_node, precision=precision, grad_full=full)
            got = T.forward(*m)
            _, res = T.misfit(got, T.tensor(0.5 * tr))
            gl, gm = T.adjoint_gradient(*m, res)
            assert rel_l2(gl.cpu().numpy(), gl_o) <= tol
            assert rel_l2(gm.cpu().numpy(), gm_o) <= tol
            T.close()
    S.close()


# Tiles of 5x4x2 bricks: 8, 180 and 648 of them, so that the sources' gradient
# terms are summed in three groups, in two (of two sources and one), and in one.
@pytest.mark.parametrize("ne,full", [((6, 5, 3), True), ((30, 24, 10), False), ((40, 36, 18), False)])
def test_gradient_of_several_sources_is_the_sum_of_each(P, ne, full):
    """FP64, a few steps: other orders of the same sums, 1e-12."""
    wl = W.tiny(ne_int=ne, npml_side=1, npml_bottom=1, nsteps=3, nsrc=3, seed=5)
    want = None
    for k in (slice(0, 1), slice(1, 2), slice(2, 3), slice(0, 3)):
        T = P.Solver(wl.prob, wl.src_node[k], wl.src_dir[k], wl.rec_node, grad_full=full)
        m = [T.tensor(a) for a in (wl.rho, wl.lam, wl.mu, wl.wavelet[k])]
        tr = T.forward(*m)
        _, res = T.misfit(tr, 0.5 * tr)
        g = [x.cpu().numpy() for x in T.adjoint_gradient(*m, res)]
        T.close()
        if k == slice(0, 3):
            assert all(np.abs(a).max() > 0 and rel_l2(a, b) <= 1e-12 for a, b in zip(g, want))
        else:
            want = g if want is None else [a + b for a, b in zip(want, g)]


@pytest.mark.parametrize("nrec", [1, 127, 128, 129, 169])
def test_traces_do_not_depend_on_the_number_of_receivers(P, nrec):
    """Receivers are recorded by workgroups of 128 of the next step's first launch, the
    last step's by a launch of its own: every step's traces against a solver that
    holds the receivers in another order, bit for bit."""
    wl = W.tiny(ne_int=(6, 6, 2), npml_side=1, npml_bottom=1, nsteps=5, nsrc=2, seed=3)
    assert len(wl.rec_node) == 169
    order = np.random.default_rng(nrec).permutation(169)
    for precision in (P.FWI_FP64, P.FWI_FP32):
        got = []
        for rec in (wl.rec_node[:nrec], wl.rec_node[order]):
            S = P.Solver(wl.prob, wl.src_node, wl.src_dir, np.ascontiguousarray(rec), precision=precision)
            got.append(S.forward(*(S.tensor(a) for a in (wl.rho, wl.lam, wl.mu, wl.wavelet))).cpu().numpy())
            S.close()
        back = np.argsort(order)[:nrec]
        assert got[0].shape == (2, 6, nrec, 3) and np.array_equal(got[0], got[1][:, :, back])
        assert all(np.abs(got[1][:, k]).max() > 0 for k in range(1, 6))
