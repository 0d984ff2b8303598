"""Partial-sum planes: the sums of every plane (temperature, heat flux, dJ/dQ)
formed from one staged plane, over the waves-per-workgroup counts, and the
blocked order of the cells, at sizes around its blocks of 8 columns and whole
lanes of rows: the fields and the gradient against the FP64 oracle. FP64 sums
of a few hundred terms agree to 1e-10 relative, FP32 sweeps to 1e-4 of the
largest deviation.
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4}


def check(bte, p, precision, plan, iters=4):
    import torch
    try:
        s = bte.Solver(p, precision=precision, plan=plan)
    except bte.BTEError as e:
        if "LDS" not in str(e):
            raise
        pytest.skip("the shape's staging exceeds the workgroup's LDS")
    T, q, _ = s.solve(torch.tensor(p.Q, device="cuda:0"), tol=0.0, max_iters=iters, check_every=iters)
    got = s.plan()
    s.close()
    ref = oracle.solve(p, tol=0.0, max_iters=iters)
    act = p.mask > 0
    # (the deviation can vanish: one cell between walls at T_ref +- 1 K)
    scale = max(np.abs(ref["T"] - p.T_ref)[act].max(), np.abs(p.bc_T[p.bc_kind == bi.BC_ISOTHERMAL] - p.T_ref).max())
    eT = np.abs(T.cpu().numpy() - ref["T"])[act].max() / scale
    rq = ref["q"].reshape(p.ncell, p.dim)
    eq = np.abs(q.cpu().numpy() - rq)[act].max() / np.abs(rq).max()
    assert eT < TOL[precision] and eq < TOL[precision], (got, eT, eq)
    assert not T.cpu().numpy()[~act].any()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,plan", [
    (8, 4, dict(P=1, NR=1)), (9, 5, dict(P=2, NR=2)), (7, 3, dict(P=4, NR=4)), (16, 131, dict(P=4, NR=4)),
    (33, 130, dict(P=2, R=2, NR=1)), (23, 259, dict(P=1, R=2, NR=2)), (1, 6, dict(P=4, NR=4)),
    (15, 9, dict(G=2, P=2, NR=4)),
])
def test_planes_2d(hip_lib, precision, nx, ny, plan):
    check(hip_lib, bi.random_box_2d(nx, ny, seed=2, n_bands=3, n_theta=2, n_phi=2, hole=nx > 8), precision, plan)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 65])
def test_planes_1d(hip_lib, precision, n):
    check(hip_lib, bi.film_1d(n_cells=n, n_mu=6, Q=np.linspace(0.0, 1e18, n)), precision, dict(P=2))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("P", [1, 2, 4, 8])
@pytest.mark.parametrize("n,kind", [((11, 9, 13), 1), ((8, 70, 6), 2), ((17, 5, 4), 1)])
def test_planes_3d(hip_lib, precision, P, n, kind):
    p = bi.random_box_3d(*n, seed=1, n_bands=3, n_theta=2, n_phi=2, kinds=(0, kind))
    check(hip_lib, p, precision, dict(P=P, NR=1))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,NR,P,kind", [((1, 9, 8), 1, 8, 1), ((9, 1, 17), 2, 4, 1), ((17, 16, 1), 2, 2, 2),
                                         ((100, 9, 7), 2, 8, 1), ((7, 126, 3), 2, 1, 1), ((64, 65, 2), 2, 4, 2)])
def test_period_indices_3d(hip_lib, precision, n, NR, P, kind):
    """Plane indices formed from the period table, and chunks whose boundary
    entries fill no, one or several rows of 64: thin boxes (one period of a
    block, blocks of one column), lanes of one and two rows, axes of each role
    run both ways."""
    p = bi.random_box_3d(*n, seed=4, n_bands=2, n_theta=2, n_phi=1, kinds=(0, kind))
    check(hip_lib, p, precision, dict(P=P, NR=NR))


@pytest.mark.parametrize("make", [lambda: bi.square_2d(19, L=0.1e-6, n_bands=3, n_theta=2, n_phi=2),
                                  lambda: bi.random_box_2d(13, 9, seed=3, n_bands=2, n_theta=1, n_phi=1),
                                  lambda: bi.random_box_3d(9, 5, 6, seed=5, n_bands=2, n_theta=1, n_phi=1)],
                         ids=["square", "masked", "box"])
def test_gradient_across_plane_orders(hip_lib, make):
    """dJ/dQ (the second plane) and dJ/dtau (the stored field, kept in the
    planes' order) against central differences of the FP64 oracle."""
    import torch
    p = make()
    g = np.cos(np.arange(p.ncell)) * p.mask
    s = hip_lib.Solver(p, precision="fp64")
    s.solve(torch.tensor(p.Q, device="cuda:0"), tol=1e-13, store_state=True)
    dtau, dQ, _ = s.adjoint(torch.tensor(g, device="cuda:0"), tol=1e-13)
    s.close()

    def J(q):
        return float((g * oracle.solve(q, tol=1e-14, max_iters=4000)["T"]).sum())

    e = 1e-4
    for b in range(p.B):
        t = [p.tau.copy(), p.tau.copy()]
        t[0][b] *= 1 + e
        t[1][b] *= 1 - e
        fd = (J(p.replace(tau=t[0])) - J(p.replace(tau=t[1]))) / (2 * e * p.tau[b])
        assert abs(fd - dtau[b]) < 1e-5 * np.abs(dtau * p.tau).max() / p.tau[b], (b, fd, dtau[b])
    dq = dQ.cpu().numpy()
    for c in np.flatnonzero(p.mask)[[0, p.n_active // 2, -1]]:
        h = 1e-3 * np.abs(p.Q).max()
        qs = [p.Q.copy(), p.Q.copy()]
        qs[0][c] += h
        qs[1][c] -= h
        fd = (J(p.replace(Q=qs[0])) - J(p.replace(Q=qs[1]))) / (2 * h)
        assert abs(fd - dq[c]) < 1e-5 * np.abs(dq).max(), (c, fd, dq[c])


@pytest.mark.parametrize("n", [(6, 5, 7), (48, 40, 36)])
def test_specular_update_bands(hip_lib, n):
    """The specular walls' update with a thread per band (few faces) and with
    all bands in a thread (512 workgroups of faces and ordinates and more)."""
    p = bi.random_box_3d(*n, seed=1, n_bands=3, n_theta=2, n_phi=2, kinds=(0, bi.BC_SPECULAR))
    check(hip_lib, p, "fp64", dict(P=4, NR=1))
