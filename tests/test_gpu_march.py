"""The marching correction kernel of the second-order faces at the shapes where
its register windows, segments, block links and boundary codes can go wrong:
one to four rows per lane, one chunk to many segments, last blocks of one
column, plane ranges that differ from block to block, holes, one-cell axes; a
problem on several strips, and one with two wall temperatures on one side, take
the gather kernel. FP64 against the FP64
oracle to 1e-10 relative (sums of a few hundred terms), FP32 sweeps to 1e-4 of
the largest deviation, run twice with equal results.
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4}


def check(bte, p, precision, plan=None, iters=4):
    import torch
    ref = oracle.solve(p, tol=0.0, max_iters=iters, order=2)
    act = p.mask > 0
    runs = []
    for _ in range(2):
        s = bte.Solver(p, precision=precision, plan=plan)
        s.set_order(2)
        T, q, _ = s.solve(torch.tensor(p.Q, device="cuda:0"), tol=0.0, max_iters=iters, check_every=iters)
        runs.append((T.cpu().numpy(), q.cpu().numpy()))
        s.close()
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
    T, q = runs[0]
    eT = np.abs(T - ref["T"])[act].max() / np.abs(ref["T"] - p.T_ref)[act].max()
    rq = ref["q"].reshape(p.ncell, p.dim)
    eq = np.abs(q - rq)[act].max() / np.abs(rq).max()
    assert eT < TOL[precision] and eq < TOL[precision], (eT, eq)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,kind,plan", [
    (9, 5, 1, dict(P=1, NR=1)), (40, 64, 2, dict(P=1, NR=1)), (33, 70, 1, dict(P=1, NR=2)), (1, 9, 1, dict(P=1, NR=2)),
    (70, 131, 1, dict(P=1, NR=4)), (70, 3, 2, dict(P=1, NR=4)), (150, 130, 1, dict(P=1, R=2, NR=1)),
])
def test_march_2d(hip_lib, precision, nx, ny, kind, plan):
    p = bi.random_box_2d(nx, ny, seed=2, n_bands=3, n_theta=2, n_phi=1, hole=nx > 8 and ny > 8, kinds=(0, kind))
    check(hip_lib, p, precision, plan)


def test_march_full_lanes_fp32(hip_lib):
    """All 64 lanes with four rows each, many waves in flight."""
    check(hip_lib, bi.square_2d(256, L=0.3e-6, n_bands=4, n_theta=2, n_phi=2), "fp32", iters=3)


def hot_patch():
    """A square whose left wall has two temperatures (one value per octant and axis does not do)."""
    p = bi.square_2d(30, L=0.1e-6, n_bands=2, n_theta=1, n_phi=1)
    fbc = bi.face_bc_from_mask(p.n, 2, p.mask, lambda i, j, k, f: 1 if (f == 0 and j < 12) else 0)
    return p.replace(face_bc=fbc, bc_kind=np.array([0, 0], dtype=np.int32), bc_T=np.array([300.0, 306.0]))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("make", [
    hot_patch,
    lambda: bi.film_1d(n_cells=1, n_mu=4, Q=np.full(1, 1e18)),
    lambda: bi.film_1d(n_cells=75, n_mu=8, Q=np.linspace(0, 1e18, 75)),
    lambda: bi.random_box_3d(17, 9, 13, seed=1, n_bands=2, n_theta=2, n_phi=1, kinds=(0, 1)),
    lambda: bi.random_box_3d(8, 70, 6, seed=2, n_bands=2, n_theta=1, n_phi=1, kinds=(0, 2)),
    lambda: bi.random_box_3d(5, 5, 40, seed=4, n_bands=2, n_theta=1, n_phi=1, kinds=(0, 1)),
    lambda: bi.staircase_3d(bi.BC_DIFFUSE, nx=33, ny=66, nz=18, n_bands=2, n_theta=1, n_phi=1),
    lambda: bi.finfet_3d_mixed(scale=4, n_bands=2, n_theta=1, n_phi=1),
], ids=["patch", "cell", "film", "box", "wide", "long", "staircase", "finfet"])
def test_march_layouts(hip_lib, precision, make):
    check(hip_lib, make(), precision)
