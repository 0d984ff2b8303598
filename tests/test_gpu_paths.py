"""Which alternative a handle runs, and the grid order of the partial-sum
planes, which problems take whose padding to blocks of 8 columns alone would
push them past the allocation-free solve's array: odd sizes, every octant, rows
past the grid, one and two rows per lane in 3D, films and strips. Fields against
the FP64 oracle to 1e-10 of the largest deviation (FP64 sums of some thousand
terms; FP32 sweeps 1e-4), gradients against the same problem with its planes in
blocks (1e-9: the same FP64 terms summed in another order, iterated to 1e-12).
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {"fp64": 1e-10, "fp32": 1e-4}


def film(n, n_mu=8, bands=1):
    v, tau, C = bi.band_table_synthetic(bands)
    return bi.film_1d(n_cells=n, n_mu=n_mu, Q=np.linspace(0.0, 1e18, n)).replace(v=v, tau=tau, C=C)


def grid_order(make, ks):
    """The first of make(k)'s handles whose planes are in grid order."""
    for k in ks:
        s = make(k)
        if "plane_blocks" not in s.paths():
            assert s.workspace_bytes(False) <= 64 << 20
            return s
        s.close()
    raise AssertionError("no size takes grid order")


def check(p, T, q, precision, iters):
    r = oracle.solve(p, tol=0.0, max_iters=iters)
    act = p.mask > 0
    scale = max(np.abs(r["T"] - p.T_ref)[act].max(), 1.0 if p.dim == 1 else 0.0)  # film walls: T_ref +- 1 K
    assert np.abs(T.cpu().numpy() - r["T"])[act].max() < TOL[precision] * scale
    rq = r["q"].reshape(p.ncell, p.dim)
    assert np.abs(q.cpu().numpy() - rq)[act].max() < TOL[precision] * np.abs(rq).max()
    assert not T.cpu().numpy()[~act].any()


@pytest.mark.parametrize("precision,make,plan", [
    ("fp64", lambda k: bi.random_box_2d(9, 37, seed=2, n_bands=k, n_theta=6, n_phi=6, kinds=(0, 1)), dict(NR=2)),
    ("fp32", lambda k: bi.random_box_2d(9, 37, seed=2, n_bands=2 * k, n_theta=6, n_phi=6, kinds=(0, 1)), dict(NR=4)),
    ("fp64", lambda k: bi.random_box_2d(9, 131, seed=3, n_bands=k, n_theta=4, n_phi=4, kinds=(0, 2)),
     dict(NR=1, R=2)),
    ("fp64", lambda k: bi.random_box_3d(9, 11, 13, seed=1, n_bands=k, n_theta=4, n_phi=2, kinds=(0, 1)), dict(NR=1)),
    ("fp64", lambda k: bi.random_box_3d(11, 9, 13, seed=1, n_bands=k, n_theta=4, n_phi=2, kinds=(0, 2)), dict(NR=2)),
    ("fp32", lambda k: bi.random_box_3d(9, 11, 17, seed=1, n_bands=2 * k, n_theta=4, n_phi=2, kinds=(0, 1)),
     dict(NR=2)),
    ("fp64", lambda k: film(9, n_mu=60 + 2 * k, bands=200), dict(G=2)),
], ids=["rows2", "rows4_f32", "strips", "box", "box_rows2", "box_rows2_f32", "film"])
def test_grid_order(hip_lib, precision, make, plan):
    plan = dict(dict(G=1, R=1, P=1), **plan)
    s = grid_order(lambda k: hip_lib.Solver(make(k), precision=precision, plan=plan), range(1, 80))
    p = s.problem
    Q = torch.tensor(p.Q, device="cuda")
    T, q, _ = s.solve(Q, tol=0.0, max_iters=4, check_every=4)
    check(p, T, q, precision, 4)
    if precision == "fp64":
        g = torch.tensor(np.cos(np.arange(p.ncell)) * p.mask, device="cuda")
        out = []
        for pl in (None, dict(plan, P=4, R=1)):
            if pl:
                s.set_plan(**pl)
                assert "plane_blocks" in s.paths()
            s.solve(Q, tol=1e-12, store_state=True)
            dtau, dQ, _ = s.adjoint(g, tol=1e-12)
            out.append((dtau, dQ.cpu().numpy()))
        for a, b in zip(*out):
            assert np.abs(a - b).max() < 1e-9 * np.abs(b).max()
    s.close()


def test_grid_order_of_films(hip_lib):
    """A batch of films, which one launch iterates, in grid order."""
    def make(k):
        return hip_lib.BatchSolver([film(9 + 8 * (i % 4), n_mu=20 + k, bands=25) for i in range(40)], precision="fp64",
                                   plan=dict(G=1, P=4))
    s = grid_order(make, range(46))
    assert s.paths() == {"film"}
    Ts, qs, _ = s.solve([torch.tensor(p.Q, device="cuda") for p in s.problems], tol=0.0, max_iters=6, check_every=3)
    s.close()
    for p, T, q in zip(s.problems, Ts, qs):
        check(p, T, q, "fp64", 6)


@pytest.mark.parametrize("n,n_mu,precision,count,want", [
    (20, 64, "fp32", 1, True), (20, 100, "fp32", 1, False), (20, 100, "fp64", 1, True), (20, 100, "fp32", 2, True),
    (130, 100, "fp32", 1, False), (256, 90, "fp32", 1, True), (500, 76, "fp32", 1, True),
])
def test_single_film_of_many_groups(hip_lib, n, n_mu, precision, count, want):
    """One workgroup sweeps a film, in double: a single FP32 film with many
    groups and few cells takes the general kernels."""
    ps = [film(n, n_mu=n_mu, bands=15)] * count
    s = hip_lib.BatchSolver(ps, precision=precision)
    assert ("film" in s.paths()) == want
    Ts, qs, _ = s.solve([torch.tensor(p.Q, device="cuda") for p in ps], tol=0.0, max_iters=5, check_every=3)
    s.close()
    for p, T, q in zip(ps, Ts, qs):
        check(p, T, q, precision, 5)


@pytest.mark.parametrize("make,plan,order,want", [
    (lambda: film(200), None, 1, True), (lambda: film(1024), None, 1, True), (lambda: film(1025), None, 1, False),
    (lambda: film(200), dict(G=2), 1, False), (lambda: film(200), None, 2, False),
    (lambda: film(20, n_mu=100, bands=16), None, 1, True), (lambda: film(20, n_mu=100, bands=18), None, 1, False),
])
def test_film_path(hip_lib, make, plan, order, want):
    s = hip_lib.Solver(make(), precision="fp64", plan=plan)
    s.set_order(order)
    assert ("film" in s.paths()) == want
    s.close()


def two_wall_temperatures():
    p = bi.square_2d(30, L=0.1e-6, n_bands=2, n_theta=1, n_phi=1)
    fbc = bi.face_bc_from_mask(p.n, 2, p.mask, lambda i, j, k, f: 1 if (f == 0 and j < 12) else 0)
    return p.replace(face_bc=fbc, bc_kind=np.array([0, 0], dtype=np.int32), bc_T=np.array([300.0, 306.0]))


@pytest.mark.parametrize("make,plan,want", [
    (lambda: bi.random_box_2d(9, 5, seed=2, n_bands=3, n_theta=2, n_phi=1), dict(P=1, NR=1), True),
    (lambda: bi.random_box_2d(70, 131, seed=2, n_bands=3, n_theta=2, n_phi=1), dict(P=1, NR=4), True),
    (lambda: bi.random_box_2d(150, 130, seed=2, n_bands=3, n_theta=2, n_phi=1), dict(P=1, R=2, NR=1), False),
    (lambda: bi.square_2d(256, L=0.3e-6, n_bands=4, n_theta=2, n_phi=2), None, True),
    (two_wall_temperatures, None, False),
    (lambda: film(75), None, True),
    (lambda: bi.random_box_3d(17, 9, 13, seed=1, n_bands=2, n_theta=2, n_phi=1), None, True),
    (lambda: bi.random_box_3d(8, 70, 6, seed=2, n_bands=2, n_theta=1, n_phi=1, kinds=(0, 2)), None, True),
    (lambda: bi.staircase_3d(bi.BC_DIFFUSE, nx=33, ny=66, nz=18, n_bands=2, n_theta=1, n_phi=1), None, True),
    (lambda: bi.finfet_3d_mixed(scale=4, n_bands=2, n_theta=1, n_phi=1), None, True),
])
def test_correction_path(hip_lib, make, plan, want):
    s = hip_lib.Solver(make(), precision="fp64", plan=plan)
    assert "corr_march" not in s.paths()
    s.set_order(2)
    assert ("corr_march" in s.paths()) == want
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kinds", [(0, 0), (0, 1), (0, 2)])
def test_time_sweep_of_a_film(hip_lib, precision, kinds):
    """The time reported is that of the kernel the solve runs (the general sweep
    takes five times as long), and timing changes nothing: neither the state a
    gradient starts from nor the output of an earlier solve."""
    p = film(200, n_mu=32).replace(bc_kind=np.array(kinds, dtype=np.int32))
    Q = torch.tensor(p.Q, device="cuda")
    g = torch.tensor(np.cos(np.arange(p.ncell)), device="cuda")
    out = []
    for timed in (False, True):
        s = hip_lib.Solver(p, precision=precision)
        T, q, rep = s.solve(Q, tol=0.0, max_iters=800, store_state=True)
        Tc, qc = T.clone(), q.clone()
        if timed:
            T.zero_(), q.zero_()
            ms, updates = s.time_sweep(200)
            assert updates == p.ncell * p.M * p.B
            assert 800 * ms * 1e-3 < 1.5 * rep["seconds"], (ms, rep)
            assert not T.any() and not q.any()
            T2, q2, _ = s.solve(Q, T_init=Tc, tol=0.0, max_iters=8, store_state=True)
        else:
            T2, q2, _ = s.solve(Q, T_init=Tc, tol=0.0, max_iters=8, store_state=True)
        if timed:
            s.time_sweep(7)
        dtau, dQ, _ = s.adjoint(g, tol=0.0, max_iters=16)
        assert ("film_chunk" in s.sweep_kernel_name())
        s.close()
        out.append([x.cpu().numpy() for x in (Tc, qc, T2, q2, dQ)] + [dtau])
    assert all(np.array_equal(a, b) for a, b in zip(*out))


def test_specular_update_of_many_bands(hip_lib):
    """More bands than the second dimension of a grid takes workgroups."""
    p = film(4, n_mu=2, bands=66001).replace(bc_kind=np.array([0, 2], dtype=np.int32))
    s = hip_lib.Solver(p, precision="fp64")
    assert "film" not in s.paths()
    T, q, _ = s.solve(torch.tensor(p.Q, device="cuda"), tol=0.0, max_iters=4, check_every=4)
    s.close()
    check(p, T, q, "fp64", 4)
