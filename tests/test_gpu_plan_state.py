"""A handle's state around plan changes: the order of the cells in the
partial-sum planes, a plan that is rejected, and what a bound workspace holds.
Fields against the FP64 oracle to 1e-10 of the largest deviation (FP64 sums of
a few thousand terms), or equal bit for bit where the same plan runs twice.
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LIMIT = 64 << 20  # the allocation-free solve's array


def narrow():
    """Nine columns: in blocks of 8 columns the planes take 16/9 of the grid
    order's bytes, and only grid order stays within the allocation-free array."""
    return bi.random_box_2d(9, 250, seed=2, n_bands=15, n_theta=8, n_phi=8, hole=False, kinds=(0, 0))


def blocked_plane_bytes(s, p, es):
    """The planes' bytes in blocks of 8 columns (2D, an even number of ordinates per octant and band)."""
    jobs = p.B * (p.M // 2) // s.plan()["P"]
    cells = -(-p.n[0] // 8) * 8 * p.n[1]
    return 3 * jobs * (-(-cells // 256) * 256) * es


def test_rejected_plan_keeps_the_plane_order(hip_lib):
    """Grid order is chosen for this problem; a rejected plan in between must
    not turn it into blocks, neither in the reported bytes nor, in a workspace
    of exactly those bytes, in the arrays."""
    p = narrow()
    s = hip_lib.Solver(p, precision="fp64", plan=dict(G=1, R=1, P=4, NR=2))
    n0, before = s.workspace_bytes(False), s.plan()
    assert n0 <= LIMIT < blocked_plane_bytes(s, p, 8)
    for bad in (dict(P=3), dict(NR=3), dict(R=4, P=4)):
        with pytest.raises(hip_lib.BTEError):
            s.set_plan(**bad)
        assert s.workspace_bytes(False) == n0 and s.plan() == before
    Q = torch.tensor(p.Q, device="cuda")
    T0 = torch.empty(p.ncell, dtype=torch.float64, device="cuda")
    s.solve_noalloc(Q, T0, tol=0.0, max_iters=4, check_every=4)
    r = oracle.solve(p, tol=0.0, max_iters=4)
    act = p.mask > 0
    assert np.abs(T0.cpu().numpy() - r["T"])[act].max() < 1e-10 * np.abs(r["T"] - p.T_ref)[act].max()
    ws = torch.empty(n0, dtype=torch.uint8, device="cuda")
    s.bind_workspace(ws)
    for bad in (dict(P=3), dict(P=1)):  # no such plan; a plan that does not fit
        with pytest.raises(hip_lib.BTEError):
            s.set_plan(**bad)
        assert s.plan() == before
        T, _, _ = s.solve(Q, tol=0.0, max_iters=4, check_every=4)
        assert torch.equal(T, T0)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("axes", [((0, 0, 1),), ((1, 0, 0), (0, 0, 1)), ((0, 1, 0),)], ids=["z", "xz", "y"])
def test_few_octants_stay_in_the_workspace(hip_lib, precision, axes):
    """Directions along the axes leave octants without ordinates, so that the
    planes are smaller than the tables made in them: in a workspace of exactly
    the reported bytes nothing behind it is written."""
    p = bi.square_2d(70, L=0.2e-6, n_bands=1, n_theta=1, n_phi=1)
    s = np.array([np.array(a, dtype=float) * g for a in axes for g in (1, -1)])
    p = p.replace(s=s, w=np.full(len(s), 4 * np.pi / len(s)))
    h = hip_lib.Solver(p, precision=precision)
    n = h.workspace_bytes(False)
    ws = torch.full((n + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
    h.bind_workspace(ws[:n])
    T, _, _ = h.solve(torch.tensor(p.Q, device="cuda"), tol=0.0, max_iters=4, check_every=4)
    assert (ws[n:] == 0xA5).all()
    h.close()
    r = oracle.solve(p, tol=0.0, max_iters=4)
    tol = 1e-10 if precision == "fp64" else 1e-4
    assert np.abs(T.cpu().numpy() - r["T"]).max() < tol * np.abs(r["T"] - p.T_ref).max()


def porous(nx, ny, nz, **kw):
    """One cell in ten missing at random: up to 256 inflow entries a chunk."""
    p = bi.random_box_3d(nx, ny, nz, seed=1, hole=False, kinds=(0, 1), **(kw or dict(n_bands=2, n_theta=2, n_phi=2)))
    mask = (np.random.default_rng(5).random(p.ncell) < 0.9).astype(np.uint8)
    fbc = bi.face_bc_from_mask(p.n, 3, mask, lambda i, j, k, f: 0 if f == 4 else 1)
    return p.replace(mask=mask, face_bc=fbc, Q=p.Q * mask)


@pytest.mark.parametrize("make,plan", [
    (lambda: bi.random_box_2d(16, 131, seed=2, n_bands=3, n_theta=2, n_phi=2, kinds=(0, 1)), dict(P=4, NR=4)),
    (lambda: bi.random_box_2d(23, 259, seed=3, n_bands=2, n_theta=2, n_phi=1, kinds=(0, 2)), dict(P=4, NR=4)),
    (lambda: bi.random_box_2d(2001, 70, seed=2, n_bands=2, n_theta=2, n_phi=1, hole=False, kinds=(0, 1)),
     dict(P=4, NR=2)),
    (lambda: porous(24, 64, 8), dict(P=8, NR=1)),
], ids=["rows4", "strips", "wide", "porous"])
def test_plans_within_the_lds_run(hip_lib, make, plan):
    """FP64 plans that one staged plane (double-buffered) leaves room for and
    three or four would not: fields of both face orders against the oracle,
    gradients against two waves per workgroup (both sum the same FP64 terms in
    another order, iterated to 1e-12)."""
    p = make()
    Q = torch.tensor(p.Q, device="cuda")
    act = p.mask > 0
    s = hip_lib.Solver(p, precision="fp64", plan=dict(G=1, R=1, **plan))
    assert {k: s.plan()[k] for k in plan} == plan
    for order in (1, 2):
        s.set_order(order)
        T, q, _ = s.solve(Q, tol=0.0, max_iters=4, check_every=4)
        r = oracle.solve(p, tol=0.0, max_iters=4, order=order)
        rq = r["q"].reshape(p.ncell, p.dim)
        assert np.abs(T.cpu().numpy() - r["T"])[act].max() < 1e-10 * np.abs(r["T"] - p.T_ref)[act].max()
        assert np.abs(q.cpu().numpy() - rq)[act].max() < 1e-10 * np.abs(rq).max()
    s.close()
    g = torch.tensor(np.cos(np.arange(p.ncell)) * p.mask, device="cuda")
    out = []
    for pl in (plan, dict(P=2, NR=1)):
        s = hip_lib.Solver(p, precision="fp64", plan=dict(G=1, R=1, **pl))
        s.solve(Q, tol=1e-12, store_state=True)
        dtau, dQ, _ = s.adjoint(g, tol=1e-12)
        s.close()
        out.append((dtau, dQ.cpu().numpy()))
    for a, b in zip(*out):
        assert np.abs(a - b).max() < 1e-9 * np.abs(b).max()


def test_refused_default_keeps_its_schedules(hip_lib):
    """FP64 with two rows per lane and many groups: the default plan's eight
    waves are refused after its schedules are made, and the plan that follows
    takes them over. Creating the handle then takes about as long as in FP32,
    whose first plan holds (twice as long if the schedules were made again)."""
    import time
    p = bi.random_box_3d(40, 100, 40, seed=1, n_bands=9, n_theta=4, n_phi=4)
    best = {}
    for _ in range(3):
        for precision in ("fp32", "fp64"):
            t = time.perf_counter()
            s = hip_lib.Solver(p, precision=precision)
            t = time.perf_counter() - t
            best[precision] = min(t, best.get(precision, t))
            plan = s.plan()
            s.close()
    assert (plan["P"], plan["NR"]) == (4, 2)
    assert best["fp64"] < 1.6 * best["fp32"], best


def section():
    return bi.random_box_2d(61, 100, seed=2, n_bands=15, n_theta=4, n_phi=2, kinds=(0, 1))


def tuned(hip_lib, p, path, plan):
    """A plan cache whose line for p holds `plan`."""
    s = hip_lib.Solver(p, precision="fp64")
    s.solve(torch.tensor(p.Q, device="cuda"), tol=0.0, max_iters=1, autotune_cache=path)
    s.close()
    key = open(path).read().split(" plan ")[0]
    open(path, "w").write(key + " plan " + " ".join(str(plan[k]) for k in ("G", "R", "P", "C", "NR")) + "\n")


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("how", ["G", "P", "cache"])
def test_workspace_holds_the_plan_partial_ones_start_from(hip_lib, tmp_path, how, adjoint):
    """The default plan of an FP64 section shares its planes among four waves,
    a plan given in part among two: a workspace of exactly the reported bytes
    takes both, and a plan cache that holds the latter."""
    p = section()
    Q = torch.tensor(p.Q, device="cuda")
    base = dict(G=1, R=1, P=2, C=8, NR=2)
    opt = dict(tol=0.0, max_iters=4, check_every=4, store_state=adjoint)
    s = hip_lib.Solver(p, precision="fp64")
    assert s.plan() == dict(base, P=4)
    s.bind_workspace(torch.empty(s.workspace_bytes(adjoint), dtype=torch.uint8, device="cuda"))
    s.solve(Q, **opt)
    if how == "cache":
        opt["autotune_cache"] = str(tmp_path / "plans")
        tuned(hip_lib, p, opt["autotune_cache"], base)
    else:
        s.set_plan(**{how: base[how]})
        assert s.plan() == base
    T, q, _ = s.solve(Q, **opt)
    assert s.plan() == base
    n = s.workspace_bytes(adjoint)
    s.close()
    r = oracle.solve(p, tol=0.0, max_iters=4)
    act = p.mask > 0
    assert np.abs(T.cpu().numpy() - r["T"])[act].max() < 1e-10 * np.abs(r["T"] - p.T_ref)[act].max()
    # a plan that was given reports its own bytes
    s = hip_lib.Solver(p, precision="fp64", plan=dict(P=2))
    assert s.workspace_bytes(adjoint) == n
    s.set_plan(P=4)
    assert s.workspace_bytes(adjoint) < n
    s.close()
