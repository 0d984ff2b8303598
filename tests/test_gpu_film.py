"""1D films swept in one launch per chunk: the lengths at which the cells per
lane change, one cell, unequal octants (odd numbers of directions), every wall
kind at either end, chunks of one to many iterations, batches of films and the
adjoint. Fixed iteration counts against the FP64 oracle (1e-10 relative in FP64:
sums of at most a few hundred terms; 1e-4 of the largest difference with FP32
sweeps), and against plans with two ordinates per lane, which take the general
sweep kernel (1e-11: both sum the same FP64 terms in another order).
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4}


def film(n, n_mu=8, bands=1, kinds=(0, 0)):
    p = bi.film_1d(n_cells=n, n_mu=n_mu, Q=1e17 * (1.0 + np.cos(np.arange(n))))
    if bands > 1:
        v, tau, C = bi.band_table_synthetic(bands)
        p = p.replace(v=v, tau=tau, C=C)
    return p.replace(bc_kind=np.array(kinds, dtype=np.int32))


def solve(bte, p, precision, iters, check_every, plan=None):
    import torch
    s = bte.Solver(p, precision=precision, plan=plan)
    T, q, rep = s.solve(torch.tensor(p.Q, device="cuda:0"), tol=0.0, max_iters=iters, check_every=check_every)
    s.close()
    return T.cpu().numpy(), q.cpu().numpy(), rep


def close(p, got, ref, tol):
    scale = max(np.abs(ref[0] - p.T_ref).max(), 1.0)  # the walls differ from T_ref by 1 K
    assert np.abs(got[0] - ref[0]).max() < tol * scale
    assert np.abs(got[1] - ref[1].reshape(got[1].shape)).max() < tol * np.abs(ref[1]).max()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 800, 1024, 1025])
def test_lengths(hip_lib, precision, n):
    p = film(n)
    r = oracle.solve(p, tol=0.0, max_iters=5)
    close(p, solve(hip_lib, p, precision, 5, 3), (r["T"], r["q"]), TOL[precision])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kinds", [(0, 1), (1, 0), (0, 2), (2, 0)])
@pytest.mark.parametrize("n,bands,n_mu", [(1, 1, 4), (37, 3, 6), (150, 15, 32), (600, 4, 64)])
def test_walls(hip_lib, precision, kinds, n, bands, n_mu):
    p = film(n, n_mu=n_mu, bands=bands, kinds=kinds)
    r = oracle.solve(p, tol=0.0, max_iters=7)
    close(p, solve(hip_lib, p, precision, 7, 4), (r["T"], r["q"]), TOL[precision])


@pytest.mark.parametrize("check_every", [1, 2, 3, 8])
@pytest.mark.parametrize("n_mu,bands", [(7, 1), (5, 3)])
def test_general_path_and_chunks(hip_lib, check_every, n_mu, bands):
    """Odd n_mu: the octants differ in ordinates; residuals included."""
    p = film(70, n_mu=n_mu, bands=bands)
    a = solve(hip_lib, p, "fp64", 9, check_every)
    b = solve(hip_lib, p, "fp64", 9, check_every, plan=dict(G=2))
    close(p, a, b, 1e-11)
    assert a[2]["iters"] == b[2]["iters"] == 9
    assert a[2]["eps_T"] == pytest.approx(b[2]["eps_T"], rel=1e-8)
    assert a[2]["eps_q"] == pytest.approx(b[2]["eps_q"], rel=1e-8)


@pytest.mark.parametrize("kinds", [(0, 0), (0, 1), (0, 2)])
@pytest.mark.parametrize("n", [5, 100, 300])
def test_adjoint_general_path(hip_lib, kinds, n):
    """The adjoint iteration (with reflecting walls: after a forward solve here,
    itself on the general path), its gradients and the warm start of a second
    solve. Specular walls need G = 1, so they are checked against P = 1."""
    import torch
    p = film(n, n_mu=6, bands=2, kinds=kinds)
    Q = torch.tensor(p.Q, device="cuda:0")
    g = torch.tensor(np.sin(np.arange(n)), device="cuda:0")
    out = []
    for plan in (None, dict(P=1) if kinds[1] == 2 else dict(G=2)):
        s = hip_lib.Solver(p, precision="fp64", plan=plan)
        T, q, _ = s.solve(Q, tol=1e-12, store_state=True)
        dtau, dQ, _ = s.adjoint(g, tol=1e-12)
        ds = s.adjoint_dscale()
        # (a warm start: the reflecting walls begin at the adjacent cell's equilibrium again)
        T2, _, _ = s.solve(Q, T_init=T, tol=0.0, max_iters=8)
        out.append((T.cpu().numpy(), dQ.cpu().numpy(), dtau, ds, T2.cpu().numpy()))
        s.close()
    for a, b in zip(*out):
        assert np.abs(np.asarray(a) - b).max() <= 1e-9 * np.abs(b).max()


def test_batch_of_films(hip_lib):
    import torch
    ps = [film(n, bands=3, kinds=k) for n, k in [(9, (0, 0)), (200, (0, 1)), (64, (1, 0)), (513, (0, 0))]]
    b = hip_lib.BatchSolver(ps, precision="fp64")
    Ts, qs, _ = b.solve([torch.tensor(p.Q, device="cuda:0") for p in ps], tol=0.0, max_iters=6, check_every=3)
    b.close()
    for p, T, q in zip(ps, Ts, qs):
        r = oracle.solve(p, tol=0.0, max_iters=6)
        close(p, (T.cpu().numpy(), q.cpu().numpy()), (r["T"], r["q"]), 1e-10)
