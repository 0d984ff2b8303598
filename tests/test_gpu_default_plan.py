"""The plan of a handle that none was given to: by precision, rows, walls, order
and the number of groups against the CUs; what a plan given in part is completed
from; and the fields of such plans against the oracle (FP64 sums of a few
hundred terms agree to 1e-10 relative, FP32 sweeps to 1e-4 of the largest
deviation).
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4}


def box(nx, ny, nb, nt, kind, hole=False):
    return bi.random_box_2d(nx, ny, seed=2, n_bands=nb, n_theta=nt, n_phi=2, hole=hole, kinds=(0, kind))


def shape(s):
    pl = s.plan()
    return pl["R"], pl["P"], pl["NR"]


@pytest.mark.parametrize("precision,p,want", [
    ("fp64", lambda: box(9, 64, 5, 4, 0), (1, 4, 1)), ("fp64", lambda: box(9, 65, 5, 4, 1), (1, 4, 2)),
    ("fp64", lambda: box(90, 129, 2, 1, 1, True), (2, 2, 2)), ("fp32", lambda: box(150, 256, 2, 1, 1), (2, 2, 2)),
    ("fp64", lambda: box(9, 257, 2, 1, 1), (1, 2, 4)), ("fp64", lambda: box(9, 129, 2, 1, 0), (1, 2, 4)),
    ("fp64", lambda: box(9, 131, 10, 4, 0), (1, 2, 4)), ("fp64", lambda: box(9, 131, 17, 4, 0), (1, 4, 2)), ("fp64", lambda: box(9, 131, 20, 4, 1), (1, 4, 2)),
    ("fp32", lambda: box(9, 131, 20, 4, 1), (1, 4, 4)), ("fp64", lambda: box(9, 131, 2, 1, 1), (1, 2, 4)),
    ("fp64", lambda: box(9, 64, 2, 1, 0), (1, 2, 1)),
    ("fp32", lambda: box(150, 130, 20, 8, 0), (1, 4, 2)), ("fp32", lambda: box(60, 61, 20, 8, 0), (1, 4, 1)),
    ("fp64", lambda: box(20, 130, 20, 8, 0), (1, 4, 1)),
    ("fp32", lambda: bi.random_box_3d(9, 7, 6, seed=1, n_bands=2, n_theta=1, n_phi=1), (1, 4, 1)),
    ("fp64", lambda: bi.random_box_3d(9, 7, 6, seed=1, n_bands=2, n_theta=1, n_phi=1), (1, 4, 1)),
])
def test_default_plan(hip_lib, precision, p, want):
    import torch
    p = p()
    s = hip_lib.Solver(p, precision=precision)
    assert shape(s) == want
    T, q, _ = s.solve(torch.tensor(p.Q, device="cuda:0"), tol=0.0, max_iters=4, check_every=4)
    s.close()
    ref = oracle.solve(p, tol=0.0, max_iters=4)
    act = p.mask > 0
    d = np.abs(ref["T"] - p.T_ref)[act].max()
    rq = ref["q"].reshape(p.ncell, p.dim)
    assert np.abs(T.cpu().numpy() - ref["T"])[act].max() < TOL[precision] * d
    assert np.abs(q.cpu().numpy() - rq)[act].max() < TOL[precision] * np.abs(rq).max()


def test_partial_plan_and_order(hip_lib):
    """A plan given in part keeps the other fields of one strip of four rows
    per lane (two waves per slot would not fit beside four to a plane); the
    order picks its own default, and a plan that was given stays."""
    p = box(90, 140, 2, 1, 1, True)
    s = hip_lib.Solver(p, precision="fp32", plan=dict(P=4))
    assert shape(s) == (1, 4, 4)
    s.set_order(2)
    assert shape(s) == (1, 4, 4)
    s.close()
    s = hip_lib.Solver(p, precision="fp64")
    assert shape(s) == (2, 2, 2)
    s.set_order(2)
    assert shape(s) == (1, 2, 4)
    s.set_order(1)
    assert shape(s) == (2, 2, 2)
    s.close()
