"""The 3D pencil-block layout on grids so narrow that a strip of 8 planes
takes few steps: the values that cross from strip to strip through global
memory are read ahead and have to be there by then. Against the FP64 oracle:
1e-10 of the largest deviation in FP64 (sums of some hundred terms), 1e-4 with
FP32 sweeps.
"""
import numpy as np
import pytest

import bte_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kinds", [(0, 0), (0, 1), (0, 2)])
@pytest.mark.parametrize("n", [(1, 1, 9), (11, 1, 64), (11, 4, 33), (5, 1, 100), (15, 8, 17), (16, 3, 40), (22, 1, 26),
                               (23, 2, 25), (11, 9, 40)])
def test_narrow_grids(hip_lib, precision, kinds, n):
    p = bi.random_box_3d(*n, seed=3, n_bands=3, n_theta=1, n_phi=1, kinds=kinds, hole=False)
    r = oracle.solve(p, tol=0.0, max_iters=5)
    Q = torch.tensor(p.Q, device="cuda")
    for plan in (dict(P=1, C=8), dict(P=4, C=8), dict(G=2, P=2, C=8)):
        if plan.get("G") == 2 and kinds[1] == bi.BC_SPECULAR:
            continue
        s = hip_lib.Solver(p, precision=precision, plan=dict(dict(G=1, NR=-1), **plan))
        T, q, _ = s.solve(Q, tol=0.0, max_iters=5, check_every=5)
        s.close()
        tol = 1e-10 if precision == "fp64" else 1e-4
        rq = r["q"].reshape(p.ncell, 3)
        assert np.abs(T.cpu().numpy() - r["T"]).max() < tol * np.abs(r["T"] - p.T_ref).max(), plan
        assert np.abs(q.cpu().numpy() - rq).max() < tol * np.abs(rq).max(), plan
