"""GMRES on a right-hand side, start vector or matrix that is not finite ends with
the first cycle instead of spending the budget on cycles that stop at once."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [50, 20_000])
@pytest.mark.parametrize("where", ["b", "x0", "A"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_ends_early(n, mixed, where, value):
    import torch
    import paper_2411_10143_amd as ck
    A = M.convection_diffusion_2d(int(n ** 0.5), 10.0)
    b, x0 = M.vector(A.n, 1), np.zeros(A.n)
    if where == "b":
        b[A.n // 2] = value
    elif where == "x0":
        x0[A.n // 3] = value
    else:
        A.val[len(A.val) // 2] = value
    say(f"gmres not finite n={A.n} mixed={mixed} {where}={value}")
    Mx = ck.Matrix.from_csr(A, keep_fp32=True)
    x = torch.from_numpy(x0).cuda()
    r = ck.gmres_solve(Mx.handle, torch.from_numpy(b).cuda(), x, tol=1e-10, max_iter=5000,
                       precision=ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64)
    assert r["status"] in (ck.CK_E_NOT_CONVERGED, ck.CK_E_BREAKDOWN), r
    assert r["iterations"] <= 60, r
    Mx.close()
