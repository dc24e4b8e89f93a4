"""Single solves at the row counts where CG leaves the one-workgroup kernels
(4,096 and 6,144 in FP64, 8,192 in mixed precision), and GMRES of systems
smaller than its restart."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _solve(A, b, cg, mixed, tol, **kw):
    import torch
    import paper_2411_10143_amd as ck
    Mx = ck.Matrix.from_csr(A, keep_fp32=mixed)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    f = ck.cg_solve if cg else ck.gmres_solve
    r = f(Mx.handle, torch.from_numpy(b).cuda(), x, tol=tol,
          precision=ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64, **kw)
    Mx.close()
    return x.cpu().numpy(), r


@pytest.mark.parametrize("mixed,n", [(False, 4096), (False, 4097), (False, 6144), (False, 6145),
                                     (True, 8191), (True, 8192), (True, 8193), (False, 16385)])
def test_cg_at_the_limits(orc, mixed, n):
    import paper_2411_10143_amd as ck
    A = M.laplacian_1d(n)
    A.val[A.col == np.repeat(np.arange(n), np.diff(A.rp))] = 3.0
    b = M.vector(n, 7)
    say(f"cg n={n} mixed={mixed}")
    x, r = _solve(A, b, True, mixed, 1e-10)
    assert r["status"] == ck.CK_OK and orc.relres(A, b, x) <= 1e-10
    ref = orc.cg(A, b, tol=1e-10)
    if not mixed:
        assert abs(r["iterations"] - ref["iters"]) <= 3


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 29, 30, 31, 64, 257, 8192])
def test_gmres_of_few_rows(orc, n, mixed):
    import paper_2411_10143_amd as ck
    A = M.diagonally_dominant(M.uniform_random(n, 60 + n, 1, min(n, 20)))
    b = M.vector(n, 8)
    say(f"gmres n={n} mixed={mixed}")
    x, r = _solve(A, b, False, mixed, 1e-10)
    assert r["status"] == ck.CK_OK and orc.relres(A, b, x) <= 1e-10
    for m in (1, 5):
        x, r = _solve(A, b, False, mixed, 1e-8, restart=m, max_iter=4000)
        assert r["status"] == ck.CK_OK and orc.relres(A, b, x) <= 1e-8, m
