"""Multi-kernel GMRES at the restart lengths where its kernels change (groups of
eight basis columns, coefficients in registers or LDS) and at the row counts
where its blocks take one more row per thread: iterates against the oracle's
modified Gram-Schmidt, through a restart and at every stop inside a cycle."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _run(ck, h, b, **kw):
    import torch
    x = torch.zeros(b.shape[0], dtype=torch.float64, device="cuda")
    r = ck.gmres_solve(h, torch.from_numpy(b).cuda(), x, **kw)
    return x.cpu().numpy(), r


@pytest.mark.parametrize("m", [1, 2, 7, 8, 9, 16, 17, 24, 25, 32, 33, 40, 41, 48, 56, 57, 63, 64])
def test_restart_lengths(orc, m):
    import paper_2411_10143_amd as ck
    A = M.convection_diffusion_2d(129, 10.0)           # 16,641 rows
    b = orc.spmv(A, M.vector(A.n, 11))
    Mx = ck.Matrix.from_csr(A, keep_fp32=True)
    cfg = ck.config_from_id(ck.ID_DIA)
    for k in sorted({1, m - 1, m, m + 1, 2 * m + 3} - {0}):
        say(f"gmres m={m} k={k}")
        x, r = _run(ck, Mx.handle, b, tol=1e-14, max_iter=k, restart=m, config=cfg)
        ref = orc.gmres(A, b, m=m, tol=1e-14, maxit=k)
        assert r["iterations"] == k
        # both are the minimal-residual iterate; the orthogonalisations differ
        # in rounding only (2^-53 times a condition of about 1e4)
        assert np.max(np.abs(x - ref["x"])) <= 1e-10 * np.max(np.abs(ref["x"]))
    xm, rm = _run(ck, Mx.handle, b, tol=1e-6, restart=m, config=cfg,
                  precision=ck.CK_PREC_MIXED, max_iter=40 * m)
    assert rm["iterations"] <= 40 * m
    Mx.close()


@pytest.mark.parametrize("n", [16385, 131071, 131072, 131073, 262145])
def test_row_counts(orc, n):
    import paper_2411_10143_amd as ck
    A = M.diagonally_dominant(M.uniform_random(n, 3, 1, 6))
    xs = M.vector(n, 5)
    b = orc.spmv(A, xs)
    Mx = ck.Matrix.from_csr(A, keep_fp32=True)
    for prec in (ck.CK_PREC_FP64, ck.CK_PREC_MIXED):
        say(f"gmres rows n={n} precision={prec}")
        x, r = _run(ck, Mx.handle, b, tol=1e-11, precision=prec)
        assert r["status"] == ck.CK_OK
        assert orc.relres(A, b, x) <= 1.01e-11
    Mx.close()
