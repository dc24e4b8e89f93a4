"""The one-workgroup CG where its threads and rows per thread change (256, 512,
1,024, 2,048 and 4,096 rows), with the diagonal apart and not (a row with three
entries after its diagonal), and its stop test under scaled right-hand sides."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _two_more(A):
    """Two stored zeros after the middle row's last entry: the same sums, but
    three entries after the diagonal."""
    i = A.n // 2
    k1 = A.rp[i + 1]
    last = A.col[k1 - 1]
    cols = np.concatenate([A.col[:k1], np.array([last + 1, last + 2], A.col.dtype), A.col[k1:]])
    vals = np.concatenate([A.val[:k1], np.zeros(2), A.val[k1:]])
    rp = A.rp.copy()
    rp[i + 1:] += 2
    return M.CSR(A.n, A.ncols, rp, cols, vals)


def _solve(A, b, **kw):
    import torch
    import paper_2411_10143_amd as ck
    Mx = ck.Matrix.from_csr(A)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r = ck.cg_solve(Mx.handle, torch.from_numpy(b).cuda(), x, **kw)
    Mx.close()
    return x.cpu().numpy(), r


@pytest.mark.parametrize("n", [1, 8, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096])
def test_forms_agree_at_the_thread_counts(orc, n):
    import paper_2411_10143_amd as ck
    A = M.laplacian_1d(n)
    A.val[A.col == np.repeat(np.arange(n), np.diff(A.rp))] = 2.5   # well conditioned
    b = M.vector(n, 3)
    say(f"cg workgroup n={n}")
    x, r = _solve(A, b, tol=1e-10)
    assert r["status"] == ck.CK_OK and orc.relres(A, b, x) <= 1e-10
    if n >= 8:
        y, s = _solve(_two_more(A), b, tol=1e-10)
        assert s["iterations"] == r["iterations"]
        assert np.array_equal(x.view(np.int64), y.view(np.int64))


def test_rows_with_one_side_only(orc):
    """Rows of a diagonal entry alone, and rows with entries on one side of it."""
    import paper_2411_10143_amd as ck
    n = 600
    A = M.laplacian_1d(n)
    D = {i: {int(c): float(v) for c, v in zip(A.col[A.rp[i]:A.rp[i + 1]],
                                              A.val[A.rp[i]:A.rp[i + 1]])} for i in range(n)}
    for i, j in ((300, 301), (299, 300), (10, 11)):
        D[i].pop(j)
        D[j].pop(i)
    rp = np.concatenate([[0], np.cumsum([len(D[i]) for i in range(n)])]).astype(np.int32)
    col = np.array([c for i in range(n) for c in sorted(D[i])], np.int32)
    val = np.array([D[i][c] for i in range(n) for c in sorted(D[i])])
    B = M.CSR(n, n, rp, col, val, "gaps").check()
    b = M.vector(n, 4)
    x, r = _solve(B, b, tol=1e-9)
    assert r["status"] == ck.CK_OK and orc.relres(B, b, x) <= 1e-9


@pytest.mark.parametrize("tol", [1e-3, 1e-8, 1e-12])
def test_stop_test_does_not_depend_on_the_scale(tol):
    """Scaling b by a power of two scales every iterate exactly, so the solve
    stops at the same step."""
    A = M.laplacian_2d(40)
    b = M.vector(A.n, 5)
    x, r = _solve(A, b, tol=tol)
    for k in (-400, -3, 400):
        say(f"cg scaled by 2^{k} tol {tol}")
        y, s = _solve(A, np.ldexp(b, k), tol=tol)
        assert s["iterations"] == r["iterations"] and s["status"] == r["status"]
        assert np.array_equal(np.ldexp(x, k), y)
