"""Small systems with long or uneven rows: the single-workgroup kernels read
such rows a run of entries at a time, so the edges are those of the runs."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _longer_row(A, row, length):
    """A with stored zeros appended to `row` until it has `length` entries;
    every row sum keeps its bits."""
    k0, k1 = int(A.rp[row]), int(A.rp[row + 1])
    free = np.arange(int(A.col[k1 - 1]) + 1, A.n, dtype=A.col.dtype)[:length - (k1 - k0)]
    assert k1 - k0 + free.size == length
    rp = A.rp.copy()
    rp[row + 1:] += free.size
    return M.CSR(A.n, A.n, rp, np.concatenate([A.col[:k1], free, A.col[k1:]]),
                 np.concatenate([A.val[:k1], np.zeros(free.size), A.val[k1:]]))


def _solve(A, b, **kw):
    import torch
    import paper_2411_10143_amd as ck
    Mx = ck.Matrix.from_csr(A, keep_fp32=True)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r = ck.cg_solve(Mx.handle, torch.from_numpy(b).cuda(), x, tol=1e-10, **kw)
    Mx.close()
    return x.cpu().numpy(), r


def _shifted_lap1d(n):
    A = M.laplacian_1d(n)
    A.val[A.col == np.repeat(np.arange(n), np.diff(A.rp))] = 3.0
    return A


@pytest.mark.parametrize("n", [200, 500, 900, 2000, 4096])
def test_long_rows_of_a_workgroup_keep_the_bits(orc, n):
    """Zeros stored after the entries of three rows change which form of the
    product runs and how many runs of entries a row takes, but no sum."""
    A = _shifted_lap1d(n)
    b = M.vector(n, 3)
    want, r0 = _solve(A, b)
    assert orc.relres(A, b, want) <= 1e-10
    for length in (17, 23, 24, 25, 31, 32, 33, 40, 41, n // 2 - 8):
        B = A
        for row in (0, 7, n // 2):
            B = _longer_row(B, row, length)
        say(f"long rows n={n} length={length}")
        x, r = _solve(B, b)
        assert r["iterations"] == r0["iterations"]
        assert np.array_equal(x.view(np.int64), want.view(np.int64)), length
