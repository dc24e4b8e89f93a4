"""Small systems at the edges of the one-workgroup solvers: the row counts
where the threads of a slot change (1,024), where its vectors stop fitting the
workgroup (8,192), and the smallest, in the request loop and as single solves."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _spd(n):
    """tridiag(-1, 4, -1)"""
    A = M.laplacian_1d(n)
    rows = np.repeat(np.arange(n), np.diff(A.rp))
    A.val[A.col == rows] = 4.0
    return A


def _general(n):
    return M.diagonally_dominant(M.uniform_random(n, 40 + n, 1, 40))


SIZES = [1, 2, 65, 1023, 1024, 1025, 4097, 8192, 8193]


@pytest.mark.parametrize("mixed", [True, False])
def test_slots(orc, mixed):
    import torch

    import paper_2411_10143_amd as ck
    srv = ck.server_create(small_n=9000, tol=1e-11, large_workers=1,
                           precision=ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64)
    keep, want = [], []
    for t, A in enumerate([f(n) for n in SIZES for f in (_spd, _general)]):
        dev = [torch.from_numpy(v).cuda() for v in (A.rp, A.col, A.val)]
        b = orc.spmv(A, M.vector(A.n, 7 + t))
        db = torch.from_numpy(b).cuda()
        dx = torch.full_like(db, float("nan"))
        torch.cuda.synchronize()
        ck.server_add_matrix(srv, t, *dev)
        keep.append((dev, db, dx))
        want.append((A, b))
    say(f"slots n={SIZES} mixed={mixed}")
    for rounds in range(2):                  # alone one after the other, then all together
        for t, (_, db, dx) in enumerate(keep):
            ck.server_submit(srv, t, db, dx, t)
            if rounds == 0:
                ck.server_drain(srv, 60.0)
        ck.server_drain(srv, 60.0)
        done = ck.server_poll(srv)
        assert len(done) == len(keep)
        assert all(d["status"] == ck.CK_OK and d["path"] == 0 for d in done)
        got = [dx.clone() for _, _, dx in keep]
        for (A, b), x in zip(want, got):
            assert orc.relres(A, b, x.cpu().numpy()) <= 1.01e-11, A.name
        if rounds == 0:
            first = got
    assert all(torch.equal(a, b) for a, b in zip(first, got))   # bits do not depend on the mix
    ck.server_destroy(srv)


@pytest.mark.parametrize("mixed", [True, False])
@pytest.mark.parametrize("n", [1, 1024, 8192, 8193, 16384])
def test_single_solves(orc, n, mixed):
    import torch

    import paper_2411_10143_amd as ck
    prec = ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64
    for A, solve in ((_spd(n), ck.cg_solve), (_general(n), ck.gmres_solve)):
        say(f"single {solve.__name__} n={n} mixed={mixed}")
        Mx = ck.Matrix.from_csr(A, keep_fp32=True)
        b = orc.spmv(A, M.vector(n, 5))
        db = torch.from_numpy(b).cuda()
        x = torch.zeros_like(db)
        r = solve(Mx.handle, db, x, tol=1e-11, precision=prec, config=ck.config_from_id(2))
        assert r["status"] == ck.CK_OK, r
        assert orc.relres(A, b, x.cpu().numpy()) <= 1.01e-11
        # the iteration budget is kept
        x.zero_()
        r = solve(Mx.handle, db, x, tol=0.0, precision=prec, max_iter=3,
                  config=ck.config_from_id(2))
        assert r["iterations"] <= 3
        Mx.close()
