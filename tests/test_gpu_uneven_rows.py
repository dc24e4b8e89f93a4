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


def _spd(n, kind):
    """Symmetric pattern with -1 off the diagonal and the row's count + 1 on it."""
    rng = np.random.default_rng(n)
    if kind == "even":
        i, j = rng.integers(0, n, 8 * n), rng.integers(0, n, 8 * n)
    elif kind == "arrow":
        i, j = np.concatenate([np.zeros(n), np.arange(n - 1)]), \
            np.concatenate([np.arange(n), np.arange(1, n)])
    else:   # power-law row lengths
        p = np.arange(1, min(n, 2000) + 1.0) ** -1.8
        deg = rng.choice(p.size, n, p=p / p.sum()) + 1
        i, j = np.repeat(np.arange(n), deg), rng.integers(0, n, deg.sum())
    i, j = i.astype(np.int64), j.astype(np.int64)
    i, j = i[i != j], j[i != j]
    key = np.unique(np.concatenate([i * n + j, j * n + i]))
    rows, cols = np.concatenate([key // n, np.arange(n)]), np.concatenate([key % n, np.arange(n)])
    vals = np.concatenate([np.full(key.size, -1.0), np.bincount(key // n, minlength=n) + 1.0])
    o = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return M.CSR(n, n, rp, cols[o].astype(np.int32), vals[o])


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [300, 1000])
def test_given_lanes_are_the_lanes_that_run(orc, n, mixed):
    """From x0 = 0 the first residual is b in any order, so two solves differ in
    their first iterates only if their inner products sum rows differently."""
    import paper_2411_10143_amd as ck
    A = _spd(n, "even")
    b = M.vector(n, 4)
    prec = ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64
    got = {}
    for cid in (0, 2, 4):
        say(f"lanes n={n} mixed={mixed} config={cid}")
        x, r = _solve(A, b, config=ck.config_from_id(cid), max_iter=6, precision=prec)
        assert r["iterations"] == 6 and r["final_config"] == cid
        ref = orc.cg(A, b, tol=1e-30, maxit=6)["x"]
        assert np.linalg.norm(x - ref) <= (1e-4 if mixed else 1e-10) * np.linalg.norm(ref)
        got[cid] = x
    assert not np.array_equal(got[0], got[2]) and not np.array_equal(got[2], got[4])


@pytest.mark.parametrize("kind", ["arrow", "powerlaw"])
@pytest.mark.parametrize("mixed", [False, True])
def test_hub_rows(orc, kind, mixed):
    import torch
    import paper_2411_10143_amd as ck
    prec = ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64
    srv = ck.server_create(tol=1e-10, large_workers=1, precision=prec)
    keep = []
    for t, n in enumerate((70, 1000, 4097, 6144, 8192)):
        A = _spd(n, kind)
        b = M.vector(n, 6)
        for kw in ({}, {"config": ck.config_from_id(3)}, {"async_": ck.CK_EXEC_SEQUENTIAL}):
            say(f"hub rows {kind} n={n} mixed={mixed} {kw}")
            x, r = _solve(A, b, precision=prec, **kw)
            assert r["status"] == ck.CK_OK and orc.relres(A, b, x) <= 1.01e-10, (n, kw, r)
        dev = [torch.from_numpy(v).cuda() for v in (A.rp, A.col, A.val)]
        db = torch.from_numpy(b).cuda()
        dx = torch.full_like(db, float("nan"))
        torch.cuda.synchronize()
        ck.server_add_matrix(srv, t, *dev)
        keep.append((A, b, dev, db, dx))
    got = []
    for rounds in range(2):                  # one after the other, then all together
        say(f"hub rows {kind} mixed={mixed} requests")
        for t, (_, _, _, db, dx) in enumerate(keep):
            ck.server_submit(srv, t, db, dx, t)
            if rounds == 0:
                ck.server_drain(srv, 60.0)
        ck.server_drain(srv, 60.0)
        assert all(d["status"] == ck.CK_OK for d in ck.server_poll(srv))
        got.append([dx.cpu().numpy() for *_, dx in keep])
        for (A, b, *_), x in zip(keep, got[-1]):
            assert orc.relres(A, b, x) <= 1.01e-10, A.n
    assert all(np.array_equal(a, b) for a, b in zip(*got))
    ck.server_destroy(srv)
