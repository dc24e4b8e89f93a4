"""DIA with equal values on every diagonal: the constant form gives the bits of
the dense form, and exports the same layout, at the diagonal counts where its
masks and kernels change."""
import numpy as np
import pytest

from helpers import say, spmv_bound
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _diagonals(n, ncols, offsets, seed, drop):
    """Diagonal k holds value k + 0.5 (diagonal 0's may be -0.0), a share of
    the slots missing."""
    rng = np.random.default_rng(seed)
    rows, cols, vals = [], [], []
    for k, d in enumerate(offsets):
        i = np.arange(max(0, -d), min(n, ncols - d))
        i = i[rng.random(i.shape[0]) >= drop] if drop else i
        rows.append(i)
        cols.append(i + d)
        vals.append(np.full(i.shape[0], k + 0.5 if k else -0.0))
    r, c, v = (np.concatenate(t) for t in (rows, cols, vals))
    order = np.lexsort((c, r))
    r, c, v = r[order], c[order], v[order]
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    return M.CSR(n, ncols, rp.astype(np.int32), c.astype(np.int32), v, "diagonals").check()


@pytest.mark.parametrize("drop", [0.0, 0.3])
@pytest.mark.parametrize("nd", [1, 2, 3, 5, 7, 8, 9, 13, 15, 16, 19, 27, 32, 33])
def test_constant_diagonals(orc, nd, drop):
    import torch

    import paper_2411_10143_amd as ck
    n, ncols = 1283, 1283 if nd % 2 else 1300
    offsets = [(k - nd // 2) * (37 if k % 2 else 1) for k in range(nd)]
    offsets = sorted(set(offsets))
    A = _diagonals(n, ncols, offsets, nd, drop)
    say(f"constant diagonals nd={nd} drop={drop}")
    dia = ck.config_from_id(ck.ID_DIA)
    Mx = ck.Matrix.from_csr(A, keep_fp32=True)
    ck.spmv_convert(Mx.handle, dia)
    # the same matrix with one value changed keeps dense values
    B = M.CSR(A.n, A.ncols, A.rp, A.col, A.val.copy(), "changed")
    k = A.nnz // 2
    row = int(np.searchsorted(A.rp, k, side="right")) - 1
    B.val[k] = np.nextafter(B.val[k], 100.0)
    Mb = ck.Matrix.from_csr(B, keep_fp32=True)
    ck.spmv_convert(Mb.handle, dia)
    _, rnd, pitch, off, dv = orc.to_dia(A)
    gnd, gpitch, goff, gdv = ck.export_dia(Mx.handle)
    assert (gnd, gpitch) == (rnd, pitch) and np.array_equal(goff.cpu().numpy(), off)
    assert np.array_equal(gdv.cpu().numpy().view(np.uint64), dv.view(np.uint64))
    rng = np.random.default_rng(2)
    x, y0 = rng.uniform(-1, 1, ncols), rng.uniform(-1, 1, n)
    other = np.arange(n) != row
    for fp32 in (False, True):
        dt = torch.float32 if fp32 else torch.float64
        apply = ck.spmv_apply_f32 if fp32 else ck.spmv_apply
        dx = torch.from_numpy(x).to(dt).cuda()
        for alpha, beta in ((1.0, 0.0), (-0.5, 2.0)):
            got = []
            for h in (Mx.handle, Mb.handle):
                dy = torch.from_numpy(y0).to(dt).cuda()
                apply(h, dx, dy, alpha, beta, dia)
                got.append(dy.cpu().numpy())
            bits = np.uint32 if fp32 else np.uint64
            assert np.array_equal(got[0].view(bits)[other], got[1].view(bits)[other])
            if not fp32:
                ref = orc.spmv(A, x, alpha, beta, y0)
                assert np.all(np.abs(got[0] - ref)
                              <= spmv_bound(orc, A, x, alpha, beta, y0, 2.0 ** -53))
    # a non-finite x reaches every row whose slot on a kept diagonal has that column
    x[5] = np.inf
    dx = torch.from_numpy(x).cuda()
    ys = []
    for h in (Mx.handle, Mb.handle):
        dy = torch.zeros(n, dtype=torch.float64, device="cuda")
        ck.spmv_apply(h, dx, dy, 1.0, 0.0, dia)
        ys.append(dy.cpu().numpy())
    assert np.array_equal(ys[0][other], ys[1][other], equal_nan=True)
    Mx.close()
    Mb.close()
