"""The CSR-panel copy at the edges of its conversion: rows around the lengths
from which a row is counted by search (64) and copied by a whole workgroup
(512), several of them in one group of 32 rows, columns on both sides of every
panel boundary, row counts around 32, and four to twenty-four panels."""
import numpy as np
import pytest

from helpers import say, spmv_bound
from synth import matrices as M

pytestmark = pytest.mark.gpu

# (panels, columns); rows of even length that fill four panels take four
PANELS = [(4, 30_000), (8, 30_000), (8, 2_000_003), (16, 2_100_000), (24, 4_400_001)]


def _rows(lengths, ncols, P, seed):
    """Rows of the given lengths; every other row starts with the columns next
    to the panel boundaries (they depend on the panels, P of them)."""
    rng = np.random.default_rng(seed)
    W = -(-ncols // P)
    edge = np.unique([c for p in range(P) for c in (p * W, min((p + 1) * W, ncols) - 1)])
    cols = []
    for j, r in enumerate(lengths):
        c = rng.choice(ncols, r, replace=False)
        if j % 2 and r > len(edge):
            c = np.concatenate([edge, np.setdiff1d(c, edge)])[:r]
        cols.append(np.sort(c))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    col = np.concatenate(cols).astype(np.int32)
    return M.CSR(len(lengths), ncols, rp, col, rng.uniform(-1, 1, rp[-1]), "edge").check()


LENGTHS = {
    "count": [63, 64, 65, 0] * 16,
    "copy": [511, 512, 513, 40, 1025] * 13 + [600],
    "rows_31": [70] * 31,
    "rows_33": [3] * 30 + [900, 0, 20],
    "short": [0, 1, 2, 0, 0] * 300,
    "even": [34, 20, 48] * 70 + [64],          # 32 rows fit the staging of the copy
    "even_long": [180, 200, 90] * 30,          # and do not
}


@pytest.mark.parametrize("P,ncols", PANELS)
@pytest.mark.parametrize("name", list(LENGTHS))
def test_panel_edges(orc, name, P, ncols):
    import torch
    import paper_2411_10143_amd as ck
    A = _rows(LENGTHS[name], ncols, P, 7)
    say(f"panel edges {name} P={P} ncols={ncols}")
    rng = np.random.default_rng(8)
    x, y0 = rng.uniform(-1, 1, A.ncols), rng.uniform(-1, 1, A.n)
    ref = orc.spmv(A, x, -0.5, 2.0, y0)
    bound = spmv_bound(orc, A, x, -0.5, 2.0, y0, 2.0 ** -53, k_extra=3)
    Mx = ck.Matrix.from_csr(A)
    cfg = ck.config_from_id(11)
    ck.spmv_convert(Mx.handle, cfg)
    dy = torch.from_numpy(y0).cuda()
    ck.spmv_apply(Mx.handle, torch.from_numpy(x).cuda(), dy, -0.5, 2.0, cfg)
    assert np.all(np.abs(dy.cpu().numpy() - ref) <= bound), name
    Mx.close()
