"""Merge-path products at the edges of the workgroup split: rows as long as a
workgroup may reach back for its start (64 entries) and one more, runs of
empty rows, rows across workgroups, and totals around whole workgroups, with
the converted plan, without it, and as CSR-panel and COO."""
import numpy as np
import pytest

from helpers import say, spmv_bound
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _rows(lengths, ncols, seed):
    """Rows of the given lengths, columns spread over ncols."""
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    col = np.concatenate([np.sort(rng.choice(ncols, r, replace=False)) for r in lengths]
                         + [np.zeros(0)]).astype(np.int32)
    return M.CSR(len(lengths), ncols, rp, col, rng.uniform(-1, 1, rp[-1]), "edge").check()


EDGES = {
    "rows_of_63": [63] * 200,
    "rows_of_64": [64] * 200,                  # never cut
    "rows_of_65": [65] * 200,                  # cut at some starts
    "one_workgroup": [1] * 1024,               # 2048 items
    "one_more": [1] * 1024 + [1],
    "span": [1983] + [0] * 1983 + [5],         # a row, then a workgroup of empty rows
    "empty_runs": ([0] * 2100 + [3]) * 3 + [0] * 2500,
    "hub": [7] * 300 + [9000] + [0] * 70 + [64] * 40,
    "last_row_open": [2] * 500 + [4100],
}


@pytest.mark.parametrize("name", list(EDGES))
@pytest.mark.parametrize("fp32", [False, True])
def test_merge_edges(orc, name, fp32):
    import torch

    import paper_2411_10143_amd as ck
    A = _rows(EDGES[name], 12000, 3)
    say(f"merge edges {name} fp32={fp32}")
    dt = torch.float32 if fp32 else torch.float64
    rng = np.random.default_rng(4)
    x, y0 = rng.uniform(-1, 1, A.ncols), rng.uniform(-1, 1, A.n)
    if fp32:
        x, y0 = (v.astype(np.float32).astype(float) for v in (x, y0))
        A = M.CSR(A.n, A.ncols, A.rp, A.col, A.val.astype(np.float32).astype(float), A.name)
    ref = orc.spmv(A, x, -0.5, 2.0, y0)
    bound = spmv_bound(orc, A, x, -0.5, 2.0, y0, 2.0 ** (-24 if fp32 else -53), k_extra=3)
    Mx = ck.Matrix.from_csr(A, keep_fp32=fp32)
    apply = ck.spmv_apply_f32 if fp32 else ck.spmv_apply
    dx = torch.from_numpy(x).to(dt).cuda()

    def product(cid):
        dy = torch.from_numpy(y0).to(dt).cuda()
        apply(Mx.handle, dx, dy, -0.5, 2.0, ck.config_from_id(cid))
        return dy

    before = product(8)                        # no plan yet: the workgroups search
    for cid in (8, 10, 11):
        ck.spmv_convert(Mx.handle, ck.config_from_id(cid))
        got = product(cid)
        assert np.all(np.abs(got.cpu().numpy().astype(float) - ref) <= bound), (name, cid)
        if cid == 8:
            assert torch.equal(got, before)
    Mx.close()
