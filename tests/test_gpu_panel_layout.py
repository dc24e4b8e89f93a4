"""The panels reported for a matrix whose CSR-panel copy is by slices of x: those
of the documented rule, without device work, also inside a capture; and CG with
the fused dot product on such a copy."""
import numpy as np
import pytest

from helpers import say, upload
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _rows(n, ncols, lo, hi, most=None):
    """Rows of lo..hi entries over all columns, or over the first `most` of 8 parts
    except in the rows' first and last entry."""
    rng = np.random.default_rng(n + ncols)
    row = np.repeat(np.arange(n), rng.integers(lo, hi + 1, n))
    col = rng.integers(0, ncols if most is None else ncols * most // 8, row.size)
    if most is not None:
        row = np.concatenate([row, np.arange(n)])
        col = np.concatenate([col, np.full(n, ncols - 1)])
    key = np.unique(row * np.int64(ncols) + col)
    rp = np.concatenate([[0], np.cumsum(np.bincount(key // ncols, minlength=n))]).astype(np.int32)
    return M.CSR(n, ncols, rp, (key % ncols).astype(np.int32),
                 rng.uniform(-1, 1, key.size), "panels").check()


def _expected(A):
    rows = np.repeat(np.arange(A.n, dtype=np.int64), np.diff(A.rp))

    def filled(P):
        return len(np.unique(rows * P + A.col.astype(np.int64) // -(-A.ncols // P)))

    P = 4 if 4 * filled(4) > 3 * 4 * A.n else 8
    return P, -(-A.ncols // P), (P * A.n if 4 * filled(P) > 3 * P * A.n else filled(P))


CASES = {
    "four": (45_000, 45_000, 30, 50, None),
    "four_ragged": (44_999, 61_441, 31, 49, None),
    "few_columns": (700_001, 3, 2, 3, None),
    "seven": (30_001, 30_003, 60, 70, 7),
    "eight_listed": (30_001, 30_003, 60, 70, 2),     # two of four panels and the last filled
    "wide": (70_000, 300_000, 30, 40, None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_layout_of_slices(name):
    import torch
    import paper_2411_10143_amd as ck
    A = _rows(*CASES[name])
    blocks = [0]

    def alloc(nbytes, stream):
        blocks[0] += 1
        return torch.cuda.caching_allocator_alloc(nbytes, torch.cuda.current_device(), stream)

    def free(p, stream):
        torch.cuda.caching_allocator_delete(p)

    Mx = ck.Matrix(*upload(A), ncols=A.ncols, allocator=ck.CallbackAllocator(alloc, free))
    say(f"panel layout of slices {name} n={A.n} ncols={A.ncols} nnz={A.nnz}")
    before = torch.cuda.memory_allocated()
    ck.spmv_convert(Mx.handle, ck.config_from_id(11))
    assert torch.cuda.memory_allocated() - before < 16 * A.nnz      # by slices: 10 bytes and ends
    blocks[0] = 0
    want = _expected(A)
    assert ck.panel_layout(Mx.handle) == want
    assert blocks[0] == 0
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        inside = ck.panel_layout(Mx.handle)
    assert inside == want
    Mx.close()


@pytest.mark.parametrize("mixed", [False, True])
def test_cg_on_slices(orc, mixed):
    import torch
    import paper_2411_10143_amd as ck
    n, rng = 45_000, np.random.default_rng(9)
    i, j = rng.integers(0, n, 20 * n), rng.integers(0, n, 20 * n)
    i, j = i[i != j], j[i != j]
    key = np.unique(np.concatenate([i * n + j, j * n + i]))
    vals = -1.0 / (1 + np.minimum(key // n, key % n) % 7)           # symmetric
    rows, cols = np.concatenate([key // n, np.arange(n)]), np.concatenate([key % n, np.arange(n)])
    vals = np.concatenate([vals, np.bincount(key // n, -vals, minlength=n) + 0.05])
    o = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    A = M.CSR(n, n, rp, cols[o].astype(np.int32), vals[o], "spd").check()
    b = M.vector(n, 1)
    say(f"cg on slices n={n} nnz={A.nnz} mixed={mixed}")
    Mx = ck.Matrix(*upload(A), keep_fp32=True)
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    kw = dict(config=ck.config_from_id(11),
              precision=ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64)
    r = ck.cg_solve(Mx.handle, torch.from_numpy(b).cuda(), x, tol=1e-10, **kw)
    assert r["status"] == ck.CK_OK and r["final_config"] == 11
    assert orc.relres(A, b, x.cpu().numpy()) <= 1.01e-10
    if not mixed:
        ref = orc.cg(A, b, tol=1e-10)
        assert abs(r["iterations"] - ref["iters"]) <= 3
        x.zero_()
        r = ck.cg_solve(Mx.handle, torch.from_numpy(b).cuda(), x, tol=1e-30, max_iter=5, **kw)
        want = orc.cg(A, b, tol=1e-30, maxit=5)["x"]
        assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-12 * np.linalg.norm(want)
    Mx.close()
