"""CSR-panel products from slices of x: one to twenty-two slices, one to
sixteen lanes per row, row counts around the conversion's groups of 64, groups
of more entries than the conversion stages (3,072) and a wave keeps (256),
columns next to the slice boundaries, matrices just inside and outside the
rule, and the panels that are reported for them."""
import numpy as np
import pytest

from helpers import say, spmv_bound
from synth import matrices as M

pytestmark = pytest.mark.gpu


def _rows(n, ncols, lo, hi, seed, edges=False):
    """n rows of lo..hi entries, columns over all of x; with `edges` every third
    row is made of columns next to multiples of 64 (where slices may end)."""
    rng = np.random.default_rng(seed)
    length = rng.integers(lo, hi + 1, n)
    rp = np.concatenate([[0], np.cumsum(length)])
    col = rng.integers(0, ncols, rp[-1])
    row = np.repeat(np.arange(n), length)
    if edges:
        near = np.clip(64 * rng.integers(0, ncols // 64 + 1, rp[-1]) - rng.integers(0, 2, rp[-1]),
                       0, ncols - 1)
        col = np.where(row % 3 == 0, near, col)
    key = np.unique(row * np.int64(ncols) + col)
    rp = np.concatenate([[0], np.cumsum(np.bincount(key // ncols, minlength=n))]).astype(np.int32)
    return M.CSR(n, ncols, rp, (key % ncols).astype(np.int32),
                 rng.uniform(-1, 1, len(key)), "slices").check()


# rows, columns, row lengths; whether they take slices
CASES = {
    "one_slice": (15_000, 15_000, 90, 110, True),
    "one_slice_few_rows": (7_000, 15_360, 190, 210, False),       # 1,309,202 entries: 1,518 too few
    "sixteen_lanes": (7_100, 15_360, 190, 210, True),             # per row
    "two_slices": (44_992, 15_361, 25, 40, True),
    "rows_64k_plus_1": (30_017, 30_721, 60, 70, True),
    "rows_64k_minus_1": (30_015, 100_000, 55, 60, True),
    "twenty_two_slices": (65_000, 337_900, 33, 44, True),
    "long_groups": (3_001, 60_000, 500, 900, True),               # 64 rows: 45,000 entries
    "last_row_alone": (40_001, 40_000, 36, 48, True),
    "too_few_entries": (26_000, 26_000, 45, 50, False),
    "rows_too_short": (110_000, 170_000, 13, 15, False),          # 15 entries, 12 slices
    "rows_uneven": (60_000, 60_000, 4, 60, False),                # one row of 200 is added
}


def _case(name):
    n, ncols, lo, hi, taken = CASES[name]
    A = _rows(n, ncols, lo, hi, 5, edges=True)
    if name == "rows_uneven":
        long = np.arange(0, ncols, ncols // 200)[:200].astype(np.int32)
        col = np.concatenate([A.col, long])
        val = np.concatenate([A.val, np.ones(len(long))])
        rp = np.concatenate([A.rp, [len(col)]]).astype(np.int32)
        A = M.CSR(n + 1, ncols, rp, col, val, "uneven").check()
    return A, taken


@pytest.mark.parametrize("name", list(CASES))
def test_slices(orc, name):
    import torch
    import paper_2411_10143_amd as ck
    A, taken = _case(name)
    say(f"slices {name} n={A.n} ncols={A.ncols} nnz={len(A.col)}")
    cfg = ck.config_from_id(11)
    rng = np.random.default_rng(6)
    for fp32 in (False, True):
        dt = torch.float32 if fp32 else torch.float64
        x, y0 = rng.uniform(-1, 1, A.ncols), rng.uniform(-1, 1, A.n)
        B = A
        if fp32:
            x, y0 = (v.astype(np.float32).astype(float) for v in (x, y0))
            B = M.CSR(A.n, A.ncols, A.rp, A.col, A.val.astype(np.float32).astype(float), A.name)
        u = 2.0 ** (-24 if fp32 else -53)
        Mx = ck.Matrix.from_csr(A, keep_fp32=True)
        apply = ck.spmv_apply_f32 if fp32 else ck.spmv_apply
        dx = torch.from_numpy(x).to(dt).cuda()

        def product(alpha, beta):
            dy = torch.from_numpy(y0).to(dt).cuda()
            apply(Mx.handle, dx, dy, alpha, beta, cfg)
            return dy

        before = torch.cuda.memory_allocated()
        ck.spmv_convert(Mx.handle, cfg)
        grown = torch.cuda.memory_allocated() - before
        # 14 bytes per entry and the rows' ends, or 16 and the partition
        assert (grown < 16 * len(A.col)) == taken, (name, grown)
        for alpha, beta in ((1.0, 0.0), (-0.5, 2.0)):
            got = product(alpha, beta)
            ref = orc.spmv(B, x, alpha, beta, y0)
            bound = spmv_bound(orc, B, x, alpha, beta, y0, u, k_extra=3)
            assert np.all(np.abs(got.cpu().numpy().astype(float) - ref) <= bound), (name, fp32)
            assert torch.equal(got, product(alpha, beta))
        P, W, rows = ck.panel_layout(Mx.handle)
        assert P in (4, 8) and W == -(-A.ncols // P) and rows <= P * A.n
        Mx.close()


def test_slices_pass_non_finite_values_by_column(orc):
    """A NaN or an infinity in x reaches the rows that store its column, only."""
    import torch
    import paper_2411_10143_amd as ck
    A, _ = _case("two_slices")
    x = np.ones(A.ncols)
    x[[0, 7_000, A.ncols - 1]] = np.nan, np.inf, -np.inf
    hit = np.isin(A.col, [0, 7_000, A.ncols - 1])
    rows = np.unique(np.repeat(np.arange(A.n), np.diff(A.rp))[hit])
    Mx = ck.Matrix.from_csr(A)
    cfg = ck.config_from_id(11)
    ck.spmv_convert(Mx.handle, cfg)
    y = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    ck.spmv_apply(Mx.handle, torch.from_numpy(x).cuda(), y, cfg=cfg)
    bad = np.flatnonzero(~np.isfinite(y.cpu().numpy()))
    assert np.array_equal(bad, rows)
    Mx.close()


def test_slices_without_allocation_and_in_a_graph(orc):
    import torch
    import paper_2411_10143_amd as ck
    A, _ = _case("twenty_two_slices")
    Mx = ck.Matrix.from_csr(A)
    cfg = ck.config_from_id(11)
    ck.spmv_convert(Mx.handle, cfg)
    x = torch.rand(A.ncols, dtype=torch.float64, device="cuda")
    y = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    ck.spmv_apply(Mx.handle, x, y, cfg=cfg)
    want = y.clone()
    y.zero_()
    ck.spmv_apply_noalloc(Mx.handle, x, y, cfg=cfg)
    assert torch.equal(y, want)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        ck.spmv_apply(Mx.handle, x, y, cfg=cfg)      # this stream's workspace
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ck.spmv_apply(Mx.handle, x, y, cfg=cfg)
    for r in range(3):
        x.copy_(torch.rand(A.ncols, dtype=torch.float64, device="cuda"))
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        eager = torch.zeros_like(y)
        ck.spmv_apply(Mx.handle, x, eager, cfg=cfg)
        assert torch.equal(y, eager), r
    Mx.close()
