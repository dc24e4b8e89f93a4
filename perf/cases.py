"""What a user has this library do, as cases that can be timed: sparse products
on the configuration the cascade picks, the preparation of a new matrix, CG
and GMRES solves, and a burst of requests to the solver service.

The matrices are the families of the SpMV set and of the serving pool (banded
stencils, power-law rows, 8x8 diagonal blocks, uniform-random rows, Laplacians,
convection-diffusion, diagonally dominant patterns), drawn on the GPU from a
seed, with the sizes of the set: 1e4 to 2e6 rows.
"""
import math

import numpy as np
import torch

import paper_2411_10143_amd as ck

RMAX = 10_000          # longest power-law row
CENTRE = {5: 2, 9: 2, 7: 3, 13: 3, 19: 3, 27: 3}   # stencil points -> dimensions


def listed():
    return [
        # a small stencil matrix: one product is a few microseconds, so the
        # launch and the call count
        {"name": "product_banded_10k", "kind": "product", "family": "banded", "n": 10_000,
         "points": 5},
        # a small matrix with hub rows up to 10^4 entries long
        {"name": "product_powerlaw_42k", "kind": "product", "family": "powerlaw", "n": 42_418,
         "s": 1.864},
        # the large 27-point stencil of the set
        {"name": "product_banded_2m", "kind": "product", "family": "banded", "n": 2_000_000,
         "points": 27},
        # a mid-size scattered matrix in FP32 (the inner products of the mixed solvers)
        {"name": "product_uniform_180k_f32", "kind": "product", "family": "uniform",
         "n": 179_932, "fp32": True},
        # the residual r = b - A x of a large matrix with hub rows
        {"name": "residual_powerlaw_1.2m", "kind": "residual", "family": "powerlaw",
         "n": 1_235_508, "s": 1.682},
        # the largest scattered matrix of the set (row lengths 4 to 64)
        {"name": "product_uniform_2m", "kind": "product", "family": "uniform", "n": 2_000_000},
        # a matrix seen for the first time: ingest, features, cascade,
        # conversion and the first product
        {"name": "prepare_uniform_471k", "kind": "prepare", "family": "uniform", "n": 471_494},
        # the small CG of the headline metric (64 x 64 Laplacian, 1e-10)
        {"name": "cg_lap2d_64", "kind": "cg", "family": "lap2d", "n": 64, "tol": 1e-10},
        # asynchronous CG on the 3D Poisson system, 1e-10
        {"name": "cg_poisson_128", "kind": "cg", "family": "lap3d", "n": 128, "tol": 1e-10,
         "async": True},
        # eight cycles of FP64 GMRES(30) on convection-diffusion 1024^2
        {"name": "gmres_convdiff_1024", "kind": "gmres", "family": "convdiff", "n": 1024,
         "max_iter": 240},
        # mixed-precision GMRES(30) of a serving-pool member, solved to 1e-10
        {"name": "gmres_mixed_dominant_150k", "kind": "gmres", "family": "dominant",
         "n": 150_001, "tol": 1e-10, "mixed": True},
        # a burst of requests on six small matrices, batched in slots
        {"name": "serve_small_24", "kind": "serve", "n": 7_000, "requests": 24, "tol": 1e-12},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["product"] * 6 + ["residual"] * 2 + ["prepare", "cg", "gmres", "serve"])
    if kind in ("product", "residual", "prepare"):
        family = rng.choice(["banded", "powerlaw", "blocks", "uniform"])
        c = {"kind": kind, "family": family, "n": size(1e4, 1.2e6)}
        if family == "banded":
            c["points"] = rng.choice(sorted(CENTRE))
        if family == "powerlaw":
            c["s"] = round(rng.uniform(1.6, 2.5), 3)
        if kind == "product" and rng.random() < 0.3:
            c["fp32"] = True
        return c
    if kind == "cg":
        if rng.random() < 0.5:
            return {"kind": "cg", "family": "lap2d", "n": size(16, 64), "tol": 1e-10}
        return {"kind": "cg", "family": "lap3d", "n": size(30, 100), "tol": 1e-10,
                "async": rng.random() < 0.5}
    if kind == "gmres":
        if rng.random() < 0.5:
            return {"kind": "gmres", "family": "convdiff", "n": size(150, 900), "max_iter": 240}
        return {"kind": "gmres", "family": "dominant", "n": size(2e3, 1.5e5), "tol": 1e-10,
                "mixed": rng.random() < 0.7}
    return {"kind": "serve", "n": size(1.5e3, 8e3), "requests": rng.randrange(6, 48),
            "tol": 1e-12}


# ---- matrices (device CSR: rp int32, col int32, val float64) ---------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, count):
    return torch.randn(count, generator=g, device="cuda", dtype=torch.float64)


def _uniform(g, count):
    return torch.rand(count, generator=g, device="cuda", dtype=torch.float64) * 2 - 1


def _csr(n, rows, cols, vals):
    """CSR of triples already sorted by row, then column."""
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0).to(torch.int32)
    return rp, cols.to(torch.int32), vals


def _from_keys(n, key, g):
    """Distinct entries row * n + col, with N(0, 1) values."""
    key = torch.unique_consecutive(torch.sort(key).values)
    return _csr(n, key // n, key % n, _normal(g, key.numel()))


def _stencil_points(points):
    dim = CENTRE[points]
    cube = [()]
    for _ in range(dim):
        cube = [c + (o,) for c in cube for o in (-1, 0, 1)]
    if points in (9, 27):
        return dim, cube
    if points == 19:
        return dim, [c for c in cube if sum(map(abs, c)) <= 2]
    star = [c for c in cube if sum(map(abs, c)) <= 1]
    if points == 13:
        star += [tuple(2 * o for o in c) for c in star if any(c)]
    return dim, star


def _stencil(n, dims, offsets, weight=None, g=None):
    """Stencil on the first n points of a row-major grid, neighbours outside
    it dropped; weight(offset) gives the values, else they are N(0, 1)."""
    strides = [math.prod(dims[d + 1:]) for d in range(len(dims))]
    offsets = sorted(offsets, key=lambda c: sum(o * s for o, s in zip(c, strides)))
    i = torch.arange(n, device="cuda")
    cols, ok = [], []
    for c in offsets:
        good = torch.ones(n, dtype=torch.bool, device="cuda")
        for o, s, d in zip(c, strides, dims):
            at = i // s % d + o
            good &= (at >= 0) & (at < d)
        j = i + sum(o * s for o, s in zip(c, strides))
        cols.append(j)
        ok.append(good & (j >= 0) & (j < n))
    cols, ok = torch.stack(cols, 1), torch.stack(ok, 1)
    rows = i[:, None].expand(-1, len(offsets))[ok]
    if weight is None:
        vals = _normal(g, rows.numel())
    else:
        w = torch.tensor([weight(c) for c in offsets], dtype=torch.float64, device="cuda")
        vals = w.expand(n, -1)[ok]
    return _csr(n, rows, cols[ok], vals)


def _random_rows(n, lengths, g):
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), lengths)
    cols = torch.randint(0, n, (rows.numel(),), generator=g, device="cuda")
    return _from_keys(n, rows * n + cols, g)


def _zipf(s, rmax):
    k = np.arange(1, rmax + 1, dtype=np.float64)
    p = k ** -s
    return k, p / p.sum()


def _dominant(n, rp, col, val):
    """a_ii = 1 + sum of the row's other magnitudes."""
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(rp.long()))
    off = rows != col
    rows, col, val = rows[off], col[off].long(), val[off]
    i = torch.arange(n, device="cuda")
    d = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, val.abs()) + 1
    key = torch.cat([rows * n + col, i * n + i])
    order = torch.argsort(key)
    key, val = key[order], torch.cat([val, d])[order]
    return _csr(n, key // n, key % n, val)


def matrix(case, g):
    family, n = case["family"], case["n"]
    if family == "banded":
        dim, offsets = _stencil_points(case["points"])
        side = math.ceil(n ** (1.0 / dim) - 1e-9)
        rest = side ** (dim - 1)
        return _stencil(n, (math.ceil(n / rest),) + (side,) * (dim - 1), offsets, g=g)
    if family == "blocks":
        n = -(-n // 8) * 8
        i = torch.arange(n, device="cuda")
        rows = i.repeat_interleave(8)
        cols = (i // 8 * 8).repeat_interleave(8) + torch.arange(8, device="cuda").repeat(n)
        return _csr(n, rows, cols, _normal(g, 8 * n))
    if family == "powerlaw":
        cdf = torch.from_numpy(np.cumsum(_zipf(case["s"], min(RMAX, n))[1])).cuda()
        u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
        return _random_rows(n, torch.searchsorted(cdf, u).clamp(max=min(RMAX, n) - 1) + 1, g)
    if family in ("uniform", "dominant"):
        most = 64 if family == "uniform" else 32
        A = _random_rows(n, torch.randint(4, most + 1, (n,), generator=g, device="cuda"), g)
        return A if family == "uniform" else _dominant(n, *A)
    if family in ("lap2d", "lap3d"):
        dim = 2 if family == "lap2d" else 3
        offsets = _stencil_points(5 if dim == 2 else 7)[1]
        return _stencil(n ** dim, (n,) * dim, offsets,
                        weight=lambda c: -1.0 if any(c) else 2.0 * dim)
    if family == "convdiff":   # 5-point upwind, global Peclet number 10
        ph = 10.0 / (n + 1)
        return _stencil(n * n, (n, n), _stencil_points(5)[1],
                        weight=lambda c: 4 + 2 * ph if not any(c) else
                        -1 - ph if min(c) < 0 else -1.0)
    raise ValueError(family)


def _pool(case, g):
    """The small matrices of a service: a Laplacian of about n rows, then
    diagonally dominant ones of fewer."""
    n = case["n"]
    side = int(math.sqrt(n))
    pool = [matrix({"family": "lap2d", "n": side}, g), matrix({"family": "lap2d", "n": side // 2}, g)]
    for part in (1.0, 0.7, 0.4, 0.2):
        pool.append(matrix({"family": "dominant", "n": max(200, int(n * part))}, g))
    return pool


def _product(A, x):
    """A x in plain torch, in x's type."""
    rp, col, val = A
    rows = torch.repeat_interleave(torch.arange(rp.numel() - 1, device="cuda"),
                                   torch.diff(rp.long()))
    y = torch.zeros(rp.numel() - 1, dtype=x.dtype, device="cuda")
    return y.index_add_(0, rows, val.to(x.dtype) * x[col])


# ---- the calls -----------------------------------------------------------------

def _inputs(case, seed):
    """The matrix and the vectors a call on it needs, from the seed."""
    g = _gen(seed)
    if case["kind"] == "serve":
        pool = _pool(case, g)
        return pool, [_uniform(g, pool[t % len(pool)][0].numel() - 1)
                      for t in range(case["requests"])]
    A = matrix(case, g)
    n = A[0].numel() - 1
    return A, [_uniform(g, n), _uniform(g, n)]


class _Service:
    """A server and what its requests need; closed with the state."""

    def __init__(self, case, pool, stars):
        self.pool = pool
        self.b = [_product(pool[t % len(pool)], x) for t, x in enumerate(stars)]
        self.x = [torch.zeros_like(b) for b in self.b]
        torch.cuda.synchronize()
        self.srv = ck.server_create(budget_bytes=8 << 30, large_workers=1, tol=case["tol"])
        for t, A in enumerate(pool):
            ck.server_add_matrix(self.srv, t, *A)

    def __del__(self):
        if getattr(self, "srv", None):
            ck.server_destroy(self.srv)


def prepare(case, seed):
    A, vectors = _inputs(case, seed)
    kind = case["kind"]
    if kind == "serve":
        return {"case": case, "service": _Service(case, A, vectors)}
    state = {"case": case, "A": A, "x": vectors[0]}
    if kind == "prepare":
        state["y"] = torch.zeros_like(vectors[0])
        return state
    fp32 = bool(case.get("fp32") or case.get("mixed"))
    M = state["M"] = ck.Matrix(*A, keep_fp32=fp32)
    if case.get("family") == "lap2d" or case.get("async"):
        cfg = None                       # the solver's own choice
    else:
        cfg = ck.spmv_select(ck.spmv_features(M.handle, symmetry=False))
        try:
            ck.spmv_convert(M.handle, cfg)
        except ck.CkError as e:
            if e.status != ck.CK_E_UNSUPPORTED:
                raise
            cfg = ck.default_config(M.handle)
    state["cfg"] = cfg
    if kind in ("cg", "gmres"):
        state["b"] = _product(A, vectors[0])
        state["x"] = torch.zeros_like(state["b"])
        return state
    if case.get("fp32"):
        state["x"] = state["x"].float()
    state["b"] = vectors[1]
    state["y"] = torch.zeros_like(state["x"])
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "product":
        call = ck.spmv_apply_f32 if case.get("fp32") else ck.spmv_apply
        call(state["M"].handle, state["x"], state["y"], cfg=state["cfg"])
        return state["y"]
    if kind == "residual":
        state["y"].copy_(state["b"])
        ck.spmv_apply(state["M"].handle, state["x"], state["y"], alpha=-1.0, beta=1.0,
                      cfg=state["cfg"])
        return state["y"]
    if kind == "prepare":
        M = ck.Matrix(*state["A"])
        F = ck.spmv_features(M.handle, symmetry=False)
        cfg = ck.spmv_select(F)
        try:
            ck.spmv_convert(M.handle, cfg)
        except ck.CkError as e:
            if e.status != ck.CK_E_UNSUPPORTED:
                raise
            cfg = ck.default_config(M.handle)
        ck.spmv_apply(M.handle, state["x"], state["y"], cfg=cfg)
        state["M"] = M                   # the matrix before it is released here
        return {"y": state["y"], "features": np.array(F.ints(), dtype=np.int64)}
    if kind == "serve":
        s = state["service"]
        for t, (b, x) in enumerate(zip(s.b, s.x)):
            ck.server_submit(s.srv, t % len(s.pool), b, x, t)
        ck.server_drain(s.srv, 60.0)
        ck.server_poll(s.srv)
        return s.x
    state["x"].zero_()
    common = dict(tol=case.get("tol", 1e-10), async_=bool(case.get("async")),
                  precision=ck.CK_PREC_MIXED if case.get("mixed") else ck.CK_PREC_FP64,
                  max_iter=case.get("max_iter", 100_000), config=state["cfg"])
    if kind == "cg":
        ck.cg_solve(state["M"].handle, state["b"], state["x"], **common)
    else:
        ck.gmres_solve(state["M"].handle, state["b"], state["x"], restart=30, **common)
    return state["x"]


# ---- what a pass cannot do without ----------------------------------------------

def _counts(family, n, case):
    """(rows, expected entries)."""
    if family == "banded":
        return n, n * case["points"]
    if family == "blocks":
        return n, 8 * n
    if family == "powerlaw":
        k, p = _zipf(case["s"], min(RMAX, n))
        return n, int(n * float((k * p).sum()))
    if family == "uniform":
        return n, 34 * n
    if family == "dominant":
        return n, 19 * n
    rows = n ** 3 if family == "lap3d" else n * n
    return rows, (7 if family == "lap3d" else 5) * rows


def work(case):
    kind = case["kind"]
    if kind == "serve":
        n = case["n"]
        one = sum(a * b for a, b in ((5, 1.25), (19, 2.3))) * n * 12 / 6
        return {"bytes": case["requests"] * one, "flops": case["requests"] * 100 * 2 * 12 * n}
    n, nnz = _counts(case["family"], case["n"], case)
    s = 4 if case.get("fp32") else 8
    # the values and, unless the diagonals say where they are, the columns
    entries = nnz * s if case["family"] == "banded" else nnz * (s + 4) + 4 * n
    once = {"bytes": entries + 2 * s * n, "flops": 2 * nnz}
    if kind == "product":
        return once
    if kind == "residual":
        return {"bytes": once["bytes"] + s * n, "flops": 2 * nnz}
    if kind == "prepare":   # the CSR arrays in, the copies and y out
        return {"bytes": 2 * (12 * nnz + 4 * n) + 16 * n, "flops": 2 * nnz}
    if kind == "cg":        # 3.3 N steps of a stencil system, each over five vectors
        its = 3.3 * case["n"]
        small = n <= 4096   # held on the chip for the whole solve
        stencil = 8 * nnz + 10 * 8 * n
        return {"bytes": (1 if small else its) * stencil, "flops": its * (2 * nnz + 10 * n)}
    if case["family"] == "convdiff":   # two sweeps of the basis for each step
        its, step = case["max_iter"], 8 * nnz + 8 * n * (2 * 16 + 11)
        return {"bytes": its * step, "flops": its * (2 * nnz + 8 * 16 * n)}
    return {"bytes": 20 * (nnz * 8 + 4 * n * 31), "flops": 20 * (2 * nnz + 8 * 10 * n)}


# ---- the same in 64 bits ---------------------------------------------------------

def _gmres(A, b, max_iter, m=30):
    """Restarted GMRES, modified Gram-Schmidt, from zero."""
    x, done = torch.zeros_like(b), 0
    while done < max_iter:
        r = b - _product(A, x)
        beta = float(r.norm())
        V, H = [r / beta], np.zeros((m + 1, m))
        for j in range(min(m, max_iter - done)):
            w = _product(A, V[j])
            for i, v in enumerate(V):
                H[i, j] = float(torch.dot(v, w))
                w = w - H[i, j] * v
            H[j + 1, j] = float(w.norm())
            V.append(w / H[j + 1, j])
            done += 1
        k = len(V) - 1
        e = np.zeros(k + 1)
        e[0] = beta
        y = np.linalg.lstsq(H[:k + 1, :k], e, rcond=None)[0]
        for v, c in zip(V, y):
            x = x + float(c) * v
    return x


def exact(case, seed):
    A, vectors = _inputs(case, seed)
    kind = case["kind"]
    if kind == "serve":
        return vectors                    # b was made from them
    if kind in ("cg", "gmres"):
        return _gmres(A, _product(A, vectors[0]), case["max_iter"]) if "max_iter" in case \
            else vectors[0]
    if case.get("fp32"):
        return _product((A[0], A[1], A[2].float().double()), vectors[0].float().double())
    y = _product(A, vectors[0])
    if kind == "residual":
        return vectors[1] - y
    return {"y": y, "features": None} if kind == "prepare" else y
