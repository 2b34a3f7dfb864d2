"""Workloads for timing the library: each case is one call, or one short sequence of calls, of a program that uses it.

Matrices are the families the library is tested and benchmarked on (2D and 3D Laplacians, the periodic 3D Anderson
Hamiltonian, an irregular matrix with lognormal row lengths), made on the GPU from a seed and built there. ``exact`` restates
each case in plain 64-bit torch operations on the CSR arrays.
"""
import math

import numpy as np
import torch

import paper_1507_08101_amd as sc
from paper_1507_08101_amd.autograd import chebyshev, spmm

DEV = "cuda"
VALUE_BYTES = {"f64": 8, "f32": 4, "bf16": 2}
TORCH_DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
ANDERSON_W = 16.5
ANDERSON_S = (6.0 + ANDERSON_W / 2) / 0.99  # Gershgorin half-width of the spectrum, with a margin


def listed():
    return [
        # the smallest call a solver makes: a 64 x 64 grid, one vector, with the two dots of a CG step
        dict(name="small_lap2d_64_f64_b1", kind="product", matrix="lap2d", size=64, dtype="f64", b=1, sigma=1, op="dots"),
        # the KPM recurrence on the benchmark's lattice, a block of 8 random vectors, 20 products
        dict(name="kpm_anderson_128_b8", kind="kpm", matrix="anderson", size=128, dtype="f64", b=8, sigma=1, steps=20),
        # scattered columns and uneven rows: a graph-like matrix with sorted windows, 8 vectors
        dict(name="product_irregular_4m_f64_b8", kind="product", matrix="irregular", size=4_000_000, dtype="f64", b=8,
             sigma=1024, op="plain"),
        # a block whose width is no power of two, every augmentation at once (per-column shifts, axpby, chain, dots)
        dict(name="aug_anderson_96_f64_b12", kind="product", matrix="anderson", size=96, dtype="f64", b=12, sigma=1,
             op="chain"),
        # three coupled components (a vector field) on a 3D grid, single precision
        dict(name="product_lap3d_100_f32_b3", kind="product", matrix="lap3d", size=100, dtype="f32", b=3, sigma=1, op="dots"),
        # a polynomial filter on 16 vectors in single precision, 40 steps with the chained accumulation
        dict(name="filter_anderson_96_f32_b16", kind="filter", matrix="anderson", size=96, dtype="f32", b=16, sigma=1,
             steps=40),
        # one linear system with 8 right-hand sides, BF16 values refined in FP64
        dict(name="cg_mixed_lap3d_48_bf16_b8", kind="cg_mixed", size=48, dtype="bf16", b=8, tol=1e-12),
        # many independent systems of uneven sizes solved together
        dict(name="batch_cg_16_lap3d_f64_b4", kind="batch_cg", count=16, lo=20, hi=48, b=4, tol=1e-12),
        # one training step through the degree-100 Chebyshev filter (forward and backward, values as parameters)
        dict(name="cheb_step_anderson_64_f64_b1", kind="cheb", matrix="anderson", size=64, dtype="f64", b=1, sigma=1,
             degree=100, every=10),
        # one training step through a sparse layer with 8 features (forward and backward, values as parameters)
        dict(name="spmm_step_lap3d_100_f32_b8", kind="spmm", matrix="lap3d", size=100, dtype="f32", b=8, sigma=1),
        # a Rayleigh-Ritz step on a block of 32 vectors: projection, rotation into a second block, rotation in place
        dict(name="ritz_1m_m32_k32", kind="ritz", n=1_000_000, m=32, k=32, beta=0.0, kahan=False),
        # a column-major block from another library taken over row-major in single precision
        dict(name="copy_2m_col_f64_to_row_f32_b8", kind="copy", n=2_097_152, b=8, src="f64", dst="f32", src_col=True,
             dst_col=False),
    ]


def draw(rng):
    """One more case of the same ranges."""

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def matrix(most):
        # a matrix of up to `most` rows: any of the four families, windows sorted where rows are uneven
        m = rng.choice(["lap2d", "lap3d", "anderson", "irregular"])
        n = log_int(3000, max(4000, most))
        if m == "lap2d":
            return dict(matrix=m, size=max(16, int(n ** 0.5)), sigma=1)
        if m in ("lap3d", "anderson"):
            return dict(matrix=m, size=max(8, int(round(n ** (1 / 3)))), sigma=1)
        return dict(matrix=m, size=n, sigma=rng.choice([1, 256, 1024]))

    kind = rng.choice(["product", "product", "product", "kpm", "filter", "cg_mixed", "batch_cg", "cheb", "spmm", "ritz", "copy"])
    dt = rng.choice(["f64", "f64", "f32", "bf16"])
    if kind == "product":
        b = rng.choice([1, 2, 4, 8, 16, 32, log_int(1, 64), log_int(1, 64), log_int(3, 64)])
        return dict(kind=kind, dtype=dt, b=b, op=rng.choice(["plain", "dots", "kpm", "chain"]), **matrix(24_000_000 // (b + 4)))
    if kind == "kpm":
        b = rng.choice([1, 4, 8, log_int(1, 32)])
        return dict(kind=kind, matrix="anderson", size=rng.randint(12, int((8_000_000 / (b + 2)) ** (1 / 3))), dtype="f64", b=b,
                    sigma=1, steps=rng.randint(5, 40))
    if kind == "filter":
        b = log_int(1, 64)
        return dict(kind=kind, matrix="anderson", size=rng.randint(12, int((12_000_000 / (b + 2)) ** (1 / 3))), dtype=dt, b=b,
                    sigma=1, steps=rng.randint(5, 40))
    if kind == "cg_mixed":
        return dict(kind=kind, size=rng.randint(10, 48), dtype=rng.choice(["f32", "bf16"]), b=log_int(1, 16), tol=1e-12)
    if kind == "batch_cg":
        lo = rng.randint(8, 24)
        return dict(kind=kind, count=rng.randint(3, 16), lo=lo, hi=rng.randint(lo + 2, 40), b=log_int(1, 8), tol=1e-12)
    if kind == "cheb":
        b = log_int(1, 8)
        return dict(kind=kind, matrix="anderson", size=rng.randint(8, int((400_000 / (b + 0.5)) ** (1 / 3))),
                    dtype=rng.choice(["f64", "f32"]), b=b, sigma=1, degree=rng.randint(10, 100), every=rng.randint(3, 20))
    if kind == "spmm":
        b = log_int(1, 64)
        return dict(kind=kind, dtype=rng.choice(["f64", "f32"]), b=b, **matrix(8_000_000 // (b + 7)))
    if kind == "ritz":
        m, k = log_int(1, 64), log_int(1, 64)
        return dict(kind=kind, n=log_int(1000, 64_000_000 // (m + k + 4)), m=m, k=k, beta=rng.choice([0.0, 0.5]),
                    kahan=rng.random() < 0.25)
    b = log_int(1, 64)
    src, dst = rng.choice([("f64", "f64"), ("f64", "f32"), ("f32", "f64"), ("f32", "f32"), ("f64", "bf16"), ("f32", "bf16"),
                           ("bf16", "f32")])
    cols = rng.choice([(True, False), (False, True), (False, False)])
    if src == dst and cols[0] == cols[1]:
        dst = "f32" if src == "f64" else "f64"
    return dict(kind="copy", n=log_int(2000, 32_000_000 // (b + 1)), b=b, src=src, dst=dst, src_col=cols[0], dst_col=cols[1])


# ------------------------------------------------------------------------------------------------- inputs


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _uniform(g, *shape, dtype=torch.float64):
    return torch.rand(*shape, dtype=dtype, device=DEV, generator=g) * 2 - 1


def _stencil(dims, periodic, diag, off):
    """Nearest-neighbour stencil on a grid (first dimension fastest), columns sorted within a row: (rowptr, col, val)."""
    n = math.prod(dims)
    idx = torch.arange(n, dtype=torch.int64, device=DEV)
    cols, live, vals = [idx], [torch.ones_like(idx, dtype=torch.bool)], [diag]
    stride = 1
    for d in dims:
        at = (idx // stride) % d
        for step in (-1, 1):
            to = at + step
            live.append(torch.ones_like(live[0]) if periodic else (to >= 0) & (to < d))
            cols.append(idx + (to % d - at) * stride)
            vals.append(torch.full_like(diag, off))
        stride *= d
    col = torch.where(torch.stack(live, 1), torch.stack(cols, 1), n)
    col, order = col.sort(dim=1)
    val = torch.stack(vals, 1).gather(1, order)
    keep = col < n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(keep.sum(1), 0, out=rowptr[1:])
    return rowptr, col[keep].to(torch.int32), val[keep]


def _irregular(n, g):
    """Lognormal row lengths of mean 15, half of a row's columns within 5000 rows of it, half anywhere, values N(0, 1)."""
    z = torch.randn(n, dtype=torch.float64, device=DEV, generator=g)
    lens = (math.log(15.0) - 0.5 + z).exp().round().clamp(1, min(2000, n)).to(torch.int64)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=rowptr[1:])
    row = torch.repeat_interleave(torch.arange(n, device=DEV), lens)
    nnz = row.numel()
    near = torch.arange(nnz, device=DEV) - rowptr[row] < (lens[row] + 1) // 2
    w = min(5000, n - 1)
    band = (row + torch.randint(-w, w + 1, (nnz,), device=DEV, generator=g)).abs()
    band = torch.where(band >= n, 2 * (n - 1) - band, band)
    col = torch.where(near, band, torch.randint(0, n, (nnz,), device=DEV, generator=g))
    col = (row * n + col).sort().values % n
    return rowptr, col.to(torch.int32), torch.randn(nnz, dtype=torch.float64, device=DEV, generator=g)


def _csr(case, g):
    """CSR arrays with values that the case's value type holds exactly."""
    m, size = case["matrix"], case["size"]
    if m == "irregular":
        rowptr, col, val = _irregular(size, g)
    elif m == "anderson":
        eps = _uniform(g, size ** 3) * (ANDERSON_W / 2)
        rowptr, col, val = _stencil((size,) * 3, True, eps, -1.0)
    else:
        d = 2 if m == "lap2d" else 3
        diag = torch.full((size ** d,), 2.0 * d, dtype=torch.float64, device=DEV)
        rowptr, col, val = _stencil((size,) * d, False, diag, -1.0)
    return rowptr, col, val.to(TORCH_DT[case["dtype"]]).to(torch.float64)


def _laplacian(edge):
    diag = torch.full((edge ** 3,), 6.0, dtype=torch.float64, device=DEV)
    return _stencil((edge,) * 3, False, diag, -1.0)


def _build(csr, dtype, sigma=1):
    rowptr, col, val = csr
    n = rowptr.numel() - 1
    return sc.SellMatrix.from_device_csr(n, n, rowptr, col, val, C=32, sigma=sigma, dtype=dtype)


def _vec_dt(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _opts(case):
    """Augmentation options of a product case."""
    b = case["b"]
    return {"plain": dict(),
            "dots": dict(flags=sc.DOT_YY | sc.DOT_XY),
            "kpm": dict(flags=sc.SHIFT | sc.SCALE | sc.AXPBY | sc.DOT_YY | sc.DOT_XY, alpha=2.0 / 14.4, gamma=0.1, beta=-0.9),
            "chain": dict(flags=sc.VSHIFT | sc.SCALE | sc.AXPBY | sc.DOTS | sc.CHAIN, alpha=1.0 / 14.4, beta=-0.5,
                          gamma_v=np.linspace(-0.5, 0.5, b), delta=0.5, eta=0.25)}[case["op"]]


def _coef(case):
    m = np.arange(case["steps"] + 1)
    return np.exp(-0.1 * m) * np.cos(0.3 * m)


def _edges(case):
    c, lo, hi = case["count"], case["lo"], case["hi"]
    return [lo + (i * 7919 + 13) % (hi - lo + 1) for i in range(c)]


def _rotation(m, seed):
    q, _ = np.linalg.qr(np.random.default_rng(int(seed) % (1 << 62)).standard_normal((m, m)))
    return torch.from_numpy(np.ascontiguousarray(q)).to(DEV)


def _inputs(case, seed):
    """The numbers of a case, from the seed alone: shared by the timed path and its exact restatement."""
    g, kind = _gen(seed), case["kind"]
    b = case.get("b", 1)
    if kind == "ritz":
        n, m, k = case["n"], case["m"], case["k"]
        return dict(V=_uniform(g, n, m) / math.sqrt(n), W=_uniform(g, n, k) / math.sqrt(n),
                    Y=_uniform(g, m, k) / math.sqrt(m), Q=_rotation(m, seed))
    if kind == "copy":
        src = _uniform(g, case["b"], case["n"]).to(TORCH_DT[case["src"]])
        return dict(src=src.t() if case["src_col"] else src.t().contiguous())
    if kind == "cg_mixed":
        csr = _laplacian(case["size"])
        x = _uniform(g, csr[0].numel() - 1, b)
        return dict(csr=csr, x=x, rhs=_mul(csr, x))
    if kind == "batch_cg":
        csrs = [_laplacian(e) for e in _edges(case)]
        xs = [_uniform(g, c[0].numel() - 1, b) for c in csrs]
        return dict(csrs=csrs, x=torch.cat(xs), rhs=torch.cat([_mul(c, x) for c, x in zip(csrs, xs)]))
    csr = _csr(case, g)
    n, dt = csr[0].numel() - 1, _vec_dt(case)
    d = dict(csr=csr, X=_uniform(g, n, b, dtype=dt))
    if kind == "product":
        d["Y"], d["Z"] = _uniform(g, n, b, dtype=dt), _uniform(g, n, b, dtype=dt)
    elif kind in ("cheb", "spmm"):
        d["G"] = _uniform(g, n, b, dtype=dt)
    return d


def prepare(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    s = dict(case=case, **{k: v for k, v in d.items() if k not in ("csr", "csrs", "x")})
    if kind == "copy":
        n, b = d["src"].shape
        dt = TORCH_DT[case["dst"]]
        s["dst"] = torch.empty(b, n, dtype=dt, device=DEV).t() if case["dst_col"] else torch.empty(n, b, dtype=dt, device=DEV)
        return s
    if kind == "ritz":
        s["G"] = torch.empty(case["m"], case["k"], dtype=torch.float64, device=DEV)
        return s
    if kind == "cg_mixed":
        s["A"], s["lo"] = _build(d["csr"], "f64"), _build(d["csr"], case["dtype"])
        return s
    if kind == "batch_cg":
        s["A"] = sc.SellBatch([_build(c, "f64") for c in d["csrs"]])
        return s
    s["A"] = _build(d["csr"], case["dtype"], case["sigma"])
    b = case["b"]
    if kind == "product":
        s["opts"] = _opts(case)
        s["dot"] = torch.zeros(3 * b, dtype=torch.float64, device=DEV)
    elif kind == "kpm":
        s["V"], s["W"] = torch.empty_like(d["X"]), torch.empty_like(d["X"])
        s["mu"] = torch.empty((2 * case["steps"] + 1) * b, dtype=torch.float64, device=DEV)
    elif kind == "filter":
        s["coef"] = _coef(case)
    elif kind in ("cheb", "spmm"):
        s["theta"] = d["csr"][2].clone().requires_grad_(True)
        s["X"] = d["X"].requires_grad_(True)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "product":
        if case["op"] == "plain":
            sc.sell_spmmv(s["A"], s["X"], s["Y"])
            return [s["Y"]]
        sc.sell_spmmv_aug(s["A"], s["X"], s["Y"], s["Z"], dot=s["dot"], **s["opts"])
        return [s["Y"], s["Z"], s["dot"]] if case["op"] == "chain" else [s["Y"], s["dot"]]
    if kind == "kpm":
        s["V"].copy_(s["X"])  # the recurrence overwrites its starting block
        sc.sell_kpm(s["A"], s["V"], s["W"], case["steps"], ANDERSON_S, 0.0, s["mu"])
        return [s["V"], s["W"], s["mu"]]
    if kind == "filter":
        return sc.sell_cheb_filter(s["A"], s["X"], s["coef"], ANDERSON_S, 0.0)
    if kind == "cg_mixed":
        x = torch.zeros_like(s["rhs"])
        sc.sell_cg_mixed(s["A"], s["lo"], s["rhs"], x, tol=case["tol"])
        return x
    if kind == "batch_cg":
        x = torch.zeros_like(s["rhs"])
        sc.sell_batch_cg(s["A"], None, s["rhs"], x, tol=case["tol"])
        return x
    if kind in ("cheb", "spmm"):
        s["theta"].grad = s["X"].grad = None
        if kind == "cheb":
            y = chebyshev(s["theta"], s["X"], s["A"], case["degree"], ANDERSON_S, 0.0, case["every"])
        else:
            y = spmm(s["theta"], s["X"], s["A"])
        y.backward(s["G"])
        return [y, s["theta"].grad, s["X"].grad]
    if kind == "ritz":
        sc.sell_tsmttsm(s["V"], s["W"], s["G"], kahan=case["kahan"])
        sc.sell_tsmm(s["V"], s["Y"], s["W"], beta=case["beta"])
        sc.sell_tsmm_inplace(s["V"], s["Q"])
        return [s["G"], s["W"], s["V"]]
    sc.sell_bv_copy(s["dst"], s["src"])
    return s["dst"]


# ------------------------------------------------------------------------------------------------- 64 bits


def _rows(csr):
    return torch.repeat_interleave(torch.arange(csr[0].numel() - 1, device=DEV), csr[0].diff())


def _mul(csr, x):
    """A x column by column: gather, multiply, add up by row (in a fixed order)."""
    rowptr, col, val = csr[0], csr[1].to(torch.int64), csr[2]
    y = torch.empty_like(x)
    for j in range(x.shape[1]):
        y[:, j] = torch.segment_reduce(val * x[col, j], "sum", lengths=rowptr.diff())
    return y


def _mul_t(csr, x):
    """A^T x column by column."""
    row, col = _rows(csr), csr[1].to(torch.int64)
    y = torch.zeros_like(x)
    for j in range(x.shape[1]):
        y[:, j].index_add_(0, col, csr[2] * x[row, j])
    return y


def exact(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    if kind in ("cg_mixed", "batch_cg"):
        return d["x"]
    if kind == "copy":
        return d["src"].to(torch.float64)
    if kind == "ritz":
        W = d["V"] @ d["Y"] + case["beta"] * d["W"]
        return [d["V"].t() @ d["W"], W, d["V"] @ d["Q"]]
    csr, X = d["csr"], d["X"].to(torch.float64)
    if kind == "product":
        y = _mul(csr, X)
        if case["op"] == "plain":
            return [y]
        o = _opts(case)
        fl = o["flags"]
        shift = o.get("gamma", 0.0) if fl & sc.SHIFT else 0.0
        if fl & sc.VSHIFT:
            shift = torch.from_numpy(o["gamma_v"]).to(DEV)
        y = o.get("alpha", 1.0) * (y - shift * X)
        if fl & sc.AXPBY:
            y = y + o["beta"] * d["Y"].to(torch.float64)
        zero = torch.zeros(case["b"], dtype=torch.float64, device=DEV)
        dot = torch.cat([(y * y).sum(0), (X * y).sum(0), (X * X).sum(0) if fl & sc.DOT_XX else zero])
        if fl & sc.CHAIN:
            return [y, o["delta"] * d["Z"].to(torch.float64) + o["eta"] * y, dot]
        return [y, dot]
    if kind == "spmm":
        G = d["G"].to(torch.float64)
        row, col = _rows(csr), csr[1].to(torch.int64)
        dtheta = torch.zeros_like(csr[2])
        for j in range(X.shape[1]):
            dtheta += G[row, j] * X[col, j]
        return [_mul(csr, X), dtheta, _mul_t(csr, G)]
    # the Chebyshev recurrences: 7 entries in every row of the Anderson matrix
    n = X.shape[0]
    col, val = csr[1].to(torch.int64).view(n, 7), csr[2].view(n, 7)

    def scaled(v, t):
        return sum(t[:, k, None] * v[col[:, k]] for k in range(7)) / ANDERSON_S

    if kind == "filter":
        c = _coef(case)
        a, v = X, scaled(X, val)
        z = c[0] * a + c[1] * v
        for m in range(2, case["steps"] + 1):
            a, v = v, 2 * scaled(v, val) - a
            z = z + c[m] * v
        return z
    if kind == "kpm":
        M = case["steps"]
        a, v = X, scaled(X, val)
        mu0, mu1 = (a * a).sum(0), (a * v).sum(0)
        mu = [mu0, mu1, 2 * (v * v).sum(0) - mu0]
        for _ in range(1, M):
            a, v = v, 2 * scaled(v, val) - a
            mu += [2 * (a * v).sum(0) - mu1, 2 * (v * v).sum(0) - mu0]
        last = [v, a] if M % 2 == 0 else [a, v]  # v_M ends in W after an odd number of products
        return last + [torch.cat(mu)]
    t, x = val.clone().requires_grad_(True), X.clone().requires_grad_(True)
    a, v = x, scaled(x, t)
    for _ in range(1, case["degree"]):
        a, v = v, 2 * scaled(v, t) - a
    v.backward(d["G"].to(torch.float64))
    return [v.detach(), t.grad.reshape(-1), x.grad]


# ------------------------------------------------------------------------------------------------- work


def _shape(case):
    """(rows, nonzeros) of the case's matrix."""
    m, e = case["matrix"], case["size"]
    if m == "lap2d":
        return e * e, 5 * e * e - 4 * e
    if m == "lap3d":
        return e ** 3, 7 * e ** 3 - 6 * e * e
    if m == "anderson":
        return e ** 3, 7 * e ** 3
    return e, 15 * e


def _product_bytes(n, nnz, b, dtype, vectors):
    v = 8 if dtype == "f64" else 4
    return nnz * (VALUE_BYTES[dtype] + 4) + vectors * n * b * v


def work(case):
    kind, b = case["kind"], case.get("b", 1)
    if kind == "copy":
        return dict(bytes=case["n"] * b * (VALUE_BYTES[case["src"]] + VALUE_BYTES[case["dst"]]), flops=0)
    if kind == "ritz":
        n, m, k = case["n"], case["m"], case["k"]
        return dict(bytes=8 * n * (m + k + m + k * (2 if case["beta"] else 1) + 2 * m), flops=2 * n * m * (2 * k + m))
    if kind in ("cg_mixed", "batch_cg"):
        # about 5 iterations per grid point along an edge for the tolerance asked for; an iteration reads the matrix, makes
        # q from p and updates r, x and p
        total_b = total_f = 0
        dt = case.get("dtype", "f64")
        for e in [case["size"]] if kind == "cg_mixed" else _edges(case):
            n, nnz, its = e ** 3, 7 * e ** 3 - 6 * e * e, 5 * e
            total_b += its * _product_bytes(n, nnz, b, dt, 9)
            total_f += its * (2 * nnz + 10 * n) * b
        return dict(bytes=total_b, flops=total_f)
    n, nnz = _shape(case)
    dt = case["dtype"]
    if kind == "product":
        vectors = {"plain": 2, "dots": 2, "kpm": 3, "chain": 5}[case["op"]]
        return dict(bytes=_product_bytes(n, nnz, b, dt, vectors), flops=2 * nnz * b)
    if kind == "kpm":
        return dict(bytes=case["steps"] * _product_bytes(n, nnz, b, dt, 3), flops=case["steps"] * 2 * nnz * b)
    if kind == "filter":
        return dict(bytes=case["steps"] * _product_bytes(n, nnz, b, dt, 5), flops=case["steps"] * 2 * nnz * b)
    if kind == "cheb":
        # forward, recomputation and adjoint products, and a gradient that reads two vectors a step and is written once
        N = case["degree"]
        return dict(bytes=3 * N * _product_bytes(n, nnz, b, dt, 3) + 8 * nnz, flops=8 * N * nnz * b)
    # spmm: values in (theta read, stored twice), A x, A^T g, the gradient of the values
    v = 8 if dt == "f64" else 4
    return dict(bytes=8 * nnz + 2 * VALUE_BYTES[dt] * nnz + 2 * _product_bytes(n, nnz, b, dt, 2) + 12 * nnz + 2 * n * b * v,
                flops=6 * nnz * b)
