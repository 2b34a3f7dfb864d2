"""GPU tests of the construction on the device: for every matrix, chunk height and sorting
window, the device-built SELL-C-sigma arrays (permutation, chunk lengths and starts, columns,
values in the storage type) equal the host builder's bit for bit, the host builder's layout
itself being pinned to the oracle's brute-force layout; invalid input is rejected."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import abs_product, colwise_relerr, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import torch

    import paper_1507_08101_amd as sc

    assert torch.cuda.is_available()
    sc.lib()
    return sc


def _mats():
    return {
        "empty": synth.CSR(0, 0, np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0), "empty"),
        "one": synth.CSR(1, 1, np.array([0, 1], np.int64), np.zeros(1, np.int32), np.array([2.5]), "one"),
        "lap2d_64": synth.laplacian2d(64),
        "anderson_12": synth.anderson3d(12),
        "irregular_20000": synth.irregular(20000, band=1000, max_len=700, seed=71),
        "random_ragged": synth.random_sparse(333, 257, 0.03, 72, empty_rows=17, long_row=257, duplicates=True),
        "zero_rows": synth.CSR(50, 10, np.zeros(51, np.int64), np.zeros(0, np.int32), np.zeros(0), "zero_rows"),
    }


MATS = _mats()


def _dev_csr(A):
    import torch

    return (torch.from_numpy(np.ascontiguousarray(A.rowptr, dtype=np.int64)).cuda(),
            torch.from_numpy(np.ascontiguousarray(A.col, dtype=np.int32)).cuda(),
            torch.from_numpy(np.ascontiguousarray(A.val, dtype=np.float64)).cuda())


@pytest.mark.parametrize("name", list(MATS))
@pytest.mark.parametrize("C,sigma", [(1, 1), (8, 1), (32, 1), (32, 32), (32, 1024), (64, 10 ** 9), (12, 7)])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_device_build_equals_host_build(sc, name, C, sigma, dt):
    A = MATS[name]
    Mh = sc.SellMatrix.from_csr(A, C=C, sigma=sigma, dtype=dt)
    rp, co, va = _dev_csr(A)
    Md = sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rp, co, va, C=C, sigma=sigma, dtype=dt)
    ih, idv = dict(Mh.info), dict(Md.info)
    assert ih == idv, (ih, idv)
    eh, ed = Mh.export_sell(), Md.export_sell()  # (perm, cl, cs, col, val)
    for k in range(5):
        assert np.array_equal(eh[k], ed[k]), k
    # and the layout is the oracle's
    perm, cl, cs = oracle.sell_layout(A, C, min(sigma, max(A.nrows, 1)))
    assert np.array_equal(ed[0], perm) and np.array_equal(ed[1], cl) and np.array_equal(ed[2], cs)
    # the CSR comes back bit for bit (values in the storage type)
    rp2, col2, val2 = Md.export_csr()
    assert np.array_equal(rp2, A.rowptr) and np.array_equal(col2, A.col)
    Mh.close()
    Md.close()


@pytest.mark.parametrize("b", [1, 8])
def test_device_built_matrix_products(sc, b):
    import torch

    A = MATS["irregular_20000"]
    rp, co, va = _dev_csr(A)
    M = sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rp, co, va, C=32, sigma=256)
    X = synth.block_vector(A.ncols, b, 73)
    Y = torch.zeros((A.nrows, b), dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv(M, dev(X), Y)
    assert colwise_relerr(host(Y), oracle.spmmv(A, X), abs_product(A, X)) <= 1e-12
    # values-only update and the transposed product work on a device-built matrix
    newv = synth.uniform(74, A.nnz, -1, 1)
    M.update_values(dev(newv))
    A2 = synth.CSR(A.nrows, A.ncols, A.rowptr, A.col, newv)
    sc.sell_spmmv(M, dev(X), Y)
    assert colwise_relerr(host(Y), oracle.spmmv(A2, X), abs_product(A2, X)) <= 1e-12
    XT = synth.block_vector(A.nrows, b, 75)
    YT = torch.zeros((A.ncols, b), dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_T(M, dev(XT), YT, deterministic=True)
    assert colwise_relerr(host(YT), oracle.spmmv_T(A2, XT)) <= 1e-12
    M.close()


def test_device_build_rejects_invalid_csr(sc):
    A = MATS["random_ragged"]
    rp, co, va = _dev_csr(A)
    bad = co.clone()
    bad[5] = A.ncols  # column out of range
    with pytest.raises(sc.SellError):
        sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rp, bad, va)
    bad = co.clone()
    bad[-1] = -3
    with pytest.raises(sc.SellError):
        sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rp, bad, va)
    rpb = rp.clone()
    rpb[10] = rpb[12] + 1  # decreasing row pointers
    with pytest.raises(sc.SellError):
        sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rpb, co, va)
    rpb = rp.clone()
    rpb[0] = 1
    with pytest.raises(sc.SellError):
        sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rpb, co, va)
    # the library is still usable afterwards
    M = sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rp, co, va)
    M.close()


def test_device_build_full_size_anderson128(sc):
    """The benchmark's matrix (2,097,152 rows), with a sorting window: equal to the host build."""
    A = synth.anderson3d(128)
    rp, co, va = _dev_csr(A)
    for sigma in (1, 4096):
        Mh = sc.SellMatrix.from_csr(A, C=32, sigma=sigma)
        Md = sc.SellMatrix.from_device_csr(A.nrows, A.ncols, rp, co, va, C=32, sigma=sigma)
        eh, ed = Mh.export_sell(), Md.export_sell()
        for k in range(5):
            assert np.array_equal(eh[k], ed[k]), (sigma, k)
        Mh.close()
        Md.close()


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("shape,C,sigma", [("wide", 32, 1), ("tall", 12, 40), ("square", 32, 128)])
def test_device_transpose_equals_host_transpose(sc, shape, C, sigma, dt):
    """The update maps and the copy of A^T made on the device against the host's (which a failed
    device allocation falls back to, whichever of them fails): transposed products before and after
    a value update, and value gradients, bit for bit; empty rows and columns, duplicates, one long row
    and one long column."""
    import torch

    nr, nc = {"wide": (90, 401), "tall": (530, 77), "square": (300, 300)}[shape]
    A = synth.random_sparse(nr, nc, 0.03, 210, duplicates=True, empty_rows=7, long_row=60)
    col = A.col.copy()
    col[:: 5] = 3  # a long column; the columns it leaves empty stay so
    A = synth.CSR(nr, nc, A.rowptr, col, A.val)
    vt = torch.float64 if dt == "f64" else torch.float32
    b = 3
    X = torch.from_numpy(synth.block_vector(nr, b, 211)).to("cuda:0", vt)
    G = torch.from_numpy(synth.block_vector(nc, b, 212)).to("cuda:0", vt)
    newv = torch.from_numpy(synth.uniform(213, A.nnz, -2, 2)).cuda()

    def once(fail_at):
        M = sc.SellMatrix.from_csr(A, C=C, sigma=sigma, dtype=dt)
        outs = [torch.empty((nc, b), dtype=vt, device="cuda:0") for _ in range(2)]
        dval = torch.empty(A.nnz, dtype=torch.float64, device="cuda:0")
        sc.sell_debug_fail_alloc(fail_at)
        try:
            sc.sell_spmmv_T(M, X, outs[0])
        finally:
            sc.sell_debug_fail_alloc(0)
        M.update_values(newv)
        sc.sell_spmmv_T(M, X, outs[1])
        sc.sell_grad_values(M, X, G, dval)
        torch.cuda.synchronize()
        rp, c, v = M.export_csr()
        assert np.array_equal(rp, A.rowptr) and np.array_equal(c, A.col)
        M.close()
        return outs + [dval, torch.from_numpy(v)]

    want = once(0)
    ref = oracle.spmmv_T(A, X.double().cpu().numpy())
    scale = oracle.spmmv_T(synth.CSR(nr, nc, A.rowptr, A.col, np.abs(A.val)), np.abs(X.double().cpu().numpy()))
    tol = {"f64": 2.0 ** -46, "f32": 2.0 ** -17, "bf16": 2.0 ** -7}[dt]
    assert (np.abs(want[0].double().cpu().numpy() - ref) <= tol * scale + 1e-300).all()
    live = sc.sell_debug_live_allocs()
    for k in range(1, 30):
        got = once(k)
        assert all(torch.equal(u, v) for u, v in zip(got, want)), k
        assert sc.sell_debug_live_allocs() == live, k


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n,per_row,sigma", [(1, 1, 1), (256, 8, 1), (257, 8, 1), (700, 3, 1), (700, 30, 1), (700, 3, 64), (5000, 20, 4096)])
def test_value_update_equals_fresh_build(sc, n, per_row, sigma, dt):
    """A value update (workgroups of few and of many entries, rows in order and sorted) against a matrix
    built from the new values: its values, its product and that of its copy of A^T, bit for bit."""
    import torch

    A = synth.random_sparse(n, n, per_row / n, 214, empty_rows=min(5, n - 1), long_row=min(n, 400) if per_row > 8 else None)
    newv = synth.uniform(215, A.nnz, -2, 2)
    vt = torch.float64 if dt == "f64" else torch.float32
    X = torch.from_numpy(synth.block_vector(n, 2, 216)).to("cuda:0", vt)
    outs = []
    for first in (A.val, newv):
        M = sc.SellMatrix.from_csr(synth.CSR(n, n, A.rowptr, A.col, first), C=32, sigma=sigma, dtype=dt)
        Y, Z = torch.empty_like(X), torch.empty_like(X)
        if first is A.val:
            sc.sell_spmmv_T(M, X, Z)  # makes the copy of A^T, with the old values
            M.update_values(torch.from_numpy(newv).cuda())
        sc.sell_spmmv(M, X, Y)
        sc.sell_spmmv_T(M, X, Z)
        outs.append((Y, Z, torch.from_numpy(M.export_csr()[2])))
        M.close()
    assert all(torch.equal(u, v) for u, v in zip(*outs))


@pytest.mark.parametrize("dt", ["f64", "bf16"])
@pytest.mark.parametrize("nr,nc,length,sigma", [(3, 900, 800, 1), (257, 400, 65, 1), (600, 700, 250, 64), (300, 80, 9, 1)])
def test_value_update_of_long_rows(sc, nr, nc, length, sigma, dt):
    """Rows shared by several workgroups (some of a workgroup's 256 rows short, so that it deals them out
    through LDS): as a matrix built from the new values, and so its copy of A^T, bit for bit."""
    import torch

    A = synth.random_sparse(nr, nc, length / nc, 231, empty_rows=min(2, nr - 1))
    if nr > 512:  # a workgroup of short rows among those of long ones
        keep = np.ones(A.nnz, dtype=bool)
        keep[A.rowptr[256] + 40:A.rowptr[512]] = False
        rp = np.concatenate([[0], np.cumsum(np.add.reduceat(np.append(keep, 0).astype(np.int64), A.rowptr[:-1])
                                            * (np.diff(A.rowptr) > 0))])
        A = synth.CSR(nr, nc, rp, A.col[keep], A.val[keep])
    newv = synth.uniform(232, A.nnz, -2, 2)
    vt = torch.float64 if dt == "f64" else torch.float32
    X, Xt = (torch.from_numpy(synth.block_vector(m, 2, 233)).to("cuda:0", vt) for m in (nc, nr))
    outs = []
    for first in (A.val, newv):
        M = sc.SellMatrix.from_csr(synth.CSR(nr, nc, A.rowptr, A.col, first), C=32, sigma=sigma, dtype=dt)
        Y, Z = torch.empty_like(Xt), torch.empty_like(X)
        if first is A.val:
            M.update_values(torch.from_numpy(newv).cuda())  # no copy of A^T yet
            sc.sell_spmmv(M, X, Y)
            outs.append((Y.clone(),))
            M.update_values(torch.from_numpy(A.val).cuda())
            sc.sell_spmmv_T(M, Xt, Z)
            M.update_values(torch.from_numpy(newv).cuda())
        sc.sell_spmmv(M, X, Y)
        sc.sell_spmmv_T(M, Xt, Z)
        outs.append((Y, Z, torch.from_numpy(M.export_csr()[2])))
        M.close()
    assert torch.equal(outs[0][0], outs[1][0])
    assert all(torch.equal(u, v) for u, v in zip(outs[1], outs[2]))


@pytest.mark.parametrize("dt", ["f64", "bf16"])
@pytest.mark.parametrize("n,C,sigma", [(700, 32, 1), (700, 7, 64), (131, 32, 131)])
def test_device_steps_on_full_rows_and_columns(sc, n, C, sigma, dt):
    """A full row and a full column beside rows of one entry and empty ones (chunks whose entries several
    workgroups share): the device-built matrix is the host-built one entry for entry, and the transposed
    product, the row pointers (by the value gradient) and a value update hold."""
    import torch

    rows = np.concatenate([np.full(n - 2, 2), np.arange(n - 3)])
    cols = np.concatenate([np.arange(n - 2), np.full(n - 3, 5)])
    order = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=rp[1:])
    A = synth.CSR(n, n, rp, cols[order].astype(np.int32), synth.randint(234, rows.size, -3, 3).astype(np.float64))
    M = sc.SellMatrix.from_csr(A, C=C, sigma=sigma, dtype=dt)
    D = sc.SellMatrix.from_device_csr(n, n, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(A.col).cuda(),
                                      torch.from_numpy(A.val).cuda(), C=C, sigma=sigma, dtype=dt)
    for u, v in zip(sc.sell_export_sell(M.handle), sc.sell_export_sell(D.handle)):
        assert np.array_equal(u, v)
    vt = torch.float64 if dt == "f64" else torch.float32
    x, g = synth.int_block_vector(n, 3, 235), synth.int_block_vector(n, 3, 236)
    X, G = (torch.from_numpy(v).to("cuda:0", vt) for v in (x, g))
    newv = synth.randint(237, rows.size, -3, 3).astype(np.float64)
    Z, dval = torch.empty_like(X), torch.empty(A.nnz, dtype=torch.float64, device="cuda:0")
    for B in (M, D):
        sc.sell_spmmv_T(B, X, Z)
        assert np.array_equal(Z.double().cpu().numpy(), oracle.spmmv_T(A, x))
        sc.sell_grad_values(B, G, X, dval)
        assert np.array_equal(dval.cpu().numpy(), oracle.pattern_outer(A, g, x))
        B.update_values(torch.from_numpy(newv).cuda())
        sc.sell_spmmv_T(B, X, Z)
        assert np.array_equal(Z.double().cpu().numpy(), oracle.spmmv_T(synth.CSR(n, n, A.rowptr, A.col, newv), x))
        B.close()
