"""GPU parity of the HIP path (called through the C ABI) against the CPU oracle.

FP64 bar: per-column normwise relative error <= 1e-12; integer-valued inputs (exact in
every order of summation) must agree bit for bit; dots within 1e-12 * sum |x_i y_i|.
"""
import math

import numpy as np
import pytest

import oracle
import synth
from gpu_util import abs_product, assert_lowprec_product, colwise_relerr, dev, host, to_oracle_flags

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def sc():
    import torch

    import paper_1507_08101_amd as sc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sc.lib()
    return sc


def _mats():
    return {
        "lap2d_64": synth.laplacian2d(64),
        "anderson_12": synth.anderson3d(12),
        "irregular_5000": synth.irregular(5000, band=300, max_len=2000, seed=21),
        "random_ragged": synth.random_sparse(333, 333, 0.03, 22, empty_rows=17, long_row=333),
        "rect_270x190": synth.random_sparse(270, 190, 0.05, 23, empty_rows=5),
    }


MATS = _mats()


def _plain_case(sc, A, C, sigma, b, dt="f64"):
    import torch

    X = synth.block_vector(A.ncols, b, synth.SEED_X)
    M = sc.SellMatrix.from_csr(A, C=C, sigma=sigma, dtype=dt)
    Xd = dev(X)
    Yd = torch.full((A.nrows, b), float("nan"), dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv(M, Xd, Yd)
    got = host(Yd)
    M.close()
    return X, got


@pytest.mark.parametrize("name", list(MATS))
@pytest.mark.parametrize("C,sigma", [(1, 1), (8, 1), (32, 1), (32, 32), (32, 1024), (64, 1), (64, 10 ** 9),
                                     (12, 7)])
def test_spmmv_f64_matrix_shapes(sc, name, C, sigma):
    A = MATS[name]
    for b in (1, 3, 8):
        X, got = _plain_case(sc, A, C, sigma, b)
        ref = oracle.spmmv(A, X)
        assert colwise_relerr(got, ref, abs_product(A, X)) <= TOL, (name, C, sigma, b)


@pytest.mark.parametrize("b", [1, 2, 3, 4, 5, 8, 16, 17, 32, 40, 64, 70, 100])
def test_spmmv_f64_block_widths(sc, b):
    A = MATS["irregular_5000"]
    X, got = _plain_case(sc, A, 32, 256, b)
    ref = oracle.spmmv(A, X)
    assert colwise_relerr(got, ref, abs_product(A, X)) <= TOL, b


@pytest.mark.parametrize("b", [1, 4, 8, 32])
def test_spmmv_integer_inputs_bit_exact(sc, b):
    import torch

    A0 = MATS["random_ragged"]
    A = synth.CSR(A0.nrows, A0.ncols, A0.rowptr, A0.col, np.rint(8 * A0.val), "int")
    X = synth.int_block_vector(A.ncols, b, 5)
    for C, sigma in [(32, 1), (64, 333), (5, 10)]:
        M = sc.SellMatrix.from_csr(A, C=C, sigma=sigma)
        Yd = torch.zeros((A.nrows, b), dtype=torch.float64, device="cuda:0")
        sc.sell_spmmv(M, dev(X), Yd)
        assert np.array_equal(host(Yd), oracle.spmmv(A, X)), (C, sigma)
        M.close()


def test_spmmv_deterministic(sc):
    import torch

    A = MATS["irregular_5000"]
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1024)
    X = dev(synth.block_vector(A.ncols, 8, 3))
    Y1 = torch.empty((A.nrows, 8), dtype=torch.float64, device="cuda:0")
    Y2 = torch.empty_like(Y1)
    d1 = torch.zeros(24, dtype=torch.float64, device="cuda:0")
    d2 = torch.zeros_like(d1)
    sc.sell_spmmv_aug(M, X, Y1, flags=sc.DOTS | sc.SHIFT, gamma=0.7, dot=d1)
    sc.sell_spmmv_aug(M, X, Y2, flags=sc.DOTS | sc.SHIFT, gamma=0.7, dot=d2)
    torch.cuda.synchronize()
    assert torch.equal(Y1, Y2) and torch.equal(d1, d2)
    M.close()


# ------------------------------------------------------------------ augmented product


def _aug_case(sc, A, b, flags, C=32, sigma=64, integer=False, **kw):
    import torch

    if integer:
        X = synth.int_block_vector(A.ncols, b, 31)
        Y0 = synth.int_block_vector(A.nrows, b, 32)
        Z0 = synth.int_block_vector(A.nrows, b, 33)
    else:
        X = synth.block_vector(A.ncols, b, synth.SEED_X)
        Y0 = synth.block_vector(A.nrows, b, synth.SEED_Y)
        Z0 = synth.block_vector(A.nrows, b, synth.SEED_Y + 7)
    M = sc.SellMatrix.from_csr(A, C=C, sigma=sigma)
    Xd, Yd, Zd = dev(X), dev(Y0), dev(Z0)
    dot = torch.full((3 * b,), -7.0, dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_aug(M, Xd, Yd, Z=Zd, flags=flags, dot=dot, **kw)
    got_y, got_z, got_d = host(Yd), host(Zd), host(dot)
    M.close()
    ref_y, ref_z, ref_d = oracle.spmmv_aug(A, X, Y=Y0, Z=Z0, flags=to_oracle_flags(flags), **kw)
    return X, Y0, Z0, (got_y, got_z, got_d), (ref_y, ref_z, ref_d)


SCALARS = dict(alpha=0.5, beta=-2.0, gamma=0.25, gamma_v=None, delta=4.0, eta=-0.5)


@pytest.mark.parametrize("flags", list(range(256)))
def test_aug_every_flag_combination_bit_exact_on_integers(sc, flags):
    A0 = MATS["random_ragged"]
    A = synth.CSR(A0.nrows, A0.ncols, A0.rowptr, A0.col, np.rint(8 * A0.val), "int")
    b = 4
    kw = dict(SCALARS)
    kw["gamma_v"] = np.array([1.0, -2.0, 0.5, 0.0])
    X, Y0, Z0, got, ref = _aug_case(sc, A, b, flags, integer=True, **kw)
    assert np.array_equal(got[0], ref[0]), flags
    if flags & 0x80:
        assert np.array_equal(got[1], ref[1]), flags
    else:
        assert np.array_equal(got[1], Z0)  # untouched
    for g, bit in enumerate((0x10, 0x20, 0x40)):
        seg = slice(g * b, (g + 1) * b)
        if flags & bit:
            assert np.array_equal(got[2][seg], ref[2][seg]), (flags, g)
        else:
            assert np.all(got[2][seg] == -7.0), (flags, g)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("b", [1, 2, 4, 8, 16, 32])
def test_cg_product_flags_low_precision(sc, dt, b):
    """A CG iteration's product (only <y, y> and <x, y>) runs a compile-time copy of the FP32-vector
    kernels: its y is the plain product's bit for bit (no scale, shift or y input), and both dots
    match exact sums over the GPU's own y within the dot bound."""
    import torch

    A = MATS["random_ragged"]
    M = sc.SellMatrix.from_csr(A, C=32, sigma=64, dtype=dt)
    X = dev(synth.block_vector(A.ncols, b, 90 + b), torch.float32)
    Yp = torch.zeros((A.nrows, b), dtype=torch.float32, device="cuda:0")
    Ya = torch.full((A.nrows, b), 5.0, dtype=torch.float32, device="cuda:0")
    dot = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv(M, X, Yp)
    sc.sell_spmmv_aug(M, X, Ya, flags=sc.DOT_YY | sc.DOT_XY, dot=dot)
    yp, ya, x = host(Yp), host(Ya), host(X).astype(np.float64)
    M.close()
    assert np.array_equal(ya, yp), (dt, b)
    dg = host(dot)
    y64 = ya.astype(np.float64)
    for g, u in ((0, y64), (1, x)):
        for j in range(b):
            terms = (u[:, j] * y64[:, j]).tolist()
            assert abs(dg[g * b + j] - math.fsum(terms)) <= 1e-12 * math.fsum(abs(t) for t in terms), (dt, b, g, j)


@pytest.mark.parametrize("name,sigma", [("random_ragged", 64), ("irregular_5000", 1024), ("anderson_12", 1)])
@pytest.mark.parametrize("b", [4, 8, 16, 32])
def test_kpm_step_flags_bit_exact_on_integers(sc, name, sigma, b):
    """The KPM step's flag set (shift, scale, axpby, <y,y>, <x,y>) runs a compile-time copy of
    the FP64 kernel that takes each row's diagonal entry from its own x row instead of gathering
    it: bit-exact against the oracle on integer data for every width with 4 columns per lane, on
    permuted rows (sigma > 1), empty and long rows, and rows without a stored diagonal."""
    A0 = MATS[name]
    A = synth.CSR(A0.nrows, A0.ncols, A0.rowptr, A0.col, np.rint(8 * A0.val), "int")
    flags = sc.SHIFT | sc.SCALE | sc.AXPBY | sc.DOT_YY | sc.DOT_XY
    kw = dict(alpha=0.5, beta=-2.0, gamma=0.25, gamma_v=None, delta=0.0, eta=1.0)
    X, Y0, Z0, got, ref = _aug_case(sc, A, b, flags, C=32, sigma=sigma, integer=True, **kw)
    assert np.array_equal(got[0], ref[0]), (name, b)
    for g in (0, 1):
        seg = slice(g * b, (g + 1) * b)
        assert np.array_equal(got[2][seg], ref[2][seg]), (name, b, g)


@pytest.mark.parametrize("b", [1, 2, 3, 8, 32, 33])
@pytest.mark.parametrize("flags", [0x01 | 0x04 | 0x08 | 0x70, 0x02 | 0x08 | 0x80 | 0x10, 0xFF & ~0x01, 0x70])
def test_aug_random_inputs(sc, b, flags):
    A = MATS["anderson_12"]
    kw = dict(SCALARS)
    kw["gamma_v"] = synth.uniform(40, b, -1, 1)
    X, Y0, Z0, got, ref = _aug_case(sc, A, b, flags, C=32, sigma=1, **kw)
    # cancellation-safe scale: |alpha| (|A||x| + |gamma||x|) + |beta||y|
    scale = abs(kw["alpha"]) * (abs_product(A, X) + 1.0 * np.abs(X)) + abs(kw["beta"]) * np.abs(Y0)
    assert colwise_relerr(got[0], ref[0], scale) <= TOL
    if flags & 0x80:
        zscale = abs(kw["delta"]) * np.abs(Z0) + abs(kw["eta"]) * scale
        assert colwise_relerr(got[1], ref[1], zscale) <= TOL
    yref = ref[0]
    bounds = [np.sum(yref * yref, axis=0), np.sum(np.abs(X * yref), axis=0), np.sum(X * X, axis=0)]
    for g, bit in enumerate((0x10, 0x20, 0x40)):
        if flags & bit:
            seg = slice(g * b, (g + 1) * b)
            assert np.all(np.abs(got[2][seg] - ref[2][seg]) <= TOL * bounds[g] + 1e-300), (g, b)


def test_aug_beta_zero_ignores_nan_y_and_delta_zero_ignores_nan_z(sc):
    import torch

    A = MATS["lap2d_64"]
    b = 2
    X = synth.block_vector(A.ncols, b, 1)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    Yd = torch.full((A.nrows, b), float("nan"), dtype=torch.float64, device="cuda:0")
    Zd = torch.full((A.nrows, b), float("inf"), dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_aug(M, dev(X), Yd, Z=Zd, flags=sc.AXPBY | sc.CHAIN, beta=0.0, delta=0.0, eta=3.0)
    y, z = host(Yd), host(Zd)
    ref = oracle.spmmv(A, X)
    assert np.all(np.isfinite(y)) and colwise_relerr(y, ref) <= TOL
    assert np.array_equal(z, 3.0 * y)
    M.close()


def test_aug_paper_listing_sequence(sc):
    # Sec. 5.3 usage example: y = (A - gamma_j I) x, then y = (A - gamma_j I) x - 2 y with <x, y>
    import torch

    A = MATS["irregular_5000"]
    b = 4
    shift = np.array([1.0, 2.0, -1.0, 0.5])
    X = synth.block_vector(A.ncols, b, 2)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=32)
    Yd = torch.zeros((A.nrows, b), dtype=torch.float64, device="cuda:0")
    dot = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_aug(M, dev(X), Yd, flags=sc.VSHIFT, gamma_v=shift)
    sc.sell_spmmv_aug(M, dev(X), Yd, flags=sc.VSHIFT | sc.AXPBY | sc.DOT_XY, beta=-2.0, gamma_v=shift, dot=dot)
    y1, _, _ = oracle.spmmv_aug(A, X, flags=oracle.VSHIFT, gamma_v=shift)
    y2, _, d = oracle.spmmv_aug(A, X, Y=y1, flags=oracle.VSHIFT | oracle.AXPBY | oracle.DOT_XY, beta=-2.0,
                                gamma_v=shift)
    scale = 3 * (abs_product(A, X) + 2 * np.abs(X))
    assert colwise_relerr(host(Yd), y2, scale) <= TOL
    got = host(dot)[b:2 * b]
    assert np.all(np.abs(got - d[b:2 * b]) <= TOL * np.sum(np.abs(X * y2), axis=0))
    M.close()


def test_column_major_vectors(sc):
    import torch

    A = MATS["irregular_5000"]
    b = 5
    X = synth.block_vector(A.ncols, b, 9)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=128)
    Xcm = dev(X.T.copy()).t()  # column-major view (stride (1, n))
    assert Xcm.stride(0) == 1
    Ycm = torch.zeros((b, A.nrows), dtype=torch.float64, device="cuda:0").t()
    sc.sell_spmmv(M, Xcm, Ycm)
    ref = oracle.spmmv(A, X)
    assert colwise_relerr(host(Ycm), ref, abs_product(A, X)) <= TOL
    M.close()


def test_empty_and_zero_matrices(sc):
    import torch

    E = synth.CSR(0, 0, np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0), "empty")
    M = sc.SellMatrix.from_csr(E, C=32, sigma=1)
    X = torch.zeros((0, 3), dtype=torch.float64, device="cuda:0")
    Y = torch.zeros((0, 3), dtype=torch.float64, device="cuda:0")
    dot = torch.full((9,), 5.0, dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_aug(M, X, Y, flags=sc.DOTS, dot=dot)
    assert np.all(host(dot) == 0.0)
    M.close()
    Z = synth.CSR(70, 70, np.zeros(71, np.int64), np.zeros(0, np.int32), np.zeros(0), "zero")
    M = sc.SellMatrix.from_csr(Z, C=32, sigma=1)
    X = dev(synth.block_vector(70, 2, 1))
    Y = torch.full((70, 2), 9.0, dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv(M, X, Y)
    assert np.all(host(Y) == 0.0)
    M.close()


def test_bad_arguments_are_rejected_before_launch(sc):
    import torch

    A = MATS["rect_270x190"]
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    X = torch.zeros((190, 2), dtype=torch.float64, device="cuda:0")
    Y = torch.zeros((270, 2), dtype=torch.float64, device="cuda:0")
    with pytest.raises(sc.SellError) as e:
        sc.sell_spmmv(M, Y, X)  # swapped shapes
    assert e.value.code == sc.SELL_ERR_SHAPE
    with pytest.raises(sc.SellError) as e:
        sc.sell_spmmv(M, X.float(), Y.float())
    assert e.value.code == sc.SELL_ERR_DTYPE
    with pytest.raises(sc.SellError) as e:
        sc.sell_spmmv_aug(M, X, Y, flags=sc.SHIFT, gamma=1.0)  # shift needs a square matrix
    assert e.value.code == sc.SELL_ERR_SHAPE
    with pytest.raises(sc.SellError) as e:
        sc.sell_spmmv_aug(M, X, Y, flags=sc.DOT_YY)  # no dot buffer
    assert e.value.code == sc.SELL_ERR_ARG
    with pytest.raises(sc.SellError) as e:
        sc.sell_spmmv_aug(M, X, Y, flags=sc.CHAIN)  # no z
    assert e.value.code == sc.SELL_ERR_ARG
    with pytest.raises(sc.SellError) as e:
        sc.sell_spmmv_aug(M, X, Y, flags=0x100)
    assert e.value.code == sc.SELL_ERR_ARG
    M.close()


# ------------------------------------------------------------------ low precision values


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_low_precision_integer_laplacian_bit_exact(sc, dt):
    import torch

    A = synth.laplacian3d(17)  # 6 / -1 are exact in bf16; integer sums far below 2^24
    X = synth.int_block_vector(A.ncols, 8, 4)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1, dtype=dt)
    Yd = torch.zeros((A.nrows, 8), dtype=torch.float32, device="cuda:0")
    sc.sell_spmmv(M, dev(X, torch.float32), Yd)
    assert np.array_equal(host(Yd), oracle.spmmv(A, X))
    M.close()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("b", [1, 2, 3, 4, 8, 16, 32])
def test_low_precision_error_bound(sc, dt, b):
    """O7: every block width the single-matrix kernels instantiate (and a generic one, 3), on the
    irregular matrix with sigma = 1024 and the C = 32 slices, against the exact product of the
    rounded inputs within the deterministic FP32 bound."""
    import torch

    A = MATS["irregular_5000"]
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1024, dtype=dt)
    X32 = synth.block_vector(A.ncols, b, 6).astype(np.float32).astype(np.float64)
    Yd = torch.zeros((A.nrows, b), dtype=torch.float32, device="cuda:0")
    sc.sell_spmmv(M, dev(X32, torch.float32), Yd)
    got = host(Yd)
    assert_lowprec_product(got, A, X32, dt, what=(dt, b))
    # error against the unrounded FP64 product, reported rather than pinned
    err = colwise_relerr(got, oracle.spmmv(A, X32))
    print(f"{dt} b={b}: rel err vs unrounded FP64 product {err:.2e}")
    M.close()


def test_low_precision_aug_dots_in_fp64(sc):
    import torch

    A = MATS["anderson_12"]
    b = 4
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1, dtype="f32")
    X32 = synth.block_vector(A.ncols, b, 6).astype(np.float32)
    Xd = dev(X32)
    Yd = torch.zeros((A.nrows, b), dtype=torch.float32, device="cuda:0")
    dot = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_aug(M, Xd, Yd, flags=sc.SHIFT | sc.DOTS, gamma=0.5, dot=dot)
    y = host(Yd)
    x = X32.astype(np.float64)
    # the dots are FP64 sums of the stored FP32 values
    for g, (u, v) in enumerate([(y, y), (x, y), (x, x)]):
        ref = np.array([oracle.dot(u[:, j], v[:, j]) for j in range(b)])
        assert np.all(np.abs(host(dot)[g * b:(g + 1) * b] - ref) <= TOL * np.sum(np.abs(u * v), axis=0))
    M.close()


# ------------------------------------------------------------------ transpose


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("b", [1, 3, 8])
def test_transpose(sc, det, b):
    import torch

    for name in ("rect_270x190", "irregular_5000"):
        A = MATS[name]
        M = sc.SellMatrix.from_csr(A, C=32, sigma=64)
        X = synth.block_vector(A.nrows, b, 8)
        Yd = torch.full((A.ncols, b), 3.0, dtype=torch.float64, device="cuda:0")
        sc.sell_spmmv_T(M, dev(X), Yd, deterministic=det)
        got = host(Yd)
        ref = oracle.spmmv_T(A, X)
        from synth import CSR

        At = CSR(A.nrows, A.ncols, A.rowptr, A.col, np.abs(A.val))
        scale = oracle.spmmv_T(At, np.abs(X))
        assert colwise_relerr(got, ref, scale) <= TOL, (name, det)
        if det:
            Y2 = torch.zeros_like(Yd)
            sc.sell_spmmv_T(M, dev(X), Y2, deterministic=True)
            torch.cuda.synchronize()
            assert torch.equal(Yd, Y2)
        M.close()


def test_transpose_adjoint_identity(sc):
    import torch

    A = MATS["irregular_5000"]
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    u = synth.block_vector(A.nrows, 1, 10)
    v = synth.block_vector(A.ncols, 1, 11)
    ATu = torch.zeros((A.ncols, 1), dtype=torch.float64, device="cuda:0")
    Av = torch.zeros((A.nrows, 1), dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_T(M, dev(u), ATu, deterministic=False)
    sc.sell_spmmv(M, dev(v), Av)
    lhs = float(np.dot(host(ATu)[:, 0], v[:, 0]))
    rhs = float(np.dot(u[:, 0], host(Av)[:, 0]))
    assert abs(lhs - rhs) <= 1e-12 * float(np.abs(u[:, 0]) @ abs_product(A, np.abs(v))[:, 0])
    M.close()


# ------------------------------------------------------------------ block-vector copy


@pytest.mark.parametrize("src_dt,dst_dt", [("f64", "f32"), ("f64", "bf16"), ("f32", "bf16"), ("bf16", "f64"),
                                           ("f32", "f64"), ("f64", "f64")])
def test_bv_copy_conversions_and_layouts(sc, src_dt, dst_dt):
    import torch

    tmap = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
    n, b = 1001, 6
    vals = synth.normal(12, n * b).reshape(n, b) * np.exp(synth.uniform(13, n * b, -30, 30)).reshape(n, b)
    if src_dt == "bf16":
        vals = oracle.round_bf16(vals.ravel()).reshape(n, b)
    if src_dt == "f32":
        vals = vals.astype(np.float32).astype(np.float64)
    src = dev(vals, tmap[src_dt]) if src_dt != "bf16" else dev(vals).to(torch.bfloat16)
    for dst_colmajor in (False, True):
        dst = torch.zeros((b, n) if dst_colmajor else (n, b), dtype=tmap[dst_dt], device="cuda:0")
        if dst_colmajor:
            dst = dst.t()
        sc.sell_bv_copy(dst, src)
        got = host(dst)
        want = {"f64": vals, "f32": oracle.round_f32(vals.ravel()).reshape(n, b),
                "bf16": oracle.round_bf16(vals.ravel()).reshape(n, b)}[dst_dt]
        assert np.array_equal(got, want), (src_dt, dst_dt, dst_colmajor)


# ------------------------------------------------------------------ value updates


@pytest.mark.parametrize("dt", ["f64", "bf16"])
def test_update_values_device_and_host(sc, dt):
    import torch

    A = MATS["irregular_5000"]
    M = sc.SellMatrix.from_csr(A, C=32, sigma=256, dtype=dt)
    newv = synth.uniform(14, A.nnz, -3, 3)
    M.update_values(dev(newv))
    torch.cuda.synchronize()
    _, col, val = M.export_csr()
    want = newv if dt == "f64" else oracle.round_bf16(newv)
    assert np.array_equal(val, want) and np.array_equal(col, A.col)
    newv2 = synth.uniform(15, A.nnz, -3, 3)
    M.update_values(newv2)
    _, _, val2 = M.export_csr()
    assert np.array_equal(val2, newv2 if dt == "f64" else oracle.round_bf16(newv2))
    M.close()


def test_device_export_round_trip(sc):
    A = MATS["random_ragged"]
    M = sc.SellMatrix.from_csr(A, C=16, sigma=40)
    rp, col, val = M.export_csr()
    assert np.array_equal(rp, A.rowptr) and np.array_equal(col, A.col) and np.array_equal(val, A.val)
    perm, cl, cs, scol, sval = M.export_sell()
    operm, ocl, ocs = oracle.sell_layout(A, 16, 40)
    ocol, oval = oracle.sell_fill(A, 16, operm, ocl, ocs)
    assert np.array_equal(perm, operm) and np.array_equal(scol, ocol) and np.array_equal(sval, oval)
    M.close()


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("b,ld,off", [(2, 3, 1), (3, 3, 0), (4, 5, 1), (5, 5, 0), (6, 6, 0), (7, 11, 3), (8, 9, 0), (9, 9, 0),
                                      (10, 10, 0), (12, 12, 0), (16, 17, 1), (21, 21, 0), (32, 33, 1), (33, 33, 0), (45, 45, 0),
                                      (61, 61, 0), (64, 64, 0), (64, 67, 2)])
def test_contiguous_rows_of_any_width_equal_the_strided_kernel(sc, b, ld, off, dt):
    """The run-time-width kernel for contiguous rows (pieces of 2 to 4 columns, rows per wave that do
    not fill it, unaligned rows, slices of wider blocks) against the any-strides kernel on the same
    values held column-major: y and z bit for bit, the dots of the final y within a fixed-order FP64
    sum's error, nothing written beside the block, for every index batch length."""
    import torch

    A = synth.random_sparse(1003, 1003, 0.008, 190, duplicates=True, empty_rows=11, long_row=90)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=128, dtype=dt)
    vt = torch.float64 if dt == "f64" else torch.float32
    n = A.nrows
    flags = sc.VSHIFT | sc.SCALE | sc.AXPBY | sc.DOTS | sc.CHAIN
    kw = dict(flags=flags, alpha=0.7, beta=-0.3, gamma_v=np.linspace(-1, 1, b), delta=0.5, eta=-2.0)

    def rows(seed):
        t = torch.full((n + 1, ld), 9.0, dtype=vt, device="cuda:0")
        s = t[:n, off:off + b]
        s.copy_(torch.from_numpy(synth.block_vector(n, b, seed)))
        return t, s

    for batch in (5, 7, 8):
        M.set_batch(batch)
        (xt, x), (yt, y), (zt, z) = rows(191), rows(192), rows(193)
        xc, yc, zc = (v.t().contiguous().t() for v in (x, y, z))
        dot, dotc = (torch.zeros(3 * b, dtype=torch.float64, device="cuda:0") for _ in range(2))
        sc.sell_spmmv_aug(M, x, y, z, dot=dot, **kw)
        sc.sell_spmmv_aug(M, xc, yc, zc, dot=dotc, **kw)
        assert torch.equal(y, yc) and torch.equal(z, zc)
        xd, yd = xc.double(), yc.double()
        mag = torch.cat([(yd * yd).sum(0), (xd * yd).abs().sum(0), (xd * xd).sum(0)])
        assert bool(((dot - dotc).abs() <= 2 * (n + 8) * 2.0 ** -53 * mag).all())
        for t in (xt, yt, zt):
            assert bool((t[n] == 9.0).all()) and bool((t[:, :off] == 9.0).all()) and bool((t[:, off + b:] == 9.0).all())
        sc.sell_spmmv(M, x, y)
        sc.sell_spmmv(M, xc, yc)
        assert torch.equal(y, yc)
    M.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("b", [3, 6, 12, 33, 64])
def test_batch_of_any_width_equals_single_products(sc, b, dt):
    """A uniform batch at a width without a compiled kernel: y bit for bit the single products'."""
    import torch

    mats = [synth.anderson3d(6), synth.random_sparse(700, 700, 0.01, 194, empty_rows=5), synth.laplacian2d(23)]
    Ms = [sc.SellMatrix.from_csr(A, C=32, sigma=32, dtype=dt) for A in mats]
    B = sc.SellBatch(Ms)
    vt = torch.float64 if dt == "f64" else torch.float32
    X = torch.from_numpy(synth.block_vector(B.cols, b, 195)).to("cuda:0", vt)
    Y = torch.zeros((B.rows, b), dtype=vt, device="cuda:0")
    dot = torch.zeros(3 * b * len(mats), dtype=torch.float64, device="cuda:0")
    sc.sell_batch_spmmv_aug(B, X, Y, flags=sc.DOT_YY | sc.DOT_XY, dot=dot)
    at = 0
    for k, (A, M) in enumerate(zip(mats, Ms)):
        y = torch.zeros((A.nrows, b), dtype=vt, device="cuda:0")
        d = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
        x = X[at:at + A.nrows]
        sc.sell_spmmv_aug(M, x, y, flags=sc.DOT_YY | sc.DOT_XY, dot=d)
        assert torch.equal(y, Y[at:at + A.nrows])
        xd, yd = x.double(), y.double()
        mag = torch.cat([(yd * yd).sum(0), (xd * yd).abs().sum(0), torch.zeros(b, dtype=torch.float64, device="cuda:0")])
        assert bool(((dot[3 * b * k:3 * b * (k + 1)] - d).abs() <= 2 * (A.nrows + 8) * 2.0 ** -53 * mag).all())
        at += A.nrows
    B.close()
    for M in Ms:
        M.close()


@pytest.mark.parametrize("dt,b", [("f64", 1), ("f64", 4), ("f64", 8), ("f64", 12), ("f64", 32), ("f64", 64), ("bf16", 8), ("f32", 12)])
@pytest.mark.parametrize("n", [33, 700, 9000])
def test_grids_of_several_waves_equal_one_wave(sc, dt, b, n):
    """Products on grids of many workgroups (whole or half size, at least a pass of rows each) against
    one wave: y and z bit for bit, dots within a fixed-order FP64 sum's error."""
    import torch

    A = synth.irregular(n, mean_len=8.0, max_len=min(n, 300), band=50, seed=196)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=256, dtype=dt)
    vt = torch.float64 if dt == "f64" else torch.float32
    X, Y0, Z0 = (torch.from_numpy(synth.block_vector(n, b, s)).to("cuda:0", vt) for s in (197, 198, 199))
    outs = []
    for waves in (1, 0, 2, 16):
        M.set_waves(waves)
        Y, Z, P = Y0.clone(), Z0.clone(), torch.empty_like(Y0)
        dot = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
        sc.sell_spmmv_aug(M, X, Y, Z, flags=sc.SHIFT | sc.SCALE | sc.AXPBY | sc.DOTS | sc.CHAIN, alpha=0.5, beta=-1.0,
                          gamma=0.3, delta=1.0, eta=0.5, dot=dot)
        sc.sell_spmmv(M, X, P)
        outs.append((Y, Z, P, dot))
    xd, yd = X.double(), outs[0][0].double()
    mag = torch.cat([(yd * yd).sum(0), (xd * yd).abs().sum(0), (xd * xd).sum(0)])
    for o in outs[1:]:
        assert all(torch.equal(u, v) for u, v in zip(o[:3], outs[0][:3]))
        assert bool(((o[3] - outs[0][3]).abs() <= 2 * (n + 8) * 2.0 ** -53 * mag).all())
    M.close()


@pytest.mark.parametrize("dt,n,widths", [("f64", 118, (1, 3, 8, 12)), ("f32", 134, (4, 12, 16))])
def test_cache_policies_equal_general_kernel(sc, dt, n, widths):
    """Matrices either side of the cache policy's line (by b): products, their chains and a batch of
    two matrices against the general kernel over column-major operands, y and z bit for bit."""
    import torch

    A = synth.anderson3d(n)
    small = synth.anderson3d(12)
    M, S = (sc.SellMatrix.from_csr(m, C=32, sigma=1, dtype=dt) for m in (A, small))
    B = sc.SellBatch([M, S])
    vt = torch.float64 if dt == "f64" else torch.float32
    N, T = A.nrows, A.nrows + small.nrows
    for b in widths:
        x, y0, z0 = (torch.randn((T, b), dtype=vt, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(s))
                     for s in (200, 201, 202))
        xc, yc, zc = (v.t().contiguous().t() if b > 1 else v.clone() for v in (x, y0, z0))
        for flags in (sc.SHIFT | sc.SCALE | sc.AXPBY | sc.DOT_YY | sc.DOT_XY, sc.SHIFT | sc.AXPBY | sc.DOTS | sc.CHAIN):
            kw = dict(flags=flags, alpha=0.5, beta=-1.0, gamma=0.3, delta=1.0, eta=0.5)
            y, z, yg, zg, yb, zb = y0.clone(), z0.clone(), yc.clone(), zc.clone(), y0.clone(), z0.clone()
            d = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
            db = torch.zeros(6 * b, dtype=torch.float64, device="cuda:0")
            for m, lo, hi in ((M, 0, N), (S, N, T)):
                sc.sell_spmmv_aug(m, x[lo:hi], y[lo:hi], z[lo:hi], dot=d, **kw)
                g = [torch.empty((b, hi - lo), dtype=vt, device="cuda:0").t().copy_(v[lo:hi]) for v in (xc, yc, zc)]
                sc.sell_spmmv_aug(m, *g, dot=d, **kw)
                yg[lo:hi], zg[lo:hi] = g[1], g[2]
            sc.sell_batch_spmmv_aug(B, x, yb, zb, dot=db, **kw)
            assert torch.equal(y, yg) and torch.equal(z, zg)
            assert torch.equal(y, yb) and torch.equal(z, zb)
        p, pb = torch.empty_like(x), torch.empty_like(x)
        pc = torch.empty((b, N), dtype=vt, device="cuda:0").t()
        sc.sell_spmmv(M, x[:N], p[:N])
        sc.sell_spmmv(S, x[N:], p[N:])
        sc.sell_spmmv(M, torch.empty((b, N), dtype=vt, device="cuda:0").t().copy_(x[:N]), pc)
        sc.sell_batch_spmmv_aug(B, x, pb)
        assert torch.equal(p[:N], pc) and torch.equal(p, pb)
    for o in (B, M, S):
        o.close()


@pytest.mark.parametrize("C,sigma", [(32, 1), (32, 64), (12, 1), (1, 1)])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_chunks_of_one_length_equal_general_kernel(sc, dt, C, sigma):
    """Augmented products of matrices whose chunks all have one length (bounds computed) against the
    general kernel over column-major operands: y and z bit for bit, dots within a fixed-order sum's error."""
    import torch

    vt = torch.float64 if dt == "f64" else torch.float32
    for A in (synth.anderson3d(3), synth.anderson3d(7), synth.anderson3d(33)):
        n = A.nrows
        M = sc.SellMatrix.from_csr(A, C=C, sigma=sigma, dtype=dt)
        for b in (1, 2, 3, 8, 16, 33):
            x, y0, z0 = (torch.from_numpy(synth.block_vector(n, b, s)).to("cuda:0", vt) for s in (203, 204, 205))
            for flags in (sc.SHIFT | sc.SCALE | sc.AXPBY | sc.DOT_YY | sc.DOT_XY, sc.DOT_YY | sc.DOT_XY,
                          sc.SHIFT | sc.AXPBY | sc.DOTS | sc.CHAIN):
                kw = dict(flags=flags, alpha=0.5, beta=-1.0, gamma=0.3, delta=1.0, eta=0.5)
                y, z = y0.clone(), z0.clone()
                g = [torch.empty((b, n), dtype=vt, device="cuda:0").t().copy_(v) for v in (x, y0, z0)]
                d, dg = (torch.zeros(3 * b, dtype=torch.float64, device="cuda:0") for _ in range(2))
                sc.sell_spmmv_aug(M, x, y, z, dot=d, **kw)
                sc.sell_spmmv_aug(M, *g, dot=dg, **kw)
                assert torch.equal(y, g[1]) and torch.equal(z, g[2])
                xd, yd = x.double(), y.double()
                mag = torch.cat([(yd * yd).sum(0), (xd * yd).abs().sum(0), (xd * xd).sum(0)])
                assert bool(((d - dg).abs() <= 2 * (n + 8) * 2.0 ** -53 * mag).all())
        M.close()


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n,length", [(1, 300), (33, 64), (200, 63), (200, 70), (8192, 66), (8193, 66)])
def test_narrow_products_of_few_long_rows(sc, orc, dt, n, length):
    """Matrices either side of the line between the narrow kernels (rows of 64 entries, 8,192 rows) at
    widths without a compiled kernel and at unaligned ones, single and in a batch: on integer data y bit
    for bit the oracle's, the dots exact, nothing written beside the block."""
    import torch

    m = 400
    col = np.sort(synth.randint(220, n * length, 0, m - 1).reshape(n, length), axis=1).astype(np.int32).reshape(-1)
    A = synth.CSR(n, m, np.arange(n + 1, dtype=np.int64) * length, col, synth.randint(221, n * length, -2, 2).astype(np.float64))
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1, dtype=dt)
    B = sc.SellBatch([M, M])
    vt = torch.float64 if dt == "f64" else torch.float32
    for b in (2, 3, 5, 7, 9):
        x = synth.int_block_vector(m, b, 222, -3, 3)
        want = orc.spmmv(A, x)
        buf = torch.full((m + n + 2, b + 1), 9.0, dtype=vt, device="cuda:0")
        X, Y = buf[:m, 1:], buf[m:m + n, 1:]
        X.copy_(torch.from_numpy(x))
        sc.sell_spmmv(M, X, Y)
        assert np.array_equal(Y.double().cpu().numpy(), want)
        Y.fill_(0.0)
        d = torch.zeros(3 * b, dtype=torch.float64, device="cuda:0")
        sc.sell_spmmv_aug(M, X, Y, flags=sc.DOT_YY, dot=d)
        assert np.array_equal(Y.double().cpu().numpy(), want)
        assert np.array_equal(d[:b].cpu().numpy(), (want * want).sum(0))
        assert bool((buf[:, 0] == 9.0).all()) and bool((buf[m + n:] == 9.0).all())
        Xb = torch.from_numpy(np.concatenate([x, x])).to("cuda:0", vt)
        Yb = torch.empty((2 * n, b), dtype=vt, device="cuda:0")
        db = torch.zeros(6 * b, dtype=torch.float64, device="cuda:0")
        sc.sell_batch_spmmv_aug(B, Xb, Yb, flags=sc.DOT_YY, dot=db)
        assert np.array_equal(Yb.double().cpu().numpy(), np.concatenate([want, want]))
        assert np.array_equal(db.view(2, 3, b)[:, 0].cpu().numpy(), np.stack([(want * want).sum(0)] * 2))
    B.close()
    M.close()
