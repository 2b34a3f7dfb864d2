"""GPU tests of differentiation with respect to the stored matrix values: the pattern-
restricted outer product, the single-product autograd function (torch.autograd.gradcheck,
i.e. central finite differences in FP64, runs the HIP kernels), and the Chebyshev
application T_N(A(theta)) x with recompute checkpoints against the oracle's FP64 adjoint and
against finite differences."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import torch

    import paper_1507_08101_amd as sc

    assert torch.cuda.is_available()
    sc.lib()
    return sc


def _relnorm(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("b", [1, 3, 8])
def test_grad_values_matches_oracle(sc, b):
    import torch

    A = synth.random_sparse(300, 170, 0.05, 120, duplicates=True, empty_rows=7)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=64)
    G = synth.block_vector(A.nrows, b, 121)
    X = synth.block_vector(A.ncols, b, 122)
    dval = torch.full((A.nnz,), 5.0, dtype=torch.float64, device="cuda:0")
    sc.sell_grad_values(M, dev(G), dev(X), dval, alpha=2.0)
    ref = 2.0 * oracle.pattern_outer(A, G, X)
    assert _relnorm(host(dval), ref) <= 1e-14
    sc.sell_grad_values(M, dev(G), dev(X), dval, alpha=1.0, accumulate=True)
    assert _relnorm(host(dval), 1.5 * ref) <= 1e-14
    M.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("b", [1, 2, 4, 5, 7, 8, 9, 12, 16, 17, 31, 32, 33, 63, 64, 65, 70])
def test_grad_values_every_lane_group(sc, b, dt):
    """Every width class of the gradient kernel (lanes per row, shifted last pieces, slices past 64),
    rows longer than an entry batch and empty rows, sorted windows: per entry within the bound of a
    b-term FP64 sum, (b + 4) u sum |g x|."""
    import torch

    A = synth.random_sparse(301, 170, 0.04, 135, duplicates=True, empty_rows=9, long_row=150)
    M = sc.SellMatrix.from_csr(A, C=12 if b % 2 else 32, sigma=40, dtype=dt)
    vt = np.float64 if dt == "f64" else np.float32
    G = synth.block_vector(A.nrows, b, 136).astype(vt)
    X = synth.block_vector(A.ncols, b, 137).astype(vt)
    ref, mag = oracle.pattern_outer(A, G, X), oracle.pattern_outer(A, np.abs(G), np.abs(X))
    dval = torch.full((A.nnz,), 5.0, dtype=torch.float64, device="cuda:0")
    sc.sell_grad_values(M, dev(G), dev(X), dval, alpha=-0.7)
    bound = 0.7 * (b + 4) * 2.0 ** -53 * mag
    assert (np.abs(host(dval) + 0.7 * ref) <= bound).all()
    sc.sell_grad_values(M, dev(G), dev(X), dval, alpha=1.7, accumulate=True)
    assert (np.abs(host(dval) - ref) <= 4 * bound + 2.0 ** -52 * np.abs(ref)).all()
    M.close()


def test_spmm_autograd_gradcheck(sc):
    import torch

    from paper_1507_08101_amd.autograd import spmm

    A = synth.random_sparse(40, 30, 0.15, 123)
    M = sc.SellMatrix.from_csr(A, C=8, sigma=16)
    theta = torch.tensor(A.val, dtype=torch.float64, device="cuda:0", requires_grad=True)
    X = torch.tensor(synth.block_vector(30, 2, 124), device="cuda:0", requires_grad=True)
    assert torch.autograd.gradcheck(lambda t, x: spmm(t, x, M), (theta, X), eps=1e-6, atol=1e-8, rtol=1e-6)
    M.close()


def test_transpose_follows_value_updates(sc):
    import torch

    A = synth.random_sparse(120, 90, 0.06, 125)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=32)
    X = synth.block_vector(A.nrows, 2, 126)
    Y = torch.zeros((A.ncols, 2), dtype=torch.float64, device="cuda:0")
    sc.sell_spmmv_T(M, dev(X), Y, deterministic=True)  # builds the copy of A^T
    newv = synth.uniform(127, A.nnz, -2, 2)
    M.update_values(dev(newv))
    sc.sell_spmmv_T(M, dev(X), Y, deterministic=True)
    A2 = synth.CSR(A.nrows, A.ncols, A.rowptr, A.col, newv)
    assert _relnorm(host(Y), oracle.spmmv_T(A2, X)) <= 1e-14
    M.close()


def test_first_transpose_after_update_on_side_stream(sc):
    """A value update queued on a non-blocking side stream, then the first deterministic
    transposed product on that stream: the copy of A^T it builds must hold the new values."""
    import torch

    A = synth.random_sparse(2000, 1500, 0.01, 128)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=64)
    X = synth.block_vector(A.nrows, 3, 129)
    newv = synth.uniform(130, A.nnz, -2, 2)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        nv = dev(newv)
        Xd = dev(X)
        side.synchronize()
        # a long kernel queued first keeps the stream busy while the update waits behind it
        big = torch.randn(4096, 4096, dtype=torch.float64, device="cuda:0")
        for _ in range(4):
            big = big @ big * 1e-3
        M.update_values(nv)  # on the current stream: side
        Y = torch.zeros((A.ncols, 3), dtype=torch.float64, device="cuda:0")
        sc.sell_spmmv_T(M, Xd, Y, deterministic=True)
    side.synchronize()
    A2 = synth.CSR(A.nrows, A.ncols, A.rowptr, A.col, newv)
    assert _relnorm(host(Y), oracle.spmmv_T(A2, X)) <= 1e-14
    M.close()


@pytest.mark.parametrize("fn", ["spmm", "chebyshev"])
def test_autograd_two_forwards_one_handle(sc, fn):
    """Two forwards with different theta on one matrix handle before either backward: each
    backward must give the gradients of the matrix its own forward used."""
    import torch

    from paper_1507_08101_amd.autograd import chebyshev, spmm

    A = synth.anderson3d(6)
    s = (6 + 16.5 / 2) / 0.99
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    X = synth.block_vector(A.nrows, 2, 131)
    th1 = A.val.copy()
    th2 = A.val * synth.uniform(132, A.nnz, 0.5, 1.0)
    run = (lambda t, x: spmm(t, x, M)) if fn == "spmm" else (lambda t, x: chebyshev(t, x, M, 7, s, 0.0, 3))
    grads = []
    outs = []
    for th in (th1, th2):
        t = torch.tensor(th, device="cuda:0", requires_grad=True)
        x = torch.tensor(X, device="cuda:0", requires_grad=True)
        outs.append((t, x, run(t, x)))
    for t, x, y in reversed(outs):  # backward of the second forward first, then the first
        (y * y).sum().backward()
        grads.append((host(t.grad), host(x.grad)))
    grads.reverse()
    for (th, (gt, gx)) in zip((th1, th2), grads):
        Ak = synth.CSR(A.nrows, A.ncols, A.rowptr, A.col, th)
        if fn == "spmm":
            Y = oracle.spmmv(Ak, X)
            rx, rt = oracle.spmmv_T(Ak, 2 * Y), oracle.pattern_outer(Ak, 2 * Y, X)
        else:
            Y = oracle.cheb_apply(Ak, X, 7, s, 0.0)
            rx, rt = oracle.cheb_grad(Ak, X, 7, s, 0.0, 2 * Y)
        assert _relnorm(gx, rx) <= 1e-12 and _relnorm(gt, rt) <= 1e-12
    M.close()


def _anderson_case(L, b, seed):
    A = synth.anderson3d(L)
    s = (6 + 16.5 / 2) / 0.99
    X = synth.block_vector(A.nrows, b, seed)
    return A, s, X


@pytest.mark.parametrize("N,K,b", [(1, 10, 1), (7, 3, 2), (20, 6, 1), (20, 20, 3), (20, 40, 1)])
def test_chebyshev_forward_backward_vs_oracle(sc, N, K, b):
    import torch

    from paper_1507_08101_amd.autograd import chebyshev

    A, s, X = _anderson_case(10, b, 130)
    c = 0.3
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    theta = torch.tensor(A.val, dtype=torch.float64, device="cuda:0", requires_grad=True)
    Xd = torch.tensor(X, device="cuda:0", requires_grad=True)
    Y = chebyshev(theta, Xd, M, N, s, c, K)
    Yref = oracle.cheb_apply(A, X, N, s, c)
    assert _relnorm(host(Y), Yref) <= 1e-12
    loss = (Y * Y).sum()
    loss.backward()
    dX_ref, dval_ref = oracle.cheb_grad(A, X, N, s, c, 2.0 * Yref)
    assert _relnorm(host(Xd.grad), dX_ref) <= 1e-11
    assert _relnorm(host(theta.grad), dval_ref) <= 1e-11
    M.close()


@pytest.mark.parametrize("N,K,b", [(1, 1, 1), (2, 1, 2), (5, 1, 1), (6, 2, 9), (9, 4, 16), (9, 4, 20), (12, 4, 1), (40, 25, 1)])
def test_chebyshev_checkpoint_layouts(sc, N, K, b):
    """Checkpoints of every step, segments that end at N, outer products grouped over 16, 1 and fewer
    steps; the results written over the inputs (X over Y, G over dX), as separate buffers give."""
    import torch

    A, s, X = _anderson_case(8, b, 134)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    G = synth.block_vector(A.nrows, b, 135)
    Yref = oracle.cheb_apply(A, X, N, s, 0.2)
    dX_ref, dval_ref = oracle.cheb_grad(A, X, N, s, 0.2, G)
    outs = []
    for inplace in (False, True):
        Xd, Gd = dev(X), dev(G)
        Y, dX = (Xd, Gd) if inplace else (torch.empty_like(Xd), torch.empty_like(Gd))
        ck = torch.full((sc.cheb_ckpt_elems(A.nrows, b, N, K),), float("nan"), dtype=torch.float64, device="cuda:0")
        dval = torch.full((A.nnz,), float("nan"), dtype=torch.float64, device="cuda:0")
        sc.sell_cheb_forward(M, Xd, Y, N, s, 0.2, K, ck)
        sc.sell_cheb_backward(M, Gd, N, s, 0.2, K, ck, dX, dval)
        outs.append([host(t) for t in (Y, dX, dval, ck)])
        assert _relnorm(outs[-1][0], Yref) <= 1e-12
        assert _relnorm(outs[-1][1], dX_ref) <= 1e-11
        assert _relnorm(outs[-1][2], dval_ref) <= 1e-11
    for u, v in zip(*outs):
        assert np.array_equal(u, v)
    # the checkpoints are the pairs (v_kK, v_kK+1)
    pairs = outs[0][3].reshape(-1, 2, A.nrows, b)
    for k in range(pairs.shape[0]):
        for i in (0, 1):
            m = k * K + i
            want = X if m == 0 else oracle.cheb_apply(A, X, m, s, 0.2)
            assert _relnorm(pairs[k, i], want) <= 1e-12
    M.close()


def test_chebyshev_general_nonsymmetric(sc):
    # a nonsymmetric matrix exercises the A^T path of the adjoint
    import torch

    from paper_1507_08101_amd.autograd import chebyshev

    A = synth.random_sparse(500, 500, 0.01, 131, empty_rows=4)
    s, c, N, K = 3.0, 0.1, 9, 4
    X = synth.block_vector(500, 2, 132)
    W = synth.block_vector(500, 2, 133)
    M = sc.SellMatrix.from_csr(A, C=16, sigma=50)
    theta = torch.tensor(A.val, dtype=torch.float64, device="cuda:0", requires_grad=True)
    Xd = torch.tensor(X, device="cuda:0", requires_grad=True)
    Y = chebyshev(theta, Xd, M, N, s, c, K)
    (Y * dev(W)).sum().backward()
    dX_ref, dval_ref = oracle.cheb_grad(A, X, N, s, c, W)
    assert _relnorm(host(Xd.grad), dX_ref) <= 1e-11
    assert _relnorm(host(theta.grad), dval_ref) <= 1e-11
    M.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_chebyshev_degree100_anderson64(sc, dt):
    """The differentiation workload: T_100 of the 64^3 Anderson matrix, loss sum(y^2),
    checkpoints every 10 steps; FP64 against the oracle's FP64 adjoint, FP32 against the
    oracle's adjoint of the float32-rounded values, and FP64 against central differences."""
    import torch

    from paper_1507_08101_amd.autograd import chebyshev

    A, s, X = _anderson_case(64, 1, 140)
    N, K = 100, 10
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1, dtype=dt)
    vt = torch.float64 if dt == "f64" else torch.float32
    Xin = X if dt == "f64" else X.astype(np.float32).astype(np.float64)
    theta = torch.tensor(A.val, dtype=torch.float64, device="cuda:0", requires_grad=True)
    Xd = torch.tensor(Xin, dtype=vt, device="cuda:0", requires_grad=True)
    Y = chebyshev(theta, Xd, M, N, s, 0.0, K)
    loss = (Y.double() ** 2).sum()
    loss.backward()
    Ar = A if dt == "f64" else synth.CSR(A.nrows, A.ncols, A.rowptr, A.col, oracle.round_f32(A.val))
    Yref = oracle.cheb_apply(Ar, Xin, N, s)
    dX_ref, dval_ref = oracle.cheb_grad(Ar, Xin, N, s, 0.0, 2.0 * Yref)
    tol = 1e-10 if dt == "f64" else 2e-4
    assert _relnorm(host(Y), Yref) <= tol
    assert _relnorm(host(Xd.grad), dX_ref) <= tol
    assert _relnorm(host(theta.grad), dval_ref) <= tol
    if dt == "f64":
        # central differences on a few values, through the GPU forward pass
        g = host(theta.grad)
        h = 1e-6
        for p in [0, 1234567 % A.nnz, A.nnz - 1, int(np.argmax(np.abs(g)))]:
            ys = []
            for sgn in (1, -1):
                th = torch.tensor(A.val, dtype=torch.float64, device="cuda:0")
                th[p] += sgn * h
                with torch.no_grad():
                    ys.append(host(chebyshev(th, torch.tensor(X, device="cuda:0"), M, N, s, 0.0, K)))
            # L(+h) - L(-h) = sum (y+ - y-)(y+ + y-): no cancellation between two large sums
            fd = float(np.sum((ys[0] - ys[1]) * (ys[0] + ys[1]))) / (2 * h)
            assert abs(fd - g[p]) <= 1e-6 * max(abs(fd), 1e-3 * np.abs(g).max()), p
    M.close()


@pytest.mark.parametrize("n,b", [(262144 * 16 + 5, 33), (262144 * 16 * 2 + 17, 40)])
def test_grad_values_past_one_pass_of_workgroups(sc, n, b):
    """More rows than the gradient kernel's largest grid takes at once (16 a workgroup from 33 columns
    on): one entry a row, each G[i] . X[col i], and exactly nothing beside the gradient."""
    import torch

    gen = torch.Generator("cuda:0").manual_seed(223)
    rp = torch.arange(n + 1, dtype=torch.int64, device="cuda:0")
    col = torch.randint(0, 5000, (n,), dtype=torch.int32, device="cuda:0", generator=gen)
    M = sc.SellMatrix.from_device_csr(n, 5000, rp, col, torch.ones(n, dtype=torch.float64, device="cuda:0"), C=32, sigma=1,
                                      dtype="f32")
    G = torch.randint(-8, 9, (n, b), dtype=torch.int32, device="cuda:0", generator=gen).float()
    X = torch.randint(-8, 9, (5000, b), dtype=torch.int32, device="cuda:0", generator=gen).float()
    out = torch.full((n + 2,), 5.0, dtype=torch.float64, device="cuda:0")
    sc.sell_grad_values(M, G, X, out[1:n + 1])
    assert torch.equal(out[1:n + 1], (G * X[col.long()]).sum(1).double())
    assert float(out[0]) == 5.0 and float(out[n + 1]) == 5.0
    M.close()


@pytest.mark.parametrize("b", [1, 3, 8, 33])
@pytest.mark.parametrize("alpha,g,x", [(2.0 ** -600, 2.0 ** -600, 2.0 ** 900), (2.0 ** 600, 2.0 ** 600, 2.0 ** -900),
                                       (2.0 ** -1000, 2.0 ** -60, 2.0 ** 500)])
def test_grad_values_factor_leaves_the_range_in_order(sc, b, alpha, g, x):
    """alpha times the outer products, not the outer products of scaled rows: factors that leave the
    range of a double against G, but not against the sums, change nothing (exact, powers of two)."""
    import torch

    A = synth.random_sparse(60, 40, 0.1, 224, empty_rows=3)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    G, X = synth.int_block_vector(A.nrows, b, 225), synth.int_block_vector(A.ncols, b, 226)
    dval = torch.zeros(A.nnz, dtype=torch.float64, device="cuda:0")
    sc.sell_grad_values(M, dev(g * G), dev(x * X), dval, alpha=alpha)
    assert np.array_equal(host(dval), alpha * (g * x * oracle.pattern_outer(A, G, X)))
    M.close()


@pytest.mark.parametrize("N", [1, 2, 7])
def test_chebyshev_gradient_of_far_scales(sc, N):
    """A matrix with its scale, the block and the incoming gradient taken far from one by powers of two:
    the value gradient is the ordinary one, scaled."""
    import torch

    A, s, X = _anderson_case(6, 2, 227)
    G = synth.block_vector(A.nrows, 2, 228)
    outs = []
    for fm, fx, fg in ((1.0, 1.0, 1.0), (2.0 ** -500, 2.0 ** -400, 2.0 ** 600)):
        M = sc.SellMatrix.from_csr(synth.CSR(A.nrows, A.ncols, A.rowptr, A.col, fm * A.val), C=32, sigma=1)
        ck = torch.empty(sc.cheb_ckpt_elems(A.nrows, 2, N, 3), dtype=torch.float64, device="cuda:0")
        Xd, Gd = dev(fx * X), dev(fg * G)
        Y, dX = torch.empty_like(Xd), torch.empty_like(Xd)
        dval = torch.empty(A.nnz, dtype=torch.float64, device="cuda:0")
        sc.sell_cheb_forward(M, Xd, Y, N, fm * s, 0.0, 3, ck)
        sc.sell_cheb_backward(M, Gd, N, fm * s, 0.0, 3, ck, dX, dval)
        outs.append(host(dval) * fm / fg / fx)
        M.close()
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("N,K,b", [(9, 4, 1), (12, 2, 3), (40, 25, 1)])
def test_chebyshev_backward_without_room_for_groups(sc, N, K, b):
    """With no memory for the adjoint vectors of several steps the backward pass takes a step at a time;
    the other allocations still fail as out of memory, and nothing is left behind either way."""
    import torch

    A, s, X = _anderson_case(7, b, 229)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    G = dev(synth.block_vector(A.nrows, b, 230))
    ck = torch.empty(sc.cheb_ckpt_elems(A.nrows, b, N, K), dtype=torch.float64, device="cuda:0")
    Y = torch.empty((A.nrows, b), dtype=torch.float64, device="cuda:0")
    sc.sell_cheb_forward(M, dev(X), Y, N, s, 0.2, K, ck)

    def backward():
        dX, dval = torch.empty_like(G), torch.full((A.nnz,), float("nan"), dtype=torch.float64, device="cuda:0")
        sc.sell_cheb_backward(M, G, N, s, 0.2, K, ck, dX, dval)
        return host(dX), host(dval)

    want = backward()
    live = sc.sell_debug_live_allocs()
    failed = 0
    for k in range(1, 5):
        sc.sell_debug_fail_alloc(k)
        try:
            dX, dval = backward()
            assert np.array_equal(dX, want[0]) and _relnorm(dval, want[1]) <= 1e-13
        except sc.SellError as e:
            assert e.code == sc.SELL_ERR_OOM
            failed += 1
        finally:
            sc.sell_debug_fail_alloc(0)
        torch.cuda.synchronize()
        assert sc.sell_debug_live_allocs() == live
    assert failed == (1 if min(K, N) > 2 else 0)
    M.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("b", [1, 2, 4, 8, 12])
def test_chebyshev_of_operands_aligned_to_an_element(sc, b, dt):
    """The Chebyshev calls with every operand one element into a larger buffer (rows that the
    compiled widths' vector accesses may not touch): bit for bit the aligned calls, the inputs unchanged,
    nothing written beside the outputs."""
    import torch

    A, s, X0 = _anderson_case(7, b, 244)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1, dtype=dt)
    vt = torch.float64 if dt == "f64" else torch.float32
    n, N, K = A.nrows, 7, 3
    G0 = synth.block_vector(n, b, 245)
    elems = sc.cheb_ckpt_elems(n, b, N, K)
    coef = np.linspace(1.0, 0.2, N + 1)
    outs = []
    for off in (0, 1):
        bufs = []

        def buf(count, init=None):
            t = torch.full((count + 2,), 9.0, dtype=vt, device="cuda:0")
            bufs.append((t, count))
            v = t[off:off + count]
            if init is not None:
                v.copy_(torch.from_numpy(init).reshape(-1))
            return v

        X, G = buf(n * b, X0).view(n, b), buf(n * b, G0).view(n, b)
        Xc, Gc = X.clone(), G.clone()
        Y, dX, Z = (buf(n * b).view(n, b) for _ in range(3))
        ck = buf(elems)
        dval = torch.empty(A.nnz, dtype=torch.float64, device="cuda:0")
        sc.sell_cheb_forward(M, X, Y, N, s, 0.2, K, ck)
        sc.sell_cheb_backward(M, G, N, s, 0.2, K, ck, dX, dval)
        sc.sell_cheb_filter(M, X, coef, s, 0.2, Z=Z)
        assert torch.equal(X, Xc) and torch.equal(G, Gc)
        for t, count in bufs:
            assert bool((t[:off] == 9.0).all()) and bool((t[off + count:] == 9.0).all())
        outs.append([v.clone() for v in (Y, dX, Z, ck, dval)])
    assert all(torch.equal(u, v) for u, v in zip(*outs))
    M.close()


@pytest.mark.parametrize("N,K,b", [(1, 1, 1), (5, 1, 2), (6, 3, 1), (8, 3, 4)])
def test_chebyshev_operands_inside_the_checkpoints(sc, N, K, b):
    """X, then Y, anywhere in the checkpoint buffer (whole blocks and across two): the results and the
    checkpoints of separate buffers, the final Y over them."""
    import torch

    A, s, X0 = _anderson_case(6, b, 246)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    n = A.nrows
    elems, vb = sc.cheb_ckpt_elems(n, b, N, K), n * b
    X, Y, ck = dev(X0), torch.empty((n, b), dtype=torch.float64, device="cuda:0"), torch.empty(elems, dtype=torch.float64, device="cuda:0")
    sc.sell_cheb_forward(M, X, Y, N, s, 0.2, K, ck)
    for at in sorted({0, vb, vb // 2 * 2, elems - vb, max(0, elems - vb - vb // 2)}):
        c = torch.zeros(elems, dtype=torch.float64, device="cuda:0")
        xin, y = c[at:at + vb].view(n, b), torch.empty_like(Y)
        xin.copy_(X)
        sc.sell_cheb_forward(M, xin, y, N, s, 0.2, K, c)
        assert torch.equal(y, Y) and torch.equal(c, ck)
        c, want = torch.zeros_like(c), ck.clone()
        sc.sell_cheb_forward(M, X, c[at:at + vb].view(n, b), N, s, 0.2, K, c)
        want[at:at + vb] = Y.reshape(-1)
        assert torch.equal(c, want)
    M.close()


@pytest.mark.parametrize("accumulate", [False, True])
def test_value_gradient_over_its_inputs(sc, accumulate):
    """dval over G, over X, and over the checkpoints or the incoming gradient of a Chebyshev step: as
    into a buffer of its own."""
    import torch

    A, s, X0 = _anderson_case(6, 3, 247)
    M = sc.SellMatrix.from_csr(A, C=32, sigma=1)
    n, b, N, K = A.nrows, 3, 6, 2
    G0 = synth.block_vector(n, b, 248)
    size = max(A.nnz, sc.cheb_ckpt_elems(n, b, N, K)) + 8
    for which in ("G", "X"):
        buf = torch.zeros(size, dtype=torch.float64, device="cuda:0")
        v = buf[3:3 + n * b].view(n, b)
        v.copy_(torch.from_numpy(G0 if which == "G" else X0))
        other = dev(X0 if which == "G" else G0)
        want = buf[:A.nnz].clone()
        args = (v, other) if which == "G" else (other, v)
        sc.sell_grad_values(M, *(t.clone() for t in args), want, alpha=0.5, accumulate=accumulate)
        sc.sell_grad_values(M, *args, buf[:A.nnz], alpha=0.5, accumulate=accumulate)
        assert torch.equal(buf[:A.nnz], want)
    Y, dX = torch.empty((n, b), dtype=torch.float64, device="cuda:0"), torch.empty((n, b), dtype=torch.float64, device="cuda:0")
    ck, want = (torch.zeros(size, dtype=torch.float64, device="cuda:0") for _ in range(2))
    sc.sell_cheb_forward(M, dev(X0), Y, N, s, 0.2, K, ck)
    sc.sell_cheb_backward(M, dev(G0), N, s, 0.2, K, ck, dX, want)
    c = ck.clone()
    dX2 = torch.empty_like(dX)
    sc.sell_cheb_backward(M, dev(G0), N, s, 0.2, K, c, dX2, c)
    assert torch.equal(c[:A.nnz], want[:A.nnz]) and torch.equal(dX2, dX)
    buf = torch.zeros(size, dtype=torch.float64, device="cuda:0")
    g = buf[5:5 + n * b].view(n, b)
    g.copy_(torch.from_numpy(G0))
    sc.sell_cheb_backward(M, g, N, s, 0.2, K, ck, dX2, buf)
    assert torch.equal(buf[:A.nnz], want[:A.nnz]) and torch.equal(dX2, dX)
    M.close()
