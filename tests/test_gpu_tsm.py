"""GPU parity of the tall-skinny block-vector kernels against the oracle (FP64)."""
import math

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


@pytest.mark.parametrize("n,m,k", [(0, 3, 2), (1, 1, 1), (1000, 8, 8), (100003, 5, 3), (20000, 64, 64),
                                   (7777, 17, 40)])
@pytest.mark.parametrize("kahan", [False, True])
def test_tsmttsm(sc, n, m, k, kahan):
    V = synth.block_vector(n, m, 160)
    W = synth.block_vector(n, k, 161)
    X0 = synth.block_vector(m, k, 162)
    Xd = dev(X0)
    sc.sell_tsmttsm(dev(V), dev(W), Xd, alpha=2.0, beta=-0.5, kahan=kahan)
    ref = oracle.tsmttsm(V, W, 2.0, -0.5, X0, kahan=kahan)
    scale = 2.0 * np.abs(V).T @ np.abs(W) + 0.5 * np.abs(X0)
    assert np.all(np.abs(host(Xd) - ref) <= 1e-12 * scale + 1e-300)


def test_tsmttsm_kahan_accuracy_on_gpu(sc):
    n = 200000
    a = synth.normal(163, n) * np.exp(synth.uniform(164, n, -15, 15))
    V = np.stack([a, np.ones(n)], axis=1)
    W = np.stack([synth.normal(165, n), -np.ones(n) * 1e-3], axis=1)
    Xd = dev(np.zeros((2, 2)))
    sc.sell_tsmttsm(dev(V), dev(W), Xd, kahan=True)
    X = host(Xd)
    for l in range(2):
        for j in range(2):
            exact = math.fsum((V[:, l] * W[:, j]).tolist())
            bound = 4.5e-16 * abs(exact) + 1.2e-16 * float(np.sum(np.abs(V[:, l] * W[:, j])))
            assert abs(X[l, j] - exact) <= bound


@pytest.mark.parametrize("m,k", [(8, 8), (4, 12), (16, 4)])
@pytest.mark.parametrize("kahan", [False, True])
def test_tsmttsm_aligned_path_equals_element_path(sc, m, k, kahan):
    """m and k multiples of 4 with 16-byte aligned rows take the 16-byte-load kernel; the same
    values in a buffer shifted by one double (rows 8 bytes off alignment) take the per-element
    kernel. Both visit every thread's rows in the same order: equal bit for bit, and within the
    oracle's bound."""
    import torch

    n = 123457
    V = synth.block_vector(n, m, 170 + m)
    W = synth.block_vector(n, k, 180 + k)
    out = []
    for off in (0, 1):
        vb = torch.zeros(n * m + 2, dtype=torch.float64, device="cuda:0")
        wb = torch.zeros(n * k + 2, dtype=torch.float64, device="cuda:0")
        Vd = vb[off:off + n * m].view(n, m)
        Wd = wb[off:off + n * k].view(n, k)
        Vd.copy_(dev(V))
        Wd.copy_(dev(W))
        assert (Vd.data_ptr() % 16 == 0) == (off == 0)
        Xd = torch.zeros((m, k), dtype=torch.float64, device="cuda:0")
        sc.sell_tsmttsm(Vd, Wd, Xd, kahan=kahan)
        out.append(host(Xd))
    assert np.array_equal(out[0], out[1])
    ref = oracle.tsmttsm(V, W, 1.0, 0.0, np.zeros((m, k)), kahan=kahan)
    assert np.all(np.abs(out[0] - ref) <= 1e-12 * (np.abs(V).T @ np.abs(W)) + 1e-300)


def test_tsmttsm_deterministic(sc):
    import torch

    V = dev(synth.block_vector(300001, 4, 166))
    W = dev(synth.block_vector(300001, 4, 167))
    X1 = torch.zeros((4, 4), dtype=torch.float64, device="cuda:0")
    X2 = torch.zeros_like(X1)
    sc.sell_tsmttsm(V, W, X1)
    sc.sell_tsmttsm(V, W, X2)
    torch.cuda.synchronize()
    assert torch.equal(X1, X2)


@pytest.mark.parametrize("n,m,k", [(1, 1, 1), (50000, 8, 8), (12345, 3, 17), (4096, 64, 64)])
def test_tsmm(sc, n, m, k):
    V = synth.block_vector(n, m, 168)
    X = synth.block_vector(m, k, 169)
    W0 = synth.block_vector(n, k, 170)
    Wd = dev(W0)
    sc.sell_tsmm(dev(V), dev(X), Wd, alpha=0.5, beta=2.0)
    ref = oracle.tsmm(V, X, 0.5, 2.0, W0)
    scale = 0.5 * np.abs(V) @ np.abs(X) + 2.0 * np.abs(W0)
    assert np.all(np.abs(host(Wd) - ref) <= 1e-13 * scale + 1e-300)


@pytest.mark.parametrize("n,m", [(1, 1), (50001, 8), (9999, 3), (3000, 64)])
def test_tsmm_inplace(sc, n, m):
    V = synth.block_vector(n, m, 171)
    X = synth.block_vector(m, m, 172)
    Vd = dev(V)
    sc.sell_tsmm_inplace(Vd, dev(X), alpha=1.5, beta=-0.5)
    ref = oracle.tsmm_inplace(V, X, 1.5, -0.5)
    scale = 1.5 * np.abs(V) @ np.abs(X) + 0.5 * np.abs(V)
    assert np.all(np.abs(host(Vd) - ref) <= 1e-13 * scale + 1e-300)


@pytest.mark.parametrize("m,k", [(16, 17), (17, 16), (32, 32), (33, 31), (48, 49), (64, 64), (63, 12), (12, 64), (64, 1), (1, 64),
                                 (2, 8), (24, 24), (7, 7), (9, 9)])
@pytest.mark.parametrize("n", [1, 15, 17, 129, 5000])
def test_matrix_core_blocks_every_edge(sc, n, m, k):
    """The matrix-core kernels where rows, columns and terms end inside a 16 x 16 x 4 block, one
    wave's rows and several workgroups', on contiguous blocks and on slices of wider ones at an odd
    offset: element by element within the bound of a sum of FP64 products, (terms + 6) u sum |v w|,
    and rows past the block and columns beside it untouched."""
    V, W = synth.block_vector(n, m, 170), synth.block_vector(n, k, 171)
    X, Q = synth.block_vector(m, k, 172), synth.block_vector(m, m, 173)
    u = 2.0 ** -53
    g = oracle.tsmttsm(V, W, 1.5, 0.0, np.zeros((m, k)))
    gb = 1.5 * (n + 6) * u * (np.abs(V).T @ np.abs(W)) * 2
    w = oracle.tsmm(V, X, -0.5, 0.25, W)
    wb = 2 * (m + 6) * u * (0.5 * np.abs(V) @ np.abs(X) + 0.25 * np.abs(W))
    v = oracle.tsmm_inplace(V, Q, 2.0, -0.5)
    vb = 2 * (m + 6) * u * (2.0 * np.abs(V) @ np.abs(Q) + 0.5 * np.abs(V))
    for off in (0, 3):
        import torch

        def block(a):
            t = torch.full((n + 1, a.shape[1] + off), 7.0, dtype=torch.float64, device="cuda:0")
            s = t[:n, off:]
            s.copy_(torch.from_numpy(a))
            return t, s

        Vt, Vs = block(V)
        Wt, Ws = block(W)
        Gd = dev(np.full((m, k), np.nan))
        sc.sell_tsmttsm(Vs, Ws, Gd, alpha=1.5)
        assert (np.abs(host(Gd) - g) <= gb).all()
        sc.sell_tsmm(Vs, dev(X), Ws, alpha=-0.5, beta=0.25)
        assert (np.abs(host(Ws) - w) <= wb).all()
        sc.sell_tsmm_inplace(Vs, dev(Q), alpha=2.0, beta=-0.5)
        assert (np.abs(host(Vs) - v) <= vb).all()
        for t in (Vt, Wt):
            assert (host(t)[n] == 7.0).all() and (host(t)[:, :off] == 7.0).all()


def test_matrix_core_blocks_keep_nonfinite_entries_in_their_places(sc):
    """A NaN or an infinity touches the row (V X) or the row and column (V^T W) it belongs to and
    nothing else, padding of the 16 x 16 x 4 blocks included."""
    n, m, k = 100, 35, 21
    V, W, X = synth.block_vector(n, m, 174), synth.block_vector(n, k, 175), synth.block_vector(m, k, 176)
    V[41, 34], W[99, 20] = np.nan, np.inf
    Gd, Wd = dev(np.zeros((m, k))), dev(W)
    sc.sell_tsmttsm(dev(V), Wd, Gd)
    bad = ~np.isfinite(host(Gd))
    want = np.zeros((m, k), bool)
    want[34, :] = want[:, 20] = True
    assert np.array_equal(bad, want)
    sc.sell_tsmm(dev(V), dev(X), Wd)
    bad = ~np.isfinite(host(Wd))
    want = np.zeros((n, k), bool)
    want[41, :] = True
    assert np.array_equal(bad, want)


@pytest.mark.parametrize("m", [9, 12, 15, 16, 17, 19, 20])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_narrow_update_either_side_of_the_matrix_cores(sc, m, k):
    """V X + beta W of one to three columns, where beta moves the line between the kernels: element by
    element within the bound of a sum of FP64 products, with and without beta."""
    n = 1000
    V, W, X = synth.block_vector(n, m, 178), synth.block_vector(n, k, 179), synth.block_vector(m, k, 180)
    for beta in (0.0, -0.5):
        Wd = dev(W)
        sc.sell_tsmm(dev(V), dev(X), Wd, alpha=1.5, beta=beta)
        bound = 2 * (m + 6) * 2.0 ** -53 * (1.5 * np.abs(V) @ np.abs(X) + abs(beta) * np.abs(W))
        assert (np.abs(host(Wd) - oracle.tsmm(V, X, 1.5, beta, W)) <= bound).all()
