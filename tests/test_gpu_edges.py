"""Kernels at the sizes where their tiling can go wrong (tile edges, remainders, row and column
splits, unaligned bases), each against plain binary64 arithmetic."""
import numpy as np
import pytest
import torch

import paper_2211_13028_amd as rt

pytestmark = pytest.mark.gpu


def _dev(a, dtype=torch.float64, skew=0):
    """`a` on the GPU, `skew` elements past an aligned base."""
    t = torch.from_numpy(np.ascontiguousarray(a)).to(dtype)
    buf = torch.empty(t.numel() + skew, dtype=dtype, device="cuda")
    out = buf[skew:].view(t.shape)
    out.copy_(t)
    return out


# ------------------------------------------------------------------ explicit residual
# 64-column waves, 256-column workgroups, 16-row blocks, 64-row chunks, ranges of >= 128 rows;
# r1 in each of the five k lengths.  Values are exact in every dtype (multiples of 1/8), so the
# binary64 sums differ by their order only: 4096 terms of one sign, 4096 * 2^-53 < 1e-12.
@pytest.mark.parametrize("dims,r,dtype,skew", [
    ((16, 8, 8), (1, 2, 2), torch.float64, 0),
    ((17, 9, 7), (9, 3, 2), torch.float32, 0),
    ((129, 16, 16), (16, 4, 4), torch.bfloat16, 0),
    ((300, 13, 20), (17, 5, 3), torch.float32, 0),
    ((300, 13, 20), (24, 5, 3), torch.float32, 1),
    ((65, 5, 53), (25, 5, 7), torch.bfloat16, 3),
    ((257, 12, 24), (33, 4, 9), torch.float32, 0),
    ((128, 257), (64, 40), torch.float64, 1),
])
@pytest.mark.parametrize("bad", [False, True])
def test_rel_error_tiles(dims, r, dtype, skew, bad):
    rng = np.random.default_rng(sum(dims))
    X = rng.integers(-16, 17, size=dims) / 8.0
    G = rng.integers(-4, 5, size=r) / 4.0
    Us = [rng.integers(-4, 5, size=(n, k)) / 8.0 for n, k in zip(dims, r)]
    xh = G
    for k, U in enumerate(Us):
        xh = np.moveaxis(np.tensordot(xh, U, axes=([k], [1])), -1, k)
    nbad = 0
    if bad:
        flat = X.reshape(-1)
        where = np.array([0, flat.size // 2, flat.size - 1])
        flat[where] = [np.nan, np.inf, -np.inf]
        nbad = 3
    fin = np.isfinite(X)
    res2, x2 = float(((X - xh)[fin] ** 2).sum()), float((X[fin] ** 2).sum())
    e, n = rt.rtucker_rel_error(_dev(X, dtype, skew), _dev(G), [_dev(U) for U in Us], allow_nonfinite=True)
    assert n["nonfinite"] == nbad
    assert abs(n["res2"] - res2) <= 1e-12 * res2
    assert abs(n["x2"] - x2) <= 1e-12 * x2
    assert abs(n["g2"] - float((G ** 2).sum())) <= 1e-12 * float((G ** 2).sum())
    assert abs(e - (res2 / x2) ** 0.5) <= 1e-12 * e


# ------------------------------------------------------------------ QR factorisation
# 16-column panels: one column, panel edges +-1, the widest; one row more than a 64-row chunk.
# Singular values are within a factor of ten, so Q and R move by at most a few hundred roundings.
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("extra", [0, 1, 65])
def test_qr_panels(n, extra):
    m = max(n, 64 * (n // 64)) + extra
    rng = np.random.default_rng(100 * n + extra)
    u, _ = np.linalg.qr(rng.standard_normal((m, n)))
    v, _ = np.linalg.qr(rng.standard_normal((n, n)))
    Y = (u * np.linspace(1.0, 0.1, n)) @ v.T
    Q, R = rt.rtucker_qr(_dev(Y), want_r=True)
    Q, R = Q.cpu().numpy(), R.cpu().numpy()
    q, r = np.linalg.qr(Y)
    s = np.where(np.diagonal(r) < 0, -1.0, 1.0)
    assert np.all(np.tril(R, -1) == 0.0) and np.all(np.diagonal(R) > 0.0)
    assert np.abs(Q.T @ Q - np.eye(n)).max() <= 1e-13
    assert np.abs(Q - q * s).max() <= 1e-12
    assert np.abs(R - r * s[:, None]).max() <= 1e-12


# a column that repeats another one has to reach the Householder path from any panel
@pytest.mark.parametrize("n,dup", [(5, 4), (17, 16), (33, 20), (49, 48), (64, 40)])
def test_qr_breakdown_in_any_panel(n, dup):
    rng = np.random.default_rng(n)
    Y = rng.standard_normal((130, n))
    Y[:, dup] = Y[:, 0]
    Q = rt.rtucker_qr(_dev(Y)).cpu().numpy()
    assert np.abs(Q.T @ Q - np.eye(n)).max() <= 1e-13
    assert np.abs(Q @ (Q.T @ Y) - Y).max() <= 1e-12 * np.abs(Y).max()


# ------------------------------------------------------------------ binary32 sketch pass
# 128-column waves (1, 2 or 4 a slab, several column blocks), 16-row steps, 64-row windows, row
# splits, last slab of a workgroup; rows that start at any 4-byte boundary and are cut by the end
# of the tensor.  Each entry is a binary32 sum of at most 1100 products: 1100 * 2^-24 < 7e-5 of the
# sum of their magnitudes.
@pytest.mark.parametrize("dims,sp,sl", [
    ((5, 16, 16), 3, 2), ((5, 17, 19), 4, 8), ((4, 63, 127), 8, 5), ((7, 65, 128), 3, 3), ((3, 64, 129), 2, 7),
    ((2, 3, 130, 131), 5, 4), ((6, 80, 255), 4, 4), ((3, 81, 257), 7, 6), ((2, 100, 389), 7, 7),
    ((1, 700, 513), 3, 8), ((2, 40, 640), 8, 1), ((1, 1100, 66), 5, 5), ((1, 33, 1027), 6, 2),
])
@pytest.mark.parametrize("want", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("skew", [0, 1])
def test_sketch_pass_f32_tiles(dims, sp, sl, want, skew):
    rng = np.random.default_rng(sum(dims) + sp)
    X = rng.standard_normal(dims).astype(np.float32).astype(np.float64)
    fp = rng.standard_normal((sp, dims[-2])).astype(np.float32).astype(np.float64)
    fl = rng.standard_normal((sl, dims[-1])).astype(np.float32).astype(np.float64)
    Z, W = rt.rtucker_sketch_pass(_dev(X, torch.float32, skew), _dev(fp), _dev(fl), want=want)
    for got, on, ref, mag in ((Z, want[0], X @ fl.T, np.abs(X) @ np.abs(fl).T),
                              (W, want[1], fp @ X, np.abs(fp) @ np.abs(X))):
        assert (got is not None) == on
        if on:
            assert np.all(np.abs(got.double().cpu().numpy() - ref) <= 7e-5 * mag)


def test_sketch_pass_f32_nonfinite_stays_in_its_row_and_column():
    dims = (3, 40, 77)
    X = np.ones(dims)
    X[1, 17, 76] = np.inf
    Z, W = rt.rtucker_sketch_pass(_dev(X, torch.float32), _dev(np.ones((2, 40))), _dev(np.ones((2, 77))))
    Z, W = Z.cpu().numpy(), W.cpu().numpy()
    want_z = np.full((3, 40, 2), 77.0)
    want_z[1, 17] = np.inf
    want_w = np.full((3, 2, 77), 40.0)
    want_w[1, :, 76] = np.inf
    assert np.array_equal(Z, want_z) and np.array_equal(W, want_w)


# ------------------------------------------------------------------ binary32 contraction in three bfloat16 terms
# 64-column waves, four a workgroup (eight on much longer rows or k ranges), 16-row tiles of M with
# one row more, 32-k blocks, 64-k windows, splits of k, rows at any 4-byte boundary.  A binary32
# sum of K products is within (K + 8) 2^-24 of the sum of their magnitudes in any order; the
# matrix cores may truncate where an addition rounds, hence twice that.
def _contract(X, U, skew=0):
    G = rt.rtucker_core(_dev(X, torch.float32, skew), [None, _dev(U), None], modes=[1])
    return G.double().cpu().numpy()


@pytest.mark.parametrize("shape,m", [
    ((1, 1, 64), 1), ((1, 5, 65), 16), ((3, 31, 67), 17), ((2, 33, 127), 33), ((5, 64, 130), 32), ((2, 65, 191), 49),
    ((1, 100, 640), 64), ((7, 512, 66), 18), ((3, 513, 70), 17), ((2, 1030, 131), 49), ((9, 1100, 64), 33),
    ((1, 2050, 257), 48), ((33, 96, 64), 50), ((1, 4000, 64), 3),
])
@pytest.mark.parametrize("skew", [0, 3])
def test_contraction_f32_tiles(shape, m, skew):
    rng = np.random.default_rng(sum(shape) + m)
    X = rng.standard_normal(shape).astype(np.float32).astype(np.float64)
    U = rng.standard_normal((shape[1], m)).astype(np.float32).astype(np.float64)
    got = _contract(X, U, skew)
    ref = np.einsum("akb,km->amb", X, U)
    mag = np.einsum("akb,km->amb", np.abs(X), np.abs(U))
    assert np.all(np.abs(got - ref) <= 2 * (shape[1] + 8) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("K,m", [(70, 20), (600, 49)])
def test_contraction_f32_nonfinite(K, m):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((2, K, 96)).astype(np.float32).astype(np.float64)
    U = rng.standard_normal((K, m)).astype(np.float32).astype(np.float64)
    X[0, 3, 5], X[1, K - 1, 95], X[1, 40, 64] = np.inf, -np.inf, np.nan
    got = _contract(X, U)
    assert np.array_equal(got[0, :, 5], np.sign(U[3]) * np.inf)
    assert np.array_equal(got[1, :, 95], -np.sign(U[K - 1]) * np.inf)
    assert np.all(np.isnan(got[1, :, 64]))
    bad = np.zeros((2, 96), dtype=bool)
    bad[0, 5] = bad[1, 95] = bad[1, 64] = True
    fin = np.moveaxis(got, 1, 2)[~bad]
    Xf = np.where(np.isfinite(X), X, 0.0)
    ref = np.moveaxis(np.einsum("akb,km->amb", Xf, U), 1, 2)[~bad]
    mag = np.moveaxis(np.einsum("akb,km->amb", np.abs(Xf), np.abs(U)), 1, 2)[~bad]
    assert np.all(np.abs(fin - ref) <= 2 * (K + 8) * 2.0 ** -24 * mag)


# scales where a term of x or M leaves bfloat16's range; every product and sum stays in binary32's
# (the last row: its subnormals, hence the absolute part)
@pytest.mark.parametrize("sx,su", [(2.0 ** -60, 1.0), (2.0 ** -110, 1.0), (2.0 ** -125, 1.0), (2.0 ** 100, 2.0 ** -110),
                                   (2.0 ** -110, 2.0 ** 100), (2.0 ** 118, 1.0), (2.0 ** -140, 1.0)])
@pytest.mark.parametrize("K,m", [(90, 33), (700, 17)])
def test_contraction_f32_scales(sx, su, K, m):
    rng = np.random.default_rng(K + m)
    X = (rng.standard_normal((1, K, 72)) * sx).astype(np.float32).astype(np.float64)
    U = (rng.standard_normal((K, m)) * su).astype(np.float32).astype(np.float64)
    got = _contract(X, U)
    ref = np.einsum("akb,km->amb", X, U)
    mag = np.einsum("akb,km->amb", np.abs(X), np.abs(U))
    assert np.all(np.abs(got - ref) <= 2 * (K + 8) * 2.0 ** -24 * mag + K * 2.0 ** -149)


def test_contraction_f32_largest_entry():
    X = np.zeros((1, 64, 64))
    X[0, 7, 9] = float(np.finfo(np.float32).max)
    U = np.zeros((64, 20))
    U[7, 19] = 0.5
    ref = np.zeros((1, 20, 64))
    ref[0, 19, 9] = 0.5 * X[0, 7, 9]
    assert np.array_equal(_contract(X, U), ref)


# ------------------------------------------------------------------ bfloat16 contraction
# 128-column waves (eight columns a lane, at any 2-byte boundary), 16-row tiles of M, 32-k blocks, 64-k
# windows, rows past the range.  Products of bfloat16 values are exact; binary32 sums as above.
@pytest.mark.parametrize("shape,m", [
    ((256, 1, 64), 1), ((250, 5, 65), 16), ((130, 31, 131), 17), ((256, 33, 71), 33), ((43, 64, 390), 32),
    ((256, 65, 127), 49), ((3, 100, 16001), 64), ((128, 513, 129), 18), ((2, 96, 136), 20), ((300, 200, 64), 50),
])
@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("bad", [False, True])
def test_contraction_bf16_tiles(shape, m, skew, bad):
    rng = np.random.default_rng(sum(shape) + m)
    X = torch.from_numpy(rng.standard_normal(shape)).to(torch.bfloat16).double().numpy()
    U = torch.from_numpy(rng.standard_normal((shape[1], m))).to(torch.bfloat16).double().numpy()
    fin = np.ones((shape[0], shape[2]), dtype=bool)
    if bad:
        X[0, shape[1] - 1, shape[2] - 1] = np.inf
        fin[0, shape[2] - 1] = False
    got = rt.rtucker_core(_dev(X, torch.bfloat16, skew), [None, _dev(U), None], modes=[1]).double().cpu().numpy()
    Xf = np.where(np.isfinite(X), X, 0.0)
    ref = np.moveaxis(np.einsum("akb,km->amb", Xf, U, optimize=True), 1, 2)[fin]
    mag = np.moveaxis(np.einsum("akb,km->amb", np.abs(Xf), np.abs(U), optimize=True), 1, 2)[fin]
    assert np.all(np.abs(np.moveaxis(got, 1, 2)[fin] - ref) <= 2 * (shape[1] + 8) * 2.0 ** -24 * mag)
    if bad:
        want = np.sign(U[-1]) * np.inf
        assert np.array_equal(got[0, :, -1][U[-1] != 0], want[U[-1] != 0])


# ------------------------------------------------------------------ contraction of the contiguous last mode
# 64-row waves, 16-row tiles of M, 16-k (binary32) or 32-k (bfloat16) steps cut anywhere by the row's end,
# splits of k, rows at any boundary.
@pytest.mark.parametrize("shape,m", [((4, 1, 5), 1), ((2, 3, 16), 16), ((63, 1, 31), 17), ((13, 5, 33), 33), ((2, 64, 63), 64),
                                     ((3, 43, 130), 20), ((65, 1, 257), 49), ((40, 50, 519), 24)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("bad", [False, True])
def test_contraction_last_mode_tiles(shape, m, dtype, skew, bad):
    rng = np.random.default_rng(sum(shape) + m)
    K = shape[2]
    X = torch.from_numpy(rng.standard_normal(shape)).to(dtype).double().numpy()
    U = torch.from_numpy(rng.standard_normal((K, m))).to(dtype).double().numpy()
    fin = np.ones(shape[:2], dtype=bool)
    if bad:
        X[-1, -1, K - 1] = np.inf
        fin[-1, -1] = False
    got = rt.rtucker_core(_dev(X, dtype, skew), [None, None, _dev(U)], modes=[2]).double().cpu().numpy()
    Xf = np.where(np.isfinite(X), X, 0.0)
    assert np.all(np.abs(got - Xf @ U)[fin] <= (2 * (K + 8) * 2.0 ** -24 * (np.abs(Xf) @ np.abs(U)))[fin])
    if bad:
        assert np.array_equal(got[-1, -1], np.sign(U[-1]) * np.inf)


# ------------------------------------------------------------------ 16- and 8-bit sketch pass
# 128-column waves (1, 2 or 4 a slab, several column blocks), 32-row steps, eight-row and eight-column groups
# cut anywhere, row splits, rows at any boundary.  The products are exact; binary32 sums as above.
@pytest.mark.parametrize("dims,sp,sl", [
    ((5, 16, 16), 3, 2), ((5, 17, 19), 4, 8), ((4, 63, 127), 8, 5), ((7, 65, 128), 3, 3), ((3, 64, 129), 2, 7),
    ((2, 3, 130, 131), 5, 4), ((6, 80, 255), 4, 4), ((3, 81, 257), 7, 6), ((2, 100, 389), 7, 7),
    ((1, 700, 513), 3, 8), ((2, 40, 640), 8, 1), ((1, 1100, 66), 5, 5), ((1, 33, 1027), 6, 2), ((2, 96, 512), 4, 4),
])
@pytest.mark.parametrize("want", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float8_e4m3fn])
@pytest.mark.parametrize("skew", [0, 1])
def test_sketch_pass_narrow_tiles(dims, sp, sl, want, dtype, skew):
    rng = np.random.default_rng(sum(dims) + sp)

    def draw(shape):  # multiples of 1/8 up to 15/8 are exact in both types
        return rng.integers(-15, 16, size=shape) / 8.0

    X, fp, fl = draw(dims), draw((sp, dims[-2])), draw((sl, dims[-1]))
    Xd = _dev(X, torch.float32).to(dtype)
    if skew:
        buf = torch.zeros(Xd.numel() + 1, dtype=dtype, device="cuda")
        buf.view(torch.uint8)[Xd.element_size():] = Xd.reshape(-1).view(torch.uint8)
        Xd = buf[1:].view(dims)
    Z, W = rt.rtucker_sketch_pass(Xd, _dev(fp), _dev(fl), want=want)
    for got, on, ref, mag in ((Z, want[0], X @ fl.T, np.abs(X) @ np.abs(fl).T),
                              (W, want[1], fp @ X, np.abs(fp) @ np.abs(X))):
        assert (got is not None) == on
        if on:
            assert np.all(np.abs(got.double().cpu().numpy() - ref) <= 1.4e-4 * mag)


def test_sketch_pass_bf16_nonfinite_stays_in_its_row_and_column():
    dims = (3, 40, 77)
    X = np.ones(dims)
    X[1, 17, 76] = np.inf
    Z, W = rt.rtucker_sketch_pass(_dev(X, torch.bfloat16), _dev(np.ones((2, 40))), _dev(np.ones((2, 77))))
    Z, W = Z.cpu().numpy(), W.cpu().numpy()
    want_z = np.full((3, 40, 2), 77.0)
    want_z[1, 17] = np.inf
    want_w = np.full((3, 2, 77), 40.0)
    want_w[1, :, 76] = np.inf
    assert np.array_equal(Z, want_z) and np.array_equal(W, want_w)


@pytest.mark.parametrize("dims,skew", [
    ((65, 7, 5), 0), ((65, 16, 16), 0), ((65, 16, 16), 1), ((127, 9, 10), 0), ((128, 2, 32), 0), ((129, 67, 3), 0),
    ((192, 64, 3), 0), ((193, 5, 7), 1), ((257, 40, 33), 0), ((70, 1, 1), 0), ((66, 300, 301), 0),
])
def test_gram_and_subspace_of_a_long_mode(dims, skew):
    """Leading eigenvectors of the first mode's Gram matrix, M V = V diag(theta), at the edges of its
    64-wide tiles, for each of its loads and where M has fewer than 64 eigenvalues above zero.

    The iteration stops at a residual of 1e-12 theta_1; the two sums of M differ by rounding in
    chunks of at most a few thousand terms, under 1e-12 of its norm, so 2e-12 theta_1 bounds both.
    """
    rng = np.random.default_rng(sum(dims))
    n, rest = dims[0], dims[1] * dims[2]
    k = min(3, rest)
    core = np.diag(10.0 * 0.5 ** np.arange(k))
    left = np.linalg.qr(rng.standard_normal((n, k)))[0]
    right = np.linalg.qr(rng.standard_normal((rest, k)))[0]
    X = (left @ core @ right.T + 1e-4 * rng.standard_normal((n, rest))).reshape(dims).astype(np.float32)
    r = [k, 1, 1]
    _, Us, _ = rt.rtucker_sthosvd(_dev(X, torch.float32, skew), r)
    V = Us[0].cpu().numpy()
    M = X.reshape(n, -1).astype(np.float64)
    M = M @ M.T
    theta = np.diag(V.T @ M @ V)
    np.testing.assert_allclose(V.T @ V, np.eye(k), atol=1e-12)
    assert np.all(np.linalg.norm(M @ V - V * theta, axis=0) <= 2e-12 * theta[0])
    np.testing.assert_allclose(theta, np.linalg.eigvalsh(M)[::-1][:k], rtol=0, atol=2e-12 * theta[0])


# ------------------------------------------------------------------ batched sketch pass
# 64-column units (1 to 4 a row), the last one cut at any place, rows shorter than a 4-column
# group, 16-row steps, four slabs a workgroup.
@pytest.mark.parametrize("last", [(2, 3, 4, 5, 6), (15, 16, 17, 63, 64), (65, 66, 67, 68, 127), (128, 129, 130, 191, 192),
                                  (193, 194, 195, 255, 256)])
@pytest.mark.parametrize("skew", [0, 1])
def test_batched_sketch_tiles(last, skew):
    """Tensors of exact rank are recovered, whatever lies around them in memory.

    A sum of at most 256 binary32 products is good to 256 * 2^-24 = 1.5e-5 of its terms' norm and
    typically to 1e-6; a wrong column or row of a sketch costs at least 1 / 16 of the norm.
    """
    rng = np.random.default_rng(last[0])
    dims = [(a, p, q) for q, (a, p) in zip(last, [(9, 16), (4, 17), (5, 256), (31, 15), (256, 33)])]
    ranks = [[min(2, q)] * 3 for q in last]
    Xs = []
    for (a, p, q), r in zip(dims, ranks):
        u, v, w = (np.linalg.qr(rng.standard_normal((n, r[0])))[0] for n in (a, p, q))
        X = np.einsum("ir,jr,kr->ijk", u, v, w).astype(np.float32)
        buf = torch.full((X.size + 8 + skew,), float("nan"), dtype=torch.float32, device="cuda")
        t = buf[4 + skew:4 + skew + X.size].view(X.shape)
        t.copy_(torch.from_numpy(X))
        Xs.append(t)
    over = 2
    ss = [rt.rtucker_sketch_sizes(d, r, over, "rhkron") for d, r in zip(dims, ranks)]
    phis = [[_dev(rng.standard_normal((s[k], d[k]))) for k in range(3)] for s, d in zip(ss, dims)]
    Gs, Us = rt.Batch(Xs, ranks, over, phis, ss).run()
    for X, G, U, d in zip(Xs, Gs, Us, dims):
        X, G, U = X.cpu().numpy().astype(np.float64), G.cpu().numpy(), [u.cpu().numpy() for u in U]
        back = np.einsum("abc,ia,jb,kc->ijk", G, *U)
        assert np.linalg.norm(back - X) <= 1.5e-5 * np.linalg.norm(X), d


# ------------------------------------------------------------------ grouped contractions of a sketch
# Short last modes put the second level of the tree on the generic kernel: its contractions run as one
# launch when each has fewer than 32768 columns, with the sums of the split ones (K >= 128) in another.
@pytest.mark.parametrize("dims,s", [
    ((5, 6, 7), (2, 3, 2)), ((130, 129, 9), (3, 4, 5)), ((300, 17, 19), (7, 2, 3)), ((2, 513, 15), (2, 8, 3)),
    ((9, 8, 7, 6), (2, 3, 2, 3)), ((140, 3, 130, 5), (3, 2, 4, 3)), ((200, 190, 180), (5, 4, 3)), ((40, 600, 61), (8, 8, 7)),
])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("keep", [0b1111, 0b0110, 0b0001])
def test_sketch_second_level_groups(dims, s, dtype, keep):
    """Every unfolding against numpy; entries and operands are small integers over 8, so the products
    and, up to order, the binary32 sums are exact to 2^-24 per addition: K terms, K 2^-24 of their sum."""
    rng = np.random.default_rng(sum(dims))
    d = len(dims)
    X = rng.integers(-8, 9, dims) / 8.0
    phis = [rng.integers(-8, 9, (s[k], dims[k])) / 8.0 for k in range(d)]
    modes = [n for n in range(d) if keep >> n & 1]
    Ys = rt.rtucker_sketch(_dev(X, dtype), [_dev(p) for p in phis], list(s), modes)
    for n in range(d):
        if n not in modes:
            assert Ys[n] is None
            continue
        want, bound = X, np.abs(X)
        for k in range(d):
            if k != n:
                want = np.moveaxis(np.tensordot(phis[k], want, (1, k)), 0, k)
                bound = np.moveaxis(np.tensordot(np.abs(phis[k]), bound, (1, k)), 0, k)
        want, bound = (np.moveaxis(v, n, 0).reshape(dims[n], -1) for v in (want, bound))
        unit = 2.0 ** -53 if dtype == torch.float64 else 2.0 ** -24
        got = Ys[n].cpu().double().numpy()
        assert np.all(np.abs(got - want) <= sum(dims) * unit * bound + 1e-300), (n, np.abs(got - want).max())


# binary32 rows off the 16-byte grid, on both sides of the rule that sends small grids to the vector ALU: 400 row
# ranges up to 256 columns (200 past s = 4), 200 (64) beyond; up to 16 row ranges a slab, one of them cut
@pytest.mark.parametrize("dims,s", [((1, 16, 17), 3), ((399, 17, 18), 4), ((400, 17, 18), 4), ((199, 130, 45), 5), ((200, 130, 45), 5),
                                    ((199, 21, 257), 4), ((200, 21, 257), 4), ((63, 33, 258), 8), ((64, 33, 258), 8),
                                    ((2, 1031, 91), 8), ((12, 520, 513), 3)])
@pytest.mark.parametrize("want", [(True, True), (True, False), (False, True)])
def test_f32_sketch_of_few_slabs(dims, s, want):
    A, P, Q = dims
    rng = np.random.default_rng(A + P + Q + s)
    f32 = lambda *n: rng.standard_normal(n).astype(np.float32).astype(np.float64)  # noqa: E731
    X, fP, fQ = f32(A, P, Q), f32(s, P), f32(s, Q)
    print("sketch pass", dims, s, want, flush=True)
    Z, W = rt.rtucker_sketch_pass(_dev(X, torch.float32), _dev(fP), _dev(fQ), want=want)
    if want[0]:
        bound = 2 * (Q + 8) * 2.0 ** -24 * (np.abs(X) @ np.abs(fQ).T)
        assert np.all(np.abs(Z.double().cpu().numpy() - X @ fQ.T) <= bound)
    if want[1]:
        bound = 2 * (P + 8) * 2.0 ** -24 * np.matmul(np.abs(fP), np.abs(X))
        assert np.all(np.abs(W.double().cpu().numpy() - np.matmul(fP, X)) <= bound)
