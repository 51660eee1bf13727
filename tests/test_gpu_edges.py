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
