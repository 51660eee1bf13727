"""The binary32 contraction in three bfloat16 terms (64-column units; rows at any 4-byte boundary
where there are at least 256 units), against plain binary64 arithmetic."""
import numpy as np
import pytest
import torch

import paper_2211_13028_amd as rt

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _dev(a, dtype=torch.float64, skew=0):
    """`a` on the GPU, `skew` elements past an aligned base."""
    t = torch.from_numpy(np.ascontiguousarray(a)).to(dtype)
    buf = torch.empty(t.numel() + skew, dtype=dtype, device="cuda")
    out = buf[skew:].view(t.shape)
    out.copy_(t)
    return out


def _contract(X, U, skew=0):
    print("core", X.shape, U.shape, skew, flush=True)
    G = rt.rtucker_core(_dev(X, torch.float32, skew), [None, _dev(U), None], modes=[1])
    return G.double().cpu().numpy()


def _reference(X, U):
    f = lambda x, u: np.matmul(u.T, x)  # noqa: E731
    return f(X, U), f(np.abs(X), np.abs(U))


def _float32(rng, *shape):
    return rng.standard_normal(shape).astype(np.float32).astype(np.float64)


def _units(shape):
    return shape[0] * -(-shape[2] // 64)


# The last unit's columns overlap the one before it when the row ends 1 .. 3 columns into it.  A unit
# that holds an infinity is contracted once more with binary32 products: the columns of the unit
# before must be that unit's own, whichever of the two does so.
@pytest.mark.parametrize("tail", [1, 2, 3])
@pytest.mark.parametrize("where", ["before", "last"])
def test_every_column_has_one_owner(tail, where):
    rng = np.random.default_rng(tail)
    B = 64 * 256 + tail
    X, U = _float32(rng, 1, 40, B), _float32(rng, 40, 33)
    X[0, 7, B - 1 if where == "last" else B - tail - 20] = np.inf
    got = _contract(X, U)
    alone = _contract(X[:, :, :B - tail], U)
    assert np.array_equal(got[:, :, :B - tail], alone, equal_nan=True)


# Both operands are scaled by powers of two before they are split, and no size of M's entries short of
# binary32's limits changes the way a contraction is computed: a factor of 2^30 on M is a factor of
# 2^30 on every result, bit for bit.
@pytest.mark.parametrize("K,m", [(40, 20), (130, 49)])
@pytest.mark.parametrize("power", [-90, -30, 30])
def test_power_of_two_in_the_operand(K, m, power):
    rng = np.random.default_rng(K)
    X, U = _float32(rng, 2, K, 192), _float32(rng, K, m)
    assert np.array_equal(_contract(X, U * 2.0 ** power), _contract(X, U) * 2.0 ** power)


# results past 2^80 and entries past 2^104 are taken again with binary32 products, in blocks of 32 k
# with a remainder: entries one wave at a time, every row tile of M
@pytest.mark.parametrize("shape,m", [((1, 33, 128), 17), ((2, 70, 68), 33), ((1, 1, 16389), 5), ((130, 95, 131), 64)])
def test_results_outside_the_terms(shape, m):
    rng = np.random.default_rng(sum(shape))
    X, U = _float32(rng, *shape), _float32(rng, shape[1], m)
    X[0, :, 3] *= 2.0 ** 110
    X[-1, :, -1] *= 2.0 ** 90
    X[-1, shape[1] - 1, shape[2] // 2] = np.inf
    got = _contract(X, U)
    assert np.array_equal(got[-1, :, shape[2] // 2], np.sign(U[-1]) * np.inf)
    ref, mag = _reference(np.where(np.isfinite(X), X, 0.0), U)
    off = ~np.isfinite(X).all(axis=1)
    err = np.abs(np.moveaxis(got - ref, 1, 2))[~off]
    assert np.all(err <= 2 * (shape[1] + 8) * 2.0 ** -24 * np.moveaxis(mag, 1, 2)[~off])


# A sum that one product makes up is that product rounded once: the error's mean square against 64
# bits is that of the binary32 product, but for the dropped partial products.  (Each is the product of
# a second and a third term, at most 2^-8 and 2^-17 of x: two of them add less than a tenth.)
@pytest.mark.parametrize("shape", [(256, 1, 65), (1, 96, 16384)])
def test_one_product_is_rounded_once(shape):
    rng = np.random.default_rng(5)
    A, K, B = shape
    X = np.zeros(shape)
    X[:, K // 2] = _float32(rng, A, B)
    U = _float32(rng, K, 33)
    got = _contract(X, U)
    x, u = X[:, K // 2, None, :], U[K // 2][None, :, None]
    once = (x.astype(np.float32) * u.astype(np.float32)).astype(np.float64)
    rms = lambda y: float(np.sqrt(np.mean(((y - x * u) / (np.abs(x * u) + 1e-300)) ** 2)))  # noqa: E731
    assert rms(got) <= 1.1 * rms(once)


# the sums over k are no further from 64 bits than binary32 products summed four by four are
@pytest.mark.parametrize("K,spread", [(64, 0.0), (300, 0.0), (1024, 2.0)])
def test_error_of_the_sums(K, spread):
    rng = np.random.default_rng(K)
    X, U = _float32(rng, 2, K, 1024), _float32(rng, K, 33)
    X = (X * np.exp(spread * rng.standard_normal(X.shape))).astype(np.float32).astype(np.float64)
    ref, _ = _reference(X, U)
    acc = np.zeros((2, 33, 1024), dtype=np.float32)
    for k in range(0, K, 4):
        acc += np.matmul(U[k:k + 4].T, X[:, k:k + 4]).astype(np.float32)
    assert np.linalg.norm(_contract(X, U) - ref) <= np.linalg.norm(acc - ref)


# Binary32 products: up to 16 k (every count of row tiles of M, K on and off its 16-byte grid), and one
# row tile where there are at least 512 units of 128 columns.
@pytest.mark.parametrize("shape,m", [
    ((1, 1, 64), 1), ((2, 3, 68), 16), ((3, 4, 132), 17), ((1, 7, 256), 33), ((2, 13, 124), 48), ((5, 16, 128), 64),
    ((1, 15, 260), 49), ((512, 17, 64), 16), ((130, 50, 516), 9), ((600, 33, 68), 1), ((1, 130, 65536), 13),
    ((4096, 24, 64), 7), ((4096, 25, 64), 7), ((511, 40, 128), 11),
])
@pytest.mark.parametrize("bad", [False, True])
def test_binary32_products(shape, m, bad):
    rng = np.random.default_rng(sum(shape) + m)
    X, U = _float32(rng, *shape), _float32(rng, shape[1], m)
    fin = np.ones((shape[0], shape[2]), dtype=bool)
    if bad:
        X[-1, shape[1] - 1, shape[2] - 2] = -np.inf
        fin[-1, shape[2] - 2] = False
    got = _contract(X, U)
    ref, mag = _reference(np.where(np.isfinite(X), X, 0.0), U)
    err = np.abs(np.moveaxis(got - ref, 1, 2))[fin]
    assert np.all(err <= 2 * (shape[1] + 8) * 2.0 ** -24 * np.moveaxis(mag, 1, 2)[fin])
    if bad:
        assert np.array_equal(got[-1, :, shape[2] - 2], -np.sign(U[-1]) * np.inf)


# rows that start at any 4-byte boundary run on this kernel from 256 units on
@pytest.mark.parametrize("shape,m", [((256, 5, 65), 16), ((130, 31, 67), 17), ((128, 513, 70), 18), ((90, 65, 191), 49),
                                     ((2, 100, 16001), 64), ((1, 130, 16387), 33), ((64, 96, 194), 50)])
@pytest.mark.parametrize("skew", [0, 1, 3])
@pytest.mark.parametrize("bad", [False, True])
def test_ragged_rows(shape, m, skew, bad):
    assert _units(shape) >= 256 and shape[2] % 4 != 0  # the rule that takes these sizes to the kernel
    rng = np.random.default_rng(sum(shape) + m)
    X, U = _float32(rng, *shape), _float32(rng, shape[1], m)
    fin = np.ones((shape[0], shape[2]), dtype=bool)
    if bad:
        for a, b, v in ((0, 0, np.inf), (-1, shape[2] - 1, -np.inf), (shape[0] // 2, shape[2] - 3, np.nan)):
            X[a, shape[1] // 2, b] = v
            fin[a, b] = False
    got = _contract(X, U, skew)
    ref, mag = _reference(np.where(np.isfinite(X), X, 0.0), U)
    err = np.abs(np.moveaxis(got - ref, 1, 2))[fin]
    assert np.all(err <= 2 * (shape[1] + 8) * 2.0 ** -24 * np.moveaxis(mag, 1, 2)[fin])
    if bad:
        assert not np.isfinite(np.moveaxis(got, 1, 2)[~fin]).any()


# eight waves a workgroup: an unsplit k range past 768 (2049 units of 64 columns), every entry checked
def test_eight_waves_a_workgroup():
    K, B, m = 800, 131072 + 64, 49
    print("core", K, B, m, flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(1, K, B, generator=g, device="cuda")
    U = torch.randn(K, m, generator=g, device="cuda").double()
    got = rt.rtucker_core(X, [None, U, None], modes=[1])[0].double()
    Ut, Xd = U.t().contiguous(), X[0].double()
    bound = 2 * (K + 8) * 2.0 ** -24 * (Ut.abs() @ Xd.abs())
    assert bool(((got - Ut @ Xd).abs() <= bound).all())


# ------------------------------------------------------------------ bfloat16, M read from the caches
# rows on the 16-byte grid and fewer than 2048 units of 128 columns (or 8192 with at most 256 k): 32-k blocks
# cut at multiples of eight, every count of row tiles, splits of k; one element off the grid the same
# contraction runs with M in LDS.  Products are exact; binary32 sums as above.
@pytest.mark.parametrize("shape,m", [((1, 8, 64), 1), ((3, 16, 72), 17), ((2, 40, 136), 33), ((5, 72, 640), 64),
                                     ((1, 1000, 128), 50), ((2, 2048, 64), 30), ((2100, 8, 64), 16), ((700, 264, 384), 7)])
@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("bad", [False, True])
def test_bfloat16_small(shape, m, skew, bad):
    rng = np.random.default_rng(sum(shape) + m)
    X = torch.from_numpy(rng.standard_normal(shape)).to(torch.bfloat16).double().numpy()
    U = torch.from_numpy(rng.standard_normal((shape[1], m))).to(torch.bfloat16).double().numpy()
    fin = np.ones((shape[0], shape[2]), dtype=bool)
    if bad:
        X[-1, shape[1] - 1, shape[2] - 1] = np.inf
        fin[-1, shape[2] - 1] = False
    print("core bf16", shape, m, skew, flush=True)
    got = rt.rtucker_core(_dev(X, torch.bfloat16, skew), [None, _dev(U), None], modes=[1]).double().cpu().numpy()
    ref, mag = _reference(np.where(np.isfinite(X), X, 0.0), U)
    err = np.abs(np.moveaxis(got - ref, 1, 2))[fin]
    assert np.all(err <= 2 * (shape[1] + 8) * 2.0 ** -24 * np.moveaxis(mag, 1, 2)[fin])
    if bad:
        assert np.array_equal(got[-1, :, -1][U[-1] != 0], (np.sign(U[-1]) * np.inf)[U[-1] != 0])


# The two rules that give eight waves to a workgroup: rows of 131072 columns from 256 k on (every count of row
# tiles, a remainder of the 32-k block, rows off the 16-byte grid), and four row tiles with more than 768 k.
@pytest.mark.parametrize("shape,m", [((1, 256, 131072), 16), ((1, 263, 131072), 32), ((1, 270, 131077), 36), ((1, 289, 131072), 64),
                                     ((33, 777, 4100), 50), ((1, 255, 131072), 36)])
def test_eight_waves_by_row_length(shape, m):
    A, K, B = shape
    print("core", shape, m, flush=True)
    g = torch.Generator(device="cuda").manual_seed(K)
    X = torch.randn(shape, generator=g, device="cuda")
    U = torch.randn(K, m, generator=g, device="cuda").double()
    got = rt.rtucker_core(X, [None, U, None], modes=[1])
    Ut = U.t().contiguous()
    for a in range(A):
        Xd = X[a].double()
        assert bool(((got[a].double() - Ut @ Xd).abs() <= 2 * (K + 8) * 2.0 ** -24 * (Ut.abs() @ Xd.abs())).all())


# ------------------------------------------------------------------ last mode and vector ALU
# Three and four row tiles on the 16-byte grid, in parts of 64 k: with loads that carry no conditions up to
# 2^22 entries, with conditions past them; k ranges cut anywhere, splits of k.
@pytest.mark.parametrize("shape,m", [((1, 1, 4), 33), ((9, 7, 20), 48), ((65, 1, 64), 64), ((7, 1, 132), 49), ((200, 1, 520), 50),
                                     ((3, 50, 1000), 40), ((4, 1100, 960), 35)])
@pytest.mark.parametrize("bad", [False, True])
def test_last_mode_three_and_four_tiles(shape, m, bad):
    rng = np.random.default_rng(sum(shape) + m)
    K = shape[2]
    X, U = _float32(rng, *shape), _float32(rng, K, m)
    fin = np.ones(shape[:2], dtype=bool)
    if bad:
        X[-1, -1, K - 1] = np.inf
        fin[-1, -1] = False
    print("core last", shape, m, flush=True)
    got = rt.rtucker_core(_dev(X, torch.float32), [None, None, _dev(U)], modes=[2]).double().cpu().numpy()
    Xf = np.where(np.isfinite(X), X, 0.0)
    assert np.all(np.abs(got - Xf @ U)[fin] <= (2 * (K + 8) * 2.0 ** -24 * (np.abs(Xf) @ np.abs(U)))[fin])
    if bad:
        assert np.array_equal(got[-1, -1], np.sign(U[-1]) * np.inf)


# Small contractions on the vector ALU (rows shorter than 64, last modes off the 16-byte grid): sums of 64 k,
# remainders, splits of k.
@pytest.mark.parametrize("dims,mode,m", [((5, 1, 3), 1, 4), ((5, 63, 3), 1, 5), ((2, 64, 33), 1, 20), ((7, 65, 5), 1, 64),
                                         ((1, 130, 63), 1, 17), ((2, 1001, 3), 1, 9), ((9, 7, 53), 2, 40), ((3, 4, 129), 2, 20)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_vector_alu_sums(dims, mode, m, dtype):
    rng = np.random.default_rng(sum(dims) + m)
    X = torch.from_numpy(rng.standard_normal(dims)).to(dtype).double().numpy()
    U = torch.from_numpy(rng.standard_normal((dims[mode], m))).to(dtype).double().numpy()
    Us = [None] * 3
    Us[mode] = _dev(U)
    print("core", dims, mode, m, dtype, flush=True)
    got = rt.rtucker_core(_dev(X, dtype), Us, modes=[mode]).double().cpu().numpy()
    f = lambda x, u: np.moveaxis(np.tensordot(x, u, axes=([mode], [0])), -1, mode)  # noqa: E731
    assert np.all(np.abs(got - f(X, U)) <= 2 * (dims[mode] + 8) * 2.0 ** -24 * f(np.abs(X), np.abs(U)))
