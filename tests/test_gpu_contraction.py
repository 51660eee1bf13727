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
