"""Batched in-place factorisation and solve at the edges of their tiles (GPU)."""
import numpy as np
import pytest

from tests.gpu_util import device, t

pytestmark = pytest.mark.gpu


# orders one short of, at and past the 16-wide tiles and the 64-wide block
# columns, and the widest; a batch of small ones larger than what is resident
@pytest.mark.parametrize("n,batch", [(15, 2500), (16, 3), (17, 3), (63, 3), (64, 3), (65, 5), (129, 3), (257, 3),
                                     (449, 3), (511, 3), (512, 2)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_lu"])
def test_lu_in_place_at_tile_edges(n, batch, prec):
    # every second matrix keeps its rows in place, the others exchange
    # them.  Bounds: a factor entry sums at most n products of |L| <= 4 with |U|
    # (30 n u max |A|, as for the other orders), a solution two such triangular
    # solves.
    import paper_2511_10558_amd as ab
    dev = device()
    rng = np.random.default_rng(n)
    A = rng.normal(size=(batch, n, n))
    A[::2] = np.eye(n) + 0.3 / np.sqrt(n) * A[::2]
    b = rng.normal(size=(batch, n))
    LU, perm, info = ab.lu_factor(t(A, dev), precision=prec)
    assert not info.any()
    u = np.finfo(np.float64 if prec == "fp64" else np.float32).eps / 2
    z = ab.lu_solve(LU, perm, t(b, dev)).cpu().numpy()
    LU, perm = LU.cpu().numpy(), perm.cpu().numpy()
    for i in range(min(batch, 3)) if batch < 100 else (0, 1, 1023, batch - 2, batch - 1):
        L, U = np.tril(LU[i], -1) + np.eye(n), np.triu(LU[i])
        assert sorted(perm[i]) == list(range(n)) and np.abs(L).max() <= 4.0 * (1 + 1e-6)
        assert np.abs(A[i][perm[i]] - L @ U).max() <= 30 * n * u * np.abs(A[i]).max()
        res = np.abs(A[i] @ z[i] - b[i]).max() / (np.abs(A[i]).max() * np.abs(z[i]).max())
        assert res <= 60 * n * u


@pytest.mark.parametrize("n", [1, 16, 63, 64, 65, 200])
def test_lu_solve_divides(n):
    # factors of a diagonal matrix: each unknown is one quotient, rounded once
    import paper_2511_10558_amd as ab
    dev = device()
    rng = np.random.default_rng(n)
    d, b = rng.normal(size=(40, n)), rng.normal(size=(40, n))
    LU = np.zeros((40, n, n))
    LU[:, np.arange(n), np.arange(n)] = d
    import torch
    perm = torch.arange(n, dtype=torch.int32, device=dev).repeat(40, 1)
    z = ab.lu_solve(t(LU, dev), perm, t(b, dev)).cpu().numpy()
    assert np.array_equal(z, b / d)


def test_lu_solve_divides_at_the_range_ends():
    # what a quotient by way of the reciprocal loses: subnormal, huge, zero and
    # infinite pivots, quotients past the range.  One rounding each; where the
    # remainder or the quotient is subnormal a second one of a unit in the last place
    import torch
    import paper_2511_10558_amd as ab
    dev = device()
    ends = np.array([5e-324, 3e-320, 1e-309, 2.3e-308, 1e-200, 0.7, 1e200, 4e307, 1.7e308, 0.0, np.inf, np.nan])
    d, b = (v.ravel() for v in np.meshgrid(np.concatenate([ends, -ends]), ends))
    perm = torch.zeros((len(d), 1), dtype=torch.int32, device=dev)
    z = ab.lu_solve(t(d.reshape(-1, 1, 1), dev), perm, t(b.reshape(-1, 1), dev)).cpu().numpy().ravel()
    with np.errstate(all="ignore"):
        ref = b / d
    assert np.array_equal(np.isnan(z), np.isnan(ref)) and np.array_equal(np.isinf(z), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.array_equal(z[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.all(np.abs(z[fin] - ref[fin]) <= np.spacing(np.abs(ref[fin])))


# Where every row left is NaN, a row that pads the matrix to a multiple of 16 is the
# pivot (perm past n - 1).  Such a row is zero in the matrix's columns, and remains
# zero or NaN; what stands in the factors there is that row, not one of the matrix.
@pytest.mark.parametrize("n", [15, 17, 50, 65, 100, 200])
@pytest.mark.parametrize("prec", ["fp64", "fp32_lu"])
def test_lu_factor_of_nan_beside_padding(n, prec):
    import paper_2511_10558_amd as ab
    dev = device()
    rng = np.random.default_rng(n)
    A = rng.normal(size=(3, n, n)) + 3 * n * np.eye(n)
    A[0, -1, -1] = np.nan             # the last pivot
    A[1, :, 0] = np.nan               # a whole column
    A[2, n // 2] = np.nan             # a whole row
    LU, perm, _ = (v.cpu().numpy() for v in ab.lu_factor(t(A, dev), precision=prec))
    for i in range(3):
        pad = LU[i][perm[i] >= n]
        assert len(pad) > 0 and np.all(np.isnan(pad) | (pad == 0.0))
