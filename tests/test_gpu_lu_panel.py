"""Partial-pivoting LU whose panel rows are held in registers: every rows-per-
thread / width shape at both ends of its range, against LAPACK's pivots and the
backward error bound of Gaussian elimination."""
import numpy as np
import pytest
import scipy.linalg
import torch

import paper_2001_06468_amd as nrs
from gpu_util import DEV, lu_ws

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return nrs.Context(0)


def _factor(ctx, A0, dtype, pad=0):
    n = A0.shape[0]
    lda = n + pad
    A = torch.zeros((n, lda), dtype=dtype, device=DEV)
    A[:, :n] = torch.from_numpy(np.ascontiguousarray(A0.T)).to(DEV, dtype)
    ipiv = torch.empty(n, dtype=torch.int32, device=DEV)
    perm = torch.empty(n, dtype=torch.int32, device=DEV)
    sing = torch.zeros(1, dtype=torch.int32, device=DEV)
    nrs.nrs_lu_factor(ctx, A, lda, ipiv, perm, sing, lu_ws(ctx, n, A))
    return A[:, :n].T, ipiv.cpu().numpy(), perm.long(), int(sing.item())


def _backward_ok(A0, LU, perm, unit):
    """|P A - L U| <= gamma_n |L| |U| entry by entry (Higham, Theorem 9.3), the
    check's own product in FP64 adding at most as much again."""
    n = A0.shape[0]
    LU = LU.double()
    L = torch.tril(LU, -1) + torch.eye(n, dtype=torch.float64, device=DEV)
    U = torch.triu(LU)
    A = torch.from_numpy(A0).to(DEV).double()[perm]
    gamma = n * unit / (1 - n * unit)
    bound = 2 * gamma * (L.abs() @ U.abs().contiguous())
    return bool(((A - L @ U).abs() <= bound).all())


# rows a panel may have per shape: 512, 1024, 1536, 2048, 3072, 4096, 8192
@pytest.mark.parametrize("n", [2, 16, 17, 80, 512, 513, 1025, 1537, 2049, 3073, 4097, 8193])
def test_panel_shapes_fp64(ctx, n):
    rng = np.random.default_rng(n)
    A0 = rng.normal(size=(n, n))
    LU, ipiv, perm, sing = _factor(ctx, A0, torch.float64, pad=n % 3)
    assert sing == 0
    np.testing.assert_array_equal(ipiv, scipy.linalg.lu_factor(A0)[1])
    assert _backward_ok(A0, LU, perm, 2.0 ** -53)


@pytest.mark.parametrize("n", [3, 65, 513, 1537, 2049])
def test_panel_shapes_fp32(ctx, n):
    rng = np.random.default_rng(n)
    A0 = rng.normal(size=(n, n)).astype(np.float32)
    LU, _, perm, sing = _factor(ctx, A0, torch.float32, pad=1)
    assert sing == 0
    assert _backward_ok(A0, LU, perm, 2.0 ** -24)


def test_panel_exact_ties_and_swapped_rows(ctx):
    """Entries +-1 and 0 tie all the time (lowest row wins), small integers keep
    every product exact until the first division; a permutation matrix moves
    every row."""
    rng = np.random.default_rng(5)
    n = 600
    T0 = np.eye(n)[rng.permutation(n)]
    LU, ipiv, perm, sing = _factor(ctx, T0, torch.float64)
    assert sing == 0
    np.testing.assert_array_equal(ipiv, scipy.linalg.lu_factor(T0)[1])
    np.testing.assert_array_equal(LU.cpu().numpy(), np.eye(n))
    # first column all +-1: the pivot is row 0, then rows tie again
    S0 = rng.choice([-1.0, 1.0], size=(40, 40)) * 2.0 ** rng.integers(0, 2, size=(40, 40))
    LU, ipiv, perm, sing = _factor(ctx, S0, torch.float64)
    assert ipiv[0] == int(np.argmax(np.abs(S0[:, 0])))
    assert _backward_ok(S0, LU, perm, 2.0 ** -53)


@pytest.mark.parametrize("cols", [[0], [5, 15, 16], [63], [40, 64, 69]])
def test_panel_zero_columns(ctx, cols):
    """A zero column keeps its diagonal row, raises the flag and leaves the rest of
    the elimination as LAPACK does it."""
    n = 70
    A0 = np.random.default_rng(7).normal(size=(n, n))
    A0[:, cols] = 0.0
    LU, ipiv, perm, sing = _factor(ctx, A0, torch.float64)
    assert sing == 1
    import warnings
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        _, ref = scipy.linalg.lu_factor(A0)
    np.testing.assert_array_equal(ipiv, ref)
    assert _backward_ok(A0, LU, perm, 2.0 ** -53)


def test_panel_nan_column_stays_in_range(ctx):
    """Columns without a finite entry: every interchange stays inside the matrix,
    the entries before the first such column are finite."""
    n = 130
    A0 = np.random.default_rng(8).normal(size=(n, n))
    A0[:, 20] = np.nan
    LU, ipiv, perm, _ = _factor(ctx, A0, torch.float64)
    assert ((ipiv >= np.arange(n)) & (ipiv < n)).all()
    np.testing.assert_array_equal(np.sort(perm.cpu().numpy()), np.arange(n))
    assert bool(torch.isfinite(LU[:, :20]).all()) and bool(torch.isnan(LU[20, 20]))


def test_rows_above_an_infinity_stay_finite(ctx):
    """An infinite entry in a U row does not reach the rows above it (0 * inf)."""
    n = 130
    A0 = np.random.default_rng(9).normal(size=(n, n)) + 4 * n * np.eye(n)
    A0[30, 100] = np.inf
    LU, ipiv, _, _ = _factor(ctx, A0, torch.float64)
    np.testing.assert_array_equal(ipiv[:64], np.arange(64))
    assert bool(torch.isfinite(LU[:30, :]).all()) and bool(torch.isinf(LU[30, 100]))


@pytest.mark.parametrize("n,row,col", [(130, 30, 40), (130, 0, 63), (1700, 10, 20), (4200, 5, 9)])
def test_rows_above_an_infinity_stay_finite_inside_a_panel(ctx, n, row, col):
    """The same for a column of the same 64-column panel, in a later sub-panel (16, 8
    and 4 columns wide at these sizes): only the rows at and below it change."""
    A0 = np.random.default_rng(10).normal(size=(n, n)) + 4 * n * np.eye(n)
    A0[row, col] = np.inf
    LU, ipiv, _, _ = _factor(ctx, A0, torch.float64)
    # the column is eliminated as it is until its own pivot, so earlier pivots stay
    np.testing.assert_array_equal(ipiv[:col], np.arange(col))
    assert bool(torch.isfinite(LU[:row, col]).all()) and bool(torch.isinf(LU[row, col]))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("row", [20, 21, 60])
def test_panel_zero_column_with_a_nan_is_singular(ctx, dtype, row):
    """A column of zeros and one NaN has no pivot: the flag is raised wherever the NaN
    lies, the diagonal row included."""
    n = 70
    A0 = np.random.default_rng(11).normal(size=(n, n)) + 4 * n * np.eye(n)
    A0[:, 20] = 0.0
    A0[row, 20] = np.nan
    _, ipiv, _, sing = _factor(ctx, A0, dtype)
    assert sing == 1
    np.testing.assert_array_equal(ipiv[:20], np.arange(20))


# panels lose 64 rows at a time, so a shape's largest height occurs only if the order is that height
@pytest.mark.parametrize("n", [1024, 1536, 2048, 3072, 4096, 8192])
def test_panel_shapes_fp64_at_their_last_row(ctx, n):
    A0 = np.random.default_rng(n).normal(size=(n, n))
    LU, ipiv, perm, sing = _factor(ctx, A0, torch.float64)
    assert sing == 0
    np.testing.assert_array_equal(ipiv, scipy.linalg.lu_factor(A0)[1])
    assert _backward_ok(A0, LU, perm, 2.0 ** -53)


@pytest.mark.parametrize("n", [512, 1024, 3073, 4097])
def test_panel_shapes_fp32_wide(ctx, n):
    """FP32 in every rows-per-thread / width shape.  A pivot is the largest of its column
    as this elimination computed it: no multiplier is larger than one."""
    A0 = np.random.default_rng(n).normal(size=(n, n)).astype(np.float32)
    LU, ipiv, perm, sing = _factor(ctx, A0, torch.float32, pad=1)
    assert sing == 0
    assert ((ipiv >= np.arange(n)) & (ipiv < n)).all()
    assert float(torch.tril(LU, -1).abs().max()) <= 1.0
    assert _backward_ok(A0, LU, perm, 2.0 ** -24)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_panel_pivots_on_exact_arithmetic(ctx, dtype):
    """P A = L U with L of eighths and U of small integers, a power of two on the
    diagonal: every step is exact in either precision, so pivots and factors are those
    that built the matrix."""
    n = 700
    rng = np.random.default_rng(12)
    L = np.tril(rng.integers(-7, 8, size=(n, n)) / 8.0 * (rng.random((n, n)) < 0.02), -1) + np.eye(n)
    U = np.triu(rng.integers(-4, 5, size=(n, n)) * (rng.random((n, n)) < 0.02), 1).astype(float)
    U += np.diag(2.0 ** rng.integers(0, 3, size=n))
    A0 = L @ U
    swap = rng.permutation(n)
    LU, ipiv, perm, sing = _factor(ctx, A0[swap], dtype)
    assert sing == 0
    np.testing.assert_array_equal(swap[perm.cpu().numpy()], np.arange(n))
    np.testing.assert_array_equal(LU.cpu().double().numpy(), np.tril(L, -1) + U)
    # the interchanges lead to the same permutation
    at = np.arange(n)
    for j, p in enumerate(ipiv):
        at[[j, p]] = at[[p, j]]
    np.testing.assert_array_equal(at, perm.cpu().numpy())


@pytest.mark.parametrize("dtype,scales", [(torch.float64, [2.0 ** -960, 1.0, 2.0 ** 960]),
                                          (torch.float32, [2.0 ** -100, 1.0, 2.0 ** 100])])
def test_panel_pivots_outside_the_plain_range(ctx, dtype, scales):
    """Columns scaled so that pivots lie on both sides of the range in which a quotient is
    formed by the reciprocal.  Scaling a column by a power of two scales that column of U
    and changes nothing else, as long as nothing leaves the normal numbers."""
    n = 200
    rng = np.random.default_rng(13)
    A0 = rng.normal(size=(n, n))
    if dtype == torch.float32:
        A0 = A0.astype(np.float32)
    c = rng.choice(scales, size=n)
    ref, ip0, _, _ = _factor(ctx, A0, dtype)
    LU, ipiv, perm, sing = _factor(ctx, A0 * c, dtype)
    assert sing == 0
    np.testing.assert_array_equal(ipiv, ip0)
    got, ref = LU.cpu().double().numpy(), ref.cpu().double().numpy()
    np.testing.assert_array_equal(np.tril(got, -1), np.tril(ref, -1))
    np.testing.assert_array_equal(np.triu(got) / c, np.triu(ref))


def test_nan_column_stays_in_range_past_the_register_panel(ctx):
    """The same for panels of more rows than the registers of a workgroup hold."""
    n = 8260
    A0 = np.random.default_rng(14).normal(size=(n, n))
    A0[:, 20] = np.nan
    LU, ipiv, perm, sing = _factor(ctx, A0, torch.float64)
    assert sing == 1
    assert ((ipiv >= np.arange(n)) & (ipiv < n)).all()
    np.testing.assert_array_equal(np.sort(perm.cpu().numpy()), np.arange(n))
    assert bool(torch.isfinite(LU[:, :20]).all()) and bool(torch.isnan(LU[20, 20]))
