"""The nu-sorted layout where its kernel changes shape: force points around the 16
of a workgroup, quadrature points around a wave's share, segments longer than a
wave's list, quadrature points without a force point, and sizes past the
one-launch form.  Checked through the FP64 matrix, entry by entry against the
oracle's on the valid points; the error bound of a sum of L terms is L 2^-53
times the sum of their magnitudes, here at most the largest column's length."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2001_06468_amd as nrs
    from gpu_util import T, DEV, workspace


def _check(N, Q, nu, seed=0, tol_len=None):
    rng = np.random.default_rng(seed)
    x, X = rng.normal(size=(3, N)), rng.normal(size=(3, Q))
    w = 0.5 + rng.random(Q)
    body = np.full(N, -1, np.int32)
    pb = nrs.Problem(T(x), T(X), T(w), T(nu, torch.int32), T(body, torch.int32), None, 0.1, 1.0)
    ctx = nrs.Context(0)
    lda = nrs.lda_for(3 * N)
    A = torch.zeros((3 * N, lda), dtype=torch.float64, device=DEV)
    nrs.nrs_assemble(ctx, pb, 64, A, lda, workspace(ctx, pb, nrs.NRS_FP64_LU))
    B = torch.zeros_like(A)
    nrs.nrs_assemble(ctx, pb, 64, B, lda, workspace(ctx, pb, nrs.NRS_FP64_LU))
    assert torch.equal(A, B)   # the layout does not depend on the order of arrival
    ok = (nu >= 0) & (nu < N)
    ref = oracle.assemble_As(x, X[:, ok], w[ok], nu[ok].astype(np.int64), 0.1, 1.0)
    got = A.cpu().numpy()[:, :3 * N].T
    longest = np.bincount(nu[ok], minlength=1).max() if ok.any() else 1
    tol = (1e-13 + 4 * longest * 2.0 ** -53) * max(np.abs(ref).max(), 1e-300)
    np.testing.assert_allclose(got, ref, atol=tol, rtol=0)


@pytest.mark.parametrize("N,Q", [(1, 1), (1, 600), (15, 511), (16, 512), (17, 513), (33, 4100),
                                 (40, 400), (100, 5000)])
def test_layout_shapes(N, Q):
    rng = np.random.default_rng(N * 7 + Q)
    nu = rng.integers(-1, N + 1, size=Q).astype(np.int32)   # some without a force point
    _check(N, Q, nu)
    _check(N, Q, np.sort(np.clip(nu, 0, N - 1)).astype(np.int32))


def test_layout_one_segment_holds_almost_everything():
    nu = np.full(9000, 18, np.int32)
    nu[::1000] = 3
    nu[5] = 77
    _check(20, 9000, nu)


def test_layout_past_the_one_launch_form():
    rng = np.random.default_rng(3)
    Q = (1 << 17) + 5
    _check(12, Q, rng.integers(0, 12, size=Q).astype(np.int32))


# force points on both sides of the lines between the untuned assembly shapes
@pytest.mark.parametrize("N", [1536, 1537, 3073])
def test_assembly_shapes(N):
    rng = np.random.default_rng(N)
    _check(N, 2 * N, rng.integers(0, N, size=2 * N).astype(np.int32))
