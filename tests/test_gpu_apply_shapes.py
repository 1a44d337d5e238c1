"""Matrix-free product over segments of every length: force points without quadrature
points, with one, with more than a wave's share, chunks and waves that start inside a
segment, and both sides of four quadrature points per force point, where the sum changes
form.  Against the sum over all pairs in NumPy; each side adds Q terms, of a few roundings
each, so they differ by at most 2 (Q + 32) 2^-53 times the sum of the terms' magnitudes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2001_06468_amd as nrs
    from gpu_util import T, DEV, workspace


@pytest.mark.parametrize("N,Q,kind", [(1, 1, "all"), (3, 2, "all"), (70, 70, "all"),
                                      (65, 130, "sparse"), (40, 1537, "sparse"), (130, 900, "one"),
                                      (200, 5000, "all"), (50, 199, "all"), (50, 200, "all")])
def test_apply_segments(N, Q, kind):
    rng = np.random.default_rng(N + Q)
    nu = {"all": np.arange(Q) % N,
          "sparse": 5 * rng.integers(0, max(1, N // 5), size=Q),   # four of five segments empty
          "one": np.where(rng.random(Q) < 0.9, 7, rng.integers(0, N, size=Q))}[kind].astype(np.int32)
    eps, mu = 0.1, 1.5
    x, X, w = rng.normal(size=(3, N)), rng.normal(size=(3, Q)), 0.5 + rng.random(Q)
    v = rng.normal(size=(3, N))
    pb = nrs.Problem(T(x), T(X), T(w), T(nu, torch.int32), T(np.full(N, -1), torch.int32), None,
                     eps, mu)
    y = torch.empty(3 * N, dtype=torch.float64, device=DEV)
    nrs.nrs_apply(nrs.Context(0), pb, T(v.ravel()), y, workspace(nrs.Context(0), pb, nrs.NRS_FP64_LU))
    r = x[:, :, None] - X[:, None, :]
    d = (r * r).sum(0) + eps * eps
    g = w * v[:, nu]
    along = (r * g[:, None, :]).sum(0)
    a, b = (d + eps * eps) * d ** -1.5, d ** -1.5
    ref = (a * g[:, None, :] + b * along * r).sum(2)
    size = (a * np.abs(g)[:, None, :] + b * (np.abs(r) * np.abs(g)[:, None, :]).sum(0) * np.abs(r)).sum(2)
    scale = 1.0 / (8 * np.pi * mu)
    tol = 2 * (Q + 32) * 2.0 ** -53 * scale * size
    assert (np.abs(y.cpu().numpy().reshape(3, N) - scale * ref) <= tol).all()
