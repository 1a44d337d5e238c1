"""Nearest map at the sizes where its kernel changes shape (several quadrature
points per lane group from 32768 on), with groups that change inside a lane
group, points without a group, exact ties and distances that are not numbers:
equal to the plain definition, index by index."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2001_06468_amd as nrs
    from gpu_util import T, DEV


def _reference(x, X, off, g):
    """First force point of the group until one is strictly nearer."""
    nu = np.full(X.shape[1], -1, np.int32)
    for k in range(len(off) - 1):
        lo, hi = off[k], off[k + 1]
        at = np.nonzero(g == k)[0]
        if hi == lo or not len(at):
            continue
        d = x[:, lo:hi, None] - X[:, None, at]
        with np.errstate(invalid="ignore"):
            d2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
        best = np.argmin(np.where(np.isnan(d2), np.inf, d2), axis=0)
        nu[at] = lo + np.where(np.isnan(d2[0]), 0, best)
    return nu


@pytest.mark.parametrize("Q", [1, 7, 31, 33, 257, 32767, 32768, 32771, 33001])
@pytest.mark.parametrize("kind", ["runs", "shuffled", "ties"])
def test_nearest_shapes(Q, kind):
    rng = np.random.default_rng(Q)
    sizes = [5, 40, 1, 8, 300, 17] if kind != "ties" else [64]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    N = int(off[-1])
    x = rng.normal(size=(3, N))
    X = rng.normal(size=(3, Q))
    g = rng.integers(0, len(sizes), size=Q).astype(np.int32)
    if kind == "runs":
        g.sort()
    elif kind == "shuffled":
        # an index outside the groups leaves the point without one
        g[rng.random(Q) < 0.05] = len(sizes) + 3
        x[:, 2] = np.nan
        X[:, rng.random(Q) < 0.01] = np.nan
    else:
        x = rng.integers(0, 3, size=(3, N)).astype(float)
        X = rng.integers(0, 3, size=(3, Q)).astype(float)
    ctx = nrs.Context(0)
    nu = torch.empty(Q, dtype=torch.int32, device=DEV)
    nrs.nrs_nearest(ctx, T(x), off, T(X), T(g, torch.int32), nu)
    np.testing.assert_array_equal(nu.cpu().numpy(), _reference(x, X, off, g))


def test_nearest_cost_does_not_depend_on_the_order_of_groups():
    """Neighbouring points of distant groups take no more distances than sorted ones (400
    groups of 40: 40 a point; all that lie between the groups of four points are 150
    times as many).  The bound of 6 leaves room for launches and scattered loads."""
    rng = np.random.default_rng(0)
    G, k, Q = 400, 40, 40000
    x, X = T(rng.normal(size=(3, G * k))), T(rng.normal(size=(3, Q)))
    off = (np.arange(G + 1) * k).astype(np.int32)
    ctx = nrs.Context(0)
    nu = torch.empty(Q, dtype=torch.int32, device=DEV)
    ms = []
    for g in (np.sort(np.arange(Q) % G), rng.integers(0, G, size=Q)):
        gx = T(g, torch.int32)
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(4):   # the first as a warm-up
            e0.record()
            for _ in range(20):
                nrs.nrs_nearest(ctx, x, off, X, gx, nu)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        ms.append(min(times[1:]))
    assert ms[1] <= 6 * ms[0], ms
