"""One-workgroup flexible GMRES (orders up to 8192) without a preconditioner, so that a cycle
runs many Arnoldi steps: past the basis columns held in registers (8 with four rows
per thread, 4 with eight), past a second group of eight, and through restarts; orders
around 1024 rows (one row per thread), 4096 (four) and 8192 (eight).
Reference: the partial-pivoting FP64 solve of the same problem.  Tolerance: the relative
residual of 1e-12 times the condition number of these matrices, below 1e3 for the
force points' spacing and eps chosen."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2001_06468_amd as nrs
    from gpu_util import T, workspace, DEV


@pytest.fixture(scope="module")
def ctx():
    c = nrs.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _spread(N):
    """N evenly spread points on the unit sphere (golden-angle spiral): on random points,
    some of them close pairs, short restarts stagnate in any arithmetic."""
    i = np.arange(N) + 0.5
    z, phi = 1 - 2 * i / N, np.pi * (1 + 5 ** 0.5) * i
    r = np.sqrt(1 - z * z)
    return np.stack([r * np.cos(phi), r * np.sin(phi), z])


@pytest.mark.parametrize("N,restart", [(20, 8), (341, 9), (342, 60), (1365, 63), (1366, 12),
                                       (1366, 60), (2730, 17)])
def test_cycles_longer_than_the_register_columns(ctx, N, restart):
    rng = np.random.default_rng(N + restart)
    x = _spread(N)
    nu = np.repeat(np.arange(N), 4).astype(np.int32)
    X = x[:, nu] + 0.01 * rng.normal(size=(3, 4 * N))
    eps = 0.3 / N ** 0.5
    pb = nrs.Problem(T(x), T(X), T(np.full(4 * N, np.pi / N)), T(nu, torch.int32),
                     T(-np.ones(N, dtype=np.int32), torch.int32), None, eps, 1.0)
    u = T(rng.normal(size=3 * N))
    ref = torch.empty(pb.n, dtype=torch.float64, device=DEV)
    nrs.nrs_solve(ctx, pb, u, None, ref, workspace(ctx, pb, nrs.NRS_FP64_LU),
                  method=nrs.NRS_FP64_LU)
    sol = torch.empty_like(ref)
    info = nrs.nrs_solve(ctx, pb, u, None, sol, workspace(ctx, pb, nrs.NRS_GMRES_BLOCK),
                         method=nrs.NRS_GMRES_BLOCK, precond=nrs.NRS_PRECOND_EXACT,
                         gmres_restart=restart, gmres_max_iter=4000)
    print(f"n = {pb.n}, restart {restart}: {info['iterations']} iterations", flush=True)
    assert info["fell_back"] == 0 and info["method_used"] == nrs.NRS_GMRES_BLOCK, info
    assert info["iterations"] > 8
    err = (sol - ref).norm() / ref.norm()
    assert err <= 1e-8, err
