"""Network gradient at the sizes where its kernels change shape: rows of the
reduction around 16 and 64 (waves, loads in flight), points per body around the
tile edge 16 and the limit 256.  Tolerances as in test_gpu_learned.py: gradient
1e-4 of its largest entry, loss 1e-5, outputs 2e-5."""
import numpy as np
import pytest
import torch

from oracle import mlp

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2001_06468_amd as nrs
    from gpu_util import T, DEV
    from test_gpu_learned import H, _f32, _net_data


@pytest.fixture(scope="module")
def ctx():
    return nrs.Context(0)


@pytest.mark.parametrize("nsel,points", [(1, 3), (15, 2), (16, 4), (17, 5), (63, 3), (64, 1),
                                         (65, 2), (129, 4), (3, 15), (3, 16), (2, 17), (2, 31),
                                         (2, 64), (2, 65), (1, 255), (1, 256)])
def test_gradient_shapes(ctx, nsel, points):
    sizes = [points + (i % 2 if points < 255 else 0) for i in range(nsel)]
    theta, phi, off, t_pt, t_b = _net_data(100 + nsel, sizes)
    L_ref, g_ref = mlp.gradient(theta, H, phi, off, t_pt, t_b)
    y_ref, z_ref = mlp.forward(theta, H, phi, off)
    P = mlp.param_count(H)
    ws = torch.empty(nrs.nrs_mlp_grad_workspace_size(nsel), dtype=torch.uint8, device=DEV)
    grad = torch.empty(P + 1, dtype=torch.float32, device=DEV)
    bo = T(off, torch.int32)
    nrs.nrs_mlp_grad(ctx, _f32(theta), nsel, bo, _f32(phi), _f32(t_pt), _f32(t_b), grad, ws)
    g = grad.cpu().numpy()
    assert g[P] == pytest.approx(L_ref, rel=1e-5)
    np.testing.assert_allclose(g[:P], g_ref, atol=1e-4 * np.abs(g_ref).max())
    y = torch.empty((phi.shape[0], 3), dtype=torch.float32, device=DEV)
    z = torch.empty((nsel, 6), dtype=torch.float32, device=DEV)
    nrs.nrs_mlp_forward(ctx, _f32(theta), nsel, bo, _f32(phi), y, z)
    np.testing.assert_allclose(y.cpu().numpy(), y_ref, atol=2e-5 * np.abs(y_ref).max())
    np.testing.assert_allclose(z.cpu().numpy(), z_ref, atol=2e-5 * np.abs(z_ref).max())
