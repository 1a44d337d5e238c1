"""Launches over all systems of a batch: a system must get what its own launches give it.
Batches of 1 and of 70 systems (more than a wave of status records), sizes around the
workgroups' shares (one force point, 16 / 17, 64 / 65, 85 / 86 = 64 and 65 row groups) and a
system past the sizes of the one-launch layout (Q = 2^17 + 8) between small ones.
Bit-identical to the single solve of the same method: every workgroup runs the same
code on the same operands in the same order."""
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


def _problem(N, Q, seed):
    rng = np.random.default_rng(seed)
    x = rng.normal(size=(3, N))
    x *= max(1.0, N ** 0.5 / 4) / np.linalg.norm(x, axis=0)
    nu = rng.permutation(np.arange(Q) % N).astype(np.int32)   # every force point has points
    X = x[:, nu] + 0.02 * rng.normal(size=(3, Q))
    w = np.full(Q, 1.0 / Q)
    body = -np.ones(N, dtype=np.int32)
    pb = nrs.Problem(T(x), T(X), T(w), T(nu, torch.int32), T(body, torch.int32), None, 0.1, 1.5)
    return pb, T(rng.normal(size=3 * N))


SHAPES = {
    "one": [(17, 200)],
    "edges": [(1, 1), (16, 16), (64, 600), (86, 700), (17, 90), (65, 64 * 9), (85, 1024)],
    "large layout": [(21, 170), (40, (1 << 17) + 8), (22, 333)],
    "many": [(2 + k % 31, 40 + 7 * k) for k in range(70)],
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_batch_launches_match_single(ctx, name):
    probs = [_problem(N, Q, 100 + k) for k, (N, Q) in enumerate(SHAPES[name])]
    pbs, us = [p for p, _ in probs], [u for _, u in probs]
    sols = [torch.empty(p.n, dtype=torch.float64, device=DEV) for p in pbs]
    ws = torch.empty(nrs.nrs_solve_batched_workspace_size(ctx, pbs), dtype=torch.uint8, device=DEV)
    infos = nrs.nrs_solve_batched(ctx, pbs, us, sols, ws)
    for k, (pb, u) in enumerate(probs):
        one = torch.empty_like(sols[k])
        info = nrs.nrs_solve(ctx, pb, u, None, one, workspace(ctx, pb, nrs.NRS_FP32_IR),
                             method=nrs.NRS_FP32_IR)
        assert infos[k]["fell_back"] == 0 and info["fell_back"] == 0, (k, infos[k], info)
        np.testing.assert_array_equal(sols[k].cpu().numpy(), one.cpu().numpy(), err_msg=str(k))
        assert infos[k]["iterations"] == info["iterations"]
        assert infos[k]["backward_error"] == info["backward_error"]
