"""Every launch shape of the assembly gives the same matrix bit for bit, and the tuner
reports the shape that later assemblies get."""
import ctypes

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

SHAPES = [(b, t) for b in (64, 128, 256) for t in (4, 8, 16)]   # rows, force points

if torch.cuda.is_available():
    import paper_2001_06468_amd as nrs
    from paper_2001_06468_amd import _lib
    from gpu_util import T, DEV, prepare, workspace


def _shape(ctx, pb, index=None):
    """(rows, points) of FP32 and FP64 assemblies of problems like pb, after setting both to
    shape `index` if given."""
    fn = _lib.load().nrs_internal_assembly_shape
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    dims = (ctypes.c_int32 * 4)()
    sel = None if index is None else (ctypes.c_int32 * 2)(index, index)
    assert fn(ctx.handle, pb.N, pb.Q, sel, dims) == 0
    return (dims[0], dims[1]), (dims[2], dims[3])


def _free_points(N, Q):
    rng = np.random.default_rng(N)
    nu = rng.integers(0, N, size=Q).astype(np.int32)
    return nrs.Problem(T(rng.normal(size=(3, N))), T(rng.normal(size=(3, Q))),
                       T(0.5 + rng.random(Q)), T(nu, torch.int32),
                       T(np.full(N, -1), torch.int32), None, 0.1, 1.0)


def _problem(name):
    if name == "bodies":
        return prepare(synth.filament_scene(3, seed=1, Nf=37, Qf=150), 0.2)[0]
    return {"one": lambda: _free_points(1, 3), "edges": lambda: _free_points(65, 200),
            "rows": lambda: _free_points(257, 700)}[name]()


@pytest.mark.parametrize("name", ["one", "edges", "rows", "bodies"])
def test_shapes_agree(name):
    ctx, pb = nrs.Context(0), _problem(name)
    lda = nrs.lda_for(pb.n)
    ws = workspace(ctx, pb, nrs.NRS_FP32_IR)

    def matrices():
        out = []
        for bits, dt in ((32, torch.float32), (64, torch.float64)):
            A = torch.full((pb.n, lda), float("nan"), dtype=dt, device=DEV)
            nrs.nrs_assemble(ctx, pb, bits, A, lda, ws)
            A = A[:, :pb.n]
            assert bool(torch.isfinite(A).all())
            out.append(A)
        return out

    ref = matrices()   # the untuned shape
    for k, want in enumerate(SHAPES):
        assert _shape(ctx, pb, k) == (want, want)
        for A, B in zip(ref, matrices()):
            assert torch.equal(A, B), want


@pytest.mark.parametrize("name", ["edges", "bodies"])
def test_tuner_reports_the_shape_in_use(name):
    ctx, pb = nrs.Context(0), _problem(name)
    untuned = _shape(ctx, pb)
    assert set(untuned) <= set(SHAPES)
    r = nrs.nrs_autotune(ctx, pb, workspace(ctx, pb, nrs.NRS_FP32_IR))
    assert _shape(ctx, pb) == ((r["block32"], r["strip32"]), (r["block64"], r["strip64"]))
    for bits, got in zip((32, 64), _shape(ctx, pb)):
        assert r[f"ms{bits}"] <= r[f"default_ms{bits}"]
        if got == untuned[bits // 32 - 1]:   # the untuned shape is among those timed
            assert r[f"ms{bits}"] == r[f"default_ms{bits}"]
    nrs.nrs_autotune_clear(ctx)
    assert _shape(ctx, pb) == untuned


def test_untuned_shapes_by_size():
    """Both sides of the lines between the untuned shapes (no launch)."""
    ctx = nrs.Context(0)

    class Size:
        def __init__(self, N):
            self.N, self.Q = N, 10 * N

    for N, want in [(1, ((64, 4), (64, 4))), (1536, ((64, 4), (64, 4))),
                    (1537, ((128, 4), (128, 4))), (3072, ((128, 4), (128, 4))),
                    (3073, ((256, 4), (256, 4))), (5000, ((256, 4), (256, 4))),
                    (5001, ((256, 4), (128, 4))), (80000, ((256, 4), (128, 4)))]:
        assert _shape(ctx, Size(N)) == want, N
