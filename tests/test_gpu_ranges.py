"""Nearest-element searches at the ends of their range of units, shapes and distances, on the GPU."""
import numpy as np
import pytest

from paper_2606_05581_amd import workloads as W
from test_gpu_search import _log, _mesh, _points, _slivers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    from paper_2606_05581_amd import msk

    assert torch.cuda.is_available(), "GPU test needs a visible MI355X"
    c = msk.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("leaf", [1, 4, 8])
@pytest.mark.parametrize("unit", [3e4, 1e5, 1e7, 1e9])
def test_slivers_in_large_units(ctx, oracle_mod, unit, leaf):
    """Triangles without a prefilter value, tens of thousands of units from the points that ask for them: none may
    drop out before its exact test, whatever its place in its leaf. Bit for bit the brute force's answers."""
    import torch

    V, F = _slivers(3000, 3)
    V32 = (V * unit).astype(np.float32)
    mesh = ctx.build_bvh(V32, F.astype(np.int32), leaf_size=leaf)
    Q = (_points(V, 4001, 5).astype(np.float64) * unit).astype(np.float32)
    t_o, d_o, b_o = oracle_mod.Scene(V32, F, bvh=False).nearest_f32(Q.astype(np.float64))
    t, d, b = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q, device="cuda")))
    some = np.isfinite(d_o)
    print(f"[slivers] unit {unit:g}, leaf {leaf}: {int((t != t_o)[some].sum())} of {int(some.sum())} differ", flush=True)
    assert np.array_equal(d, d_o)
    assert np.array_equal(t[some], t_o[some]) and np.array_equal(b[some], b_o[some])


@pytest.mark.parametrize("leaf", [1, 4, 8])
def test_slivers_in_large_units_walk_the_same_paths(ctx, leaf):
    """Walks of the persistent and the plain form among slivers 1e5 units wide."""
    V, F = _mesh("sphere1280")
    S, G = _slivers(200, 9)
    V, F = 1e5 * np.concatenate([V, 0.4 * S]), np.concatenate([F, G + len(V)])
    case = W._point_case(V, F, 100, np.random.default_rng(2))
    case.eps = case.h / 10.0
    for exterior in (False, True):
        a, b = (_log(ctx, case, 32, exterior, leaf, form=f) for f in (0, 1))
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
