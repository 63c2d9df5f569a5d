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


@pytest.mark.parametrize("n", [1, 65, 3000])
def test_kelvin_points_far_outside_the_domain(ctx, oracle_mod, n):
    """Points up to 10^150 domain sizes away have a nearest element like any other: the oracle's distance (FP64 on
    both sides, a few roundings apart), of an element at that distance by the oracle's measure."""
    import torch

    V, F = W.icosphere_recursive(2)
    c = np.array([0.2, -0.3, 0.1])
    V32 = V.astype(np.float32)
    kv = ctx.kelvin(ctx.build_bvh(V32, F.astype(np.int32)), c)
    R = kv.info()["radius"]
    rng = np.random.default_rng(n)
    Q = rng.normal(size=(n, 3))
    Q *= R * 10.0 ** rng.choice([1, 5.9, 6.1, 12, 18, 19.5, 25, 60, 150], size=(n, 1)) / np.linalg.norm(Q, axis=1, keepdims=True)
    t_o, d_o, q_o, _ = oracle_mod.KelvinScene(V32, F, c).nearest(Q, bvh=False)
    t, d, q, l = (x.cpu().numpy() for x in ctx.kelvin_closest_points(kv, torch.tensor(Q, device="cuda")))
    assert ((t >= 0) & (t < len(F))).all()
    assert np.allclose(d, d_o, rtol=1e-10, atol=0)
    Vc = V32.astype(np.float64) - c
    for i in np.nonzero(t != t_o)[0]:
        assert oracle_mod.kelvin_tri_d2(Q[i], *Vc[F[t[i]]])[0] == pytest.approx(d_o[i], rel=1e-10)
    near = np.linalg.norm(Q, axis=1) < 1e4 * R  # farther out many points of the domain are nearest to rounding
    assert np.allclose(q[near], q_o[near], rtol=0, atol=1e-9 * R)
    assert np.allclose(l.sum(1), 1.0, rtol=0, atol=1e-6)


def test_kelvin_points_that_are_no_numbers(ctx):
    """As for flat triangles: the lowest element at an infinite distance, and the numbers beside it as ever."""
    import torch

    V, F = W.icosphere_recursive(2)
    kv = ctx.kelvin(ctx.build_bvh(V.astype(np.float32), F.astype(np.int32)), np.array([0.2, -0.3, 0.1]))
    Q = np.random.default_rng(4).normal(size=(200, 3))
    a = [x.cpu().numpy() for x in ctx.kelvin_closest_points(kv, torch.tensor(Q, device="cuda"))]
    P = Q.copy()
    P[::3, 1] = np.nan
    P[1::9, 2] = np.inf
    b = [x.cpu().numpy() for x in ctx.kelvin_closest_points(kv, torch.tensor(P, device="cuda"))]
    bad = ~np.isfinite(P).all(1)
    assert (b[0][bad] == 0).all() and np.isinf(b[1][bad]).all()
    for x, y in zip(a, b):
        assert np.array_equal(x[~bad], y[~bad])


@pytest.mark.parametrize("leaf", [0, 1, 2, 3, 4, 8])
def test_kelvin_leaf_width_is_the_one_asked_for(ctx, leaf):
    """The inverted hierarchy has at most `leaf` elements a leaf and says so: narrower leaves need more nodes."""
    V, F = W.icosphere_recursive(3)
    mesh = ctx.build_bvh(V.astype(np.float32), F.astype(np.int32))
    c = np.array([0.2, -0.1, 0.05])
    info = ctx.kelvin(mesh, c, leaf_size=leaf).info()
    assert info["leaf_size"] == (leaf if leaf else 4)
    # a 4-wide node has at most 4 leaves of `leaf` elements below it
    assert info["n_nodes"] >= len(F) / (4.0 * info["leaf_size"] * 4.0 / 3.0)
    if 0 < leaf < 4:
        assert info["n_nodes"] > ctx.kelvin(mesh, c, leaf_size=4).info()["n_nodes"]
