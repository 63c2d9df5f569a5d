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


def _shards(n, seed):
    """Triangles of all shapes and sizes: shortest altitude over longest edge from 1 to 1e-5 (short edges, flat
    angles and others alike), longest edge from 1 to 1e-5 of the scene."""
    rng = np.random.default_rng(seed)
    size, thin = 10.0 ** rng.uniform(-5, -0.3, (n, 1)), 10.0 ** rng.uniform(-5, 0, (n, 1))
    x = rng.normal(size=(n, 3))
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    y = np.cross(x, rng.normal(size=(n, 3)))
    y /= np.linalg.norm(y, axis=1, keepdims=True)
    along = np.where(rng.random((n, 1)) < 0.5, 1.0 + thin * rng.uniform(-1, 1, (n, 1)), rng.uniform(0, 1, (n, 1)))
    a = rng.uniform(-0.5, 0.5, size=(n, 3))
    t = np.stack([a, a + size * x, a + size * (along * x + thin * y)], 1)
    t = np.take_along_axis(t, rng.permuted(np.tile(np.arange(3), (n, 1)), axis=1)[:, :, None], axis=1)
    return t.reshape(-1, 3), np.arange(3 * n).reshape(n, 3)


@pytest.mark.parametrize("unit", [1.0, 1e-4, 1e5])
@pytest.mark.parametrize("n", [1, 5, 700, 9000])
def test_triangles_of_every_shape_and_size(ctx, oracle_mod, n, unit):
    """Closest points on and about the edges, over the planes and far from triangles that the prefilter bounds well,
    badly or not at all: the brute force's answers, bit for bit."""
    import torch

    V, F = _shards(n, 13)
    V32 = (V * unit).astype(np.float32)
    rng = np.random.default_rng(n)
    T = V[F[rng.integers(0, n, 6000)]]
    L = np.linalg.norm(T[:, 1] - T[:, 0], axis=1, keepdims=True)
    Q = (rng.dirichlet((0.4, 0.4, 0.4), 6000)[:, :, None] * T).sum(1)
    off = rng.normal(size=(6000, 3))
    off *= 10.0 ** rng.uniform(-7, 0, (6000, 1)) * np.where(rng.random((6000, 1)) < 0.5, L, 1.0)
    Q = ((Q + off) * unit).astype(np.float32)
    mesh = ctx.build_bvh(V32, F.astype(np.int32))
    t_o, d_o, b_o = oracle_mod.Scene(V32, F, bvh=False).nearest_f32(Q.astype(np.float64))
    t, d, b = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q, device="cuda")))
    print(f"[shards] {n} triangles, unit {unit:g}: {int((t != t_o).sum())} differ", flush=True)
    assert np.array_equal(d, d_o) and np.array_equal(t, t_o) and np.array_equal(b, b_o)


@pytest.mark.parametrize("name", ["needles", "small parts"])
def test_prefilter_bounds_thin_and_small_triangles(ctx, name):
    """Of the triangle slots that walks among needles (angles of 0.4 degrees) and outside parts of 3e-4 of the scene
    list, at most a quarter is left to the exact test (24 to 175 operations each; a listed slot costs 60, a node 68).
    Without a bound on them all but the pads are, three quarters of the slots and more."""
    from paper_2606_05581_amd import msk

    rng = np.random.default_rng(1)
    if name == "needles":
        V, F = W.torus_grid(4000, 8, 1.0, 0.3, weld_seam=True)
    else:
        G, T, *_ = W.geodesic_sphere(8)
        c = rng.normal(size=(30, 3))
        c *= 0.9 / np.linalg.norm(c, axis=1, keepdims=True)
        V, F = W.concat_meshes([(3e-4 * G + x, T) for x in c])
    V = W.normalise_unit_ball(V)
    case = W._point_case(V, F, 100, rng)
    exterior = name != "needles"
    mesh = ctx.build_bvh(case.V, case.F)
    d = ctx.estimate_dtn(mesh, ctx.rows(mesh, case.rows), ctx.basis(case.basis, case.V.shape[0]), 32, 1e-4, case.h,
                         exterior=exterior, collect_stats=1)
    i = d.info()
    exact = i["valu_flops"] - 68 * i["nodes_visited"] - 60 * i["tris_tested"]
    print(f"[prefilter] {name}: {i['tris_tested'] / i['queries_total']:.1f} slots a query, {exact / 175 / i['tris_tested']:.3f} "
          f"to {exact / 24 / i['tris_tested']:.3f} of them tested", flush=True)
    assert exact / 114 <= 0.25 * i["tris_tested"]
    for x, y in zip(*(_log(ctx, case, 16, exterior, 4, form=f) for f in (0, 1))):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("leaf", [1, 2, 4, 8])
def test_mesh_info_counts_the_bytes_of_its_slots(ctx, leaf):
    """128 bytes a slot, and leaves of whole blocks of 4 slots: one triangle a leaf takes 4, and no width less than 1."""
    V, F = _mesh("sphere1280")
    mesh = ctx.build_bvh(V.astype(np.float32), F.astype(np.int32), leaf_size=8)
    mesh.rebuild(leaf)
    info = mesh.info()
    assert info["tri_bytes"] % (4 * 128) == 0
    assert len(F) * 128 <= info["tri_bytes"] <= len(F) * 128 * 4
    if leaf == 1:
        assert info["tri_bytes"] == len(F) * 128 * 4


@pytest.mark.parametrize("share", [0.0, 1e-5, 0.02, 0.5, 1.0])
@pytest.mark.parametrize("n", [524288, 524289, 700001])
def test_far_points_in_large_calls(ctx, oracle_mod, n, share):
    """Calls of more than 524,288 points answer the far ones, and those that are no numbers, in a launch of their own:
    the same bits as calls of fewer points, and the brute force's on a sample."""
    import torch

    V, F = _mesh("sphere1280")
    V32 = V.astype(np.float32)
    mesh = ctx.build_bvh(V32, F.astype(np.int32))
    rng = np.random.default_rng(n)
    Q = (V[rng.integers(0, len(V), n)] * (1.0 + 0.05 * rng.normal(size=(n, 1)))).astype(np.float32)
    far = rng.random(n) < share
    far[-1] = share > 0
    Q[far] *= rng.uniform(2, 30, (int(far.sum()), 1)).astype(np.float32)
    Q[rng.random(n) < 1e-4 * share, 0] = np.nan
    whole = [x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q, device="cuda"))]
    parts = [ctx.closest_points(mesh, torch.tensor(Q[i:i + 50000], device="cuda")) for i in range(0, n, 50000)]
    ok = np.isfinite(Q).all(1)
    for k, x in enumerate(whole):
        y = np.concatenate([p[k].cpu().numpy() for p in parts])
        assert np.array_equal(x[ok] if k == 2 else x, y[ok] if k == 2 else y)  # (no barycentrics without a distance)
    sel = np.nonzero(ok)[0][:: max(1, n // 3000)]
    t_o, d_o, b_o = oracle_mod.Scene(V32, F, bvh=False).nearest_f32(Q[sel].astype(np.float64))
    assert np.array_equal(whole[0][sel], t_o) and np.array_equal(whole[1][sel], d_o) and np.array_equal(whole[2][sel], b_o)
