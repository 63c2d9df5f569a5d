"""Nearest-element searches shared by a wavefront, and the small dense steps,
at the sizes where they can go wrong.

The searches are exact: triangle, squared distance and barycentrics are the
CPU oracle's brute-force ones bit for bit, whatever the number of queries, the
leaf width, the position of the points or the shape of the triangles, and the
walks of the persistent form are those of the plain form, which searches with
a stack per lane. So these tests compare bits, not values.
"""
import numpy as np
import pytest

from paper_2606_05581_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    from paper_2606_05581_amd import msk

    assert torch.cuda.is_available(), "GPU test needs a visible MI355X"
    c = msk.Context(0)
    yield c
    c.close()


def _slivers(n, seed):
    """Needles and flakes: triangles with heights of 1e-7 to 1e-3 of their length, some of no height at all,
    for which an upper value of the distance in FP32 can be too low or missing."""
    rng = np.random.default_rng(seed)
    a = rng.uniform(-1, 1, size=(n, 3))
    d = rng.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    b = a + d * 10.0 ** rng.uniform(-3, 0, size=(n, 1))
    up = np.cross(d, rng.normal(size=(n, 3)))
    c = a + (b - a) * rng.uniform(0, 1, size=(n, 1)) + up * 10.0 ** rng.uniform(-7, -3, size=(n, 1))
    c[::17] = (0.5 * (a + b))[::17]  # no height
    c[::31] = b[::31]                # a repeated corner
    return np.stack([a, b, c], 1).reshape(-1, 3), np.arange(3 * n).reshape(n, 3)


def _mesh(name):
    if name == "tetrahedron":
        V = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]], float)
        return V, np.array([[0, 2, 1], [0, 1, 3], [0, 3, 2], [1, 2, 3]])
    if name == "slivers":
        return _slivers(3000, 3)
    return W.icosphere_recursive({"sphere20": 0, "sphere1280": 3, "sphere5120": 4}[name])


def _points(V, n, seed):
    """Near the surface, at corners, at and about the centre, in the box and up to 40 radii away."""
    rng = np.random.default_rng(seed)
    r = np.abs(V).max()
    kind = rng.integers(0, 5, size=n)
    Q = V[rng.integers(0, len(V), size=n)] * (1.0 + 1e-3 * rng.normal(size=(n, 1)))
    Q = np.where((kind == 1)[:, None], V[rng.integers(0, len(V), size=n)], Q)
    Q = np.where((kind == 2)[:, None], 1e-3 * r * rng.normal(size=(n, 3)), Q)
    Q = np.where((kind == 3)[:, None], rng.uniform(-1.3 * r, 1.3 * r, size=(n, 3)), Q)
    far = rng.normal(size=(n, 3))
    far *= r * 10.0 ** rng.uniform(0, 1.6, size=(n, 1)) / np.linalg.norm(far, axis=1, keepdims=True)
    Q = np.where((kind == 4)[:, None], far, Q)
    return Q.astype(np.float32)


@pytest.mark.parametrize("leaf", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("name", ["tetrahedron", "sphere20", "sphere1280", "slivers"])
def test_closest_points_of_few_and_many(ctx, oracle_mod, name, leaf):
    """1 to 20,001 points: a lane alone, a wavefront less and more one, queries that share wavefronts."""
    import torch

    V, F = _mesh(name)
    V32 = V.astype(np.float32)
    mesh = ctx.build_bvh(V32, F.astype(np.int32), leaf_size=leaf)
    sc = oracle_mod.Scene(V32, F, bvh=False)
    Q = _points(V, 20001, 5)
    t_o, d_o, b_o = sc.nearest_f32(Q.astype(np.float64))
    for n in (1, 2, 7, 63, 64, 65, 257, 1023, 20001):
        print(f"[closest points] {name}, leaf {leaf}, {n} points", flush=True)
        t, d, b = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q[:n], device="cuda")))
        assert np.array_equal(t, t_o[:n])
        assert np.array_equal(d, d_o[:n])
        assert np.array_equal(b, b_o[:n])


def test_points_equally_far_from_everything(ctx, oracle_mod):
    """The centre of a sphere is nearly as far from one triangle as from the next, so every search visits the
    whole tree at once and the shared stack fills up."""
    import torch

    V, F = _mesh("sphere5120")
    V32 = V.astype(np.float32)
    mesh = ctx.build_bvh(V32, F.astype(np.int32))
    Q = (1e-4 * np.random.default_rng(11).normal(size=(300, 3))).astype(np.float32)
    Q[0] = 0.0
    t_o, d_o, b_o = oracle_mod.Scene(V32, F, bvh=False).nearest_f32(Q.astype(np.float64))
    t, d, b = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q, device="cuda")))
    assert np.array_equal(t, t_o) and np.array_equal(d, d_o) and np.array_equal(b, b_o)


@pytest.mark.parametrize("unit", [1e-5, 1e-3, 1e4, 1e9])
def test_closest_points_in_other_units(ctx, oracle_mod, unit):
    """Products of the exact test underflow in small units (its value is off by up to 2^-149 over the square of
    twice the triangle's area); the prefilter must not drop what the exact test would still prefer."""
    import torch

    V, F = _mesh("sphere1280")
    V32 = (V * unit).astype(np.float32)
    mesh = ctx.build_bvh(V32, F.astype(np.int32))
    Q = (_points(V, 3000, 6).astype(np.float64) * unit).astype(np.float32)
    t_o, d_o, b_o = oracle_mod.Scene(V32, F, bvh=False).nearest_f32(Q.astype(np.float64))
    t, d, b = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q, device="cuda")))
    assert np.array_equal(d, d_o)
    some = np.isfinite(d_o)  # where every distance overflows the oracle names no triangle, the library the lowest
    assert np.array_equal(t[some], t_o[some]) and np.array_equal(b[some], b_o[some])


def test_points_that_are_no_numbers(ctx):
    """A coordinate without a value leaves every distance undefined: the answer is the lowest triangle at an
    infinite distance, and the numbers beside it are answered as ever."""
    import torch

    V, F = _mesh("sphere1280")
    mesh = ctx.build_bvh(V.astype(np.float32), F.astype(np.int32))
    Q = _points(V, 200, 8)
    t0, d0, b0 = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(Q, device="cuda")))
    R = Q.copy()
    R[::3, 1] = np.nan
    t, d, b = (x.cpu().numpy() for x in ctx.closest_points(mesh, torch.tensor(R, device="cuda")))
    bad = np.isnan(R).any(1)
    assert (t[bad] == 0).all() and np.isinf(d[bad]).all()
    assert np.array_equal(t[~bad], t0[~bad]) and np.array_equal(d[~bad], d0[~bad]) and np.array_equal(b[~bad], b0[~bad])


def _log(ctx, case, walks, exterior, leaf, **opts):
    from paper_2606_05581_amd import msk

    mesh = ctx.build_bvh(case.V, case.F, leaf_size=leaf)
    rows = ctx.rows(mesh, case.rows)
    basis = ctx.basis(case.basis, case.V.shape[0])
    d = ctx.estimate_dtn(mesh, rows, basis, walks, case.eps, case.h, exterior=exterior, record_log=1, **opts)
    return [d.get(f) for f in (msk.FIELD_LOG_STATUS, msk.FIELD_LOG_TRI, msk.FIELD_LOG_BARY, msk.FIELD_LOG_QUERIES,
                               msk.FIELD_ROW_DISCARDED)]


@pytest.mark.parametrize("exterior", [False, True], ids=["interior", "exterior"])
@pytest.mark.parametrize("n_rows,walks,leaf", [(2, 2, 4), (3, 21, 1), (9, 7, 8), (16, 4, 5), (33, 31, 4), (130, 66, 8)])
def test_few_walks_take_the_plain_forms_paths(ctx, n_rows, walks, leaf, exterior):
    """Launches from a few walks (several lanes to a walk) to many wavefronts of them, all leaf widths."""
    V, F = _mesh("sphere1280")
    case = W._point_case(V * np.array([1.0, 0.7, 0.5]), F, n_rows, np.random.default_rng(n_rows))
    print(f"[few walks] {n_rows} rows x {walks} walks, leaf {leaf}", flush=True)
    a = _log(ctx, case, walks, exterior, leaf, form=0)
    b = _log(ctx, case, walks, exterior, 4, form=1)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_slivers_walk_the_same_paths(ctx):
    """Meshes whose triangles have upper values that mean nothing search again with exact ones."""
    V, F = _mesh("sphere1280")
    S, G = _slivers(200, 9)
    V, F = np.concatenate([V, 0.4 * S]), np.concatenate([F, G + len(V)])
    case = W._point_case(V, F, 100, np.random.default_rng(2))
    for exterior in (False, True):
        a, b = (_log(ctx, case, 32, exterior, 4, form=f) for f in (0, 1))
        for x, y in zip(a, b):
            assert np.array_equal(x, y)


def test_batch_of_mixed_leaf_widths_and_rows(ctx):
    """One batch of hat and point rows on meshes of different leaf widths against each mesh alone: the same
    walks, so entries differ by the order of their FP64 sums only (at most 2^-53 per addition, 512 walks of
    weights below the largest entry: 1e-12 of it)."""
    from paper_2606_05581_amd import msk

    cases = [W.unit_sphere_320().cases[0]]
    for name, n in (("sphere1280", 40), ("sphere5120", 9)):
        V, F = _mesh(name)
        cases.append(W._point_case(V, F, n, np.random.default_rng(n)))
    hs = []
    for case, leaf in zip(cases, (8, 3, 4)):
        mesh = ctx.build_bvh(case.V, case.F, leaf_size=leaf)
        hs.append((mesh, ctx.rows(mesh, case.rows), ctx.basis(case.basis, case.V.shape[0])))
    plan = ctx.batch(*zip(*hs), [c.eps for c in cases], [c.h for c in cases], 64, seed=3)
    for _ in range(3):
        plan.run()
        for i, (case, h) in enumerate(zip(cases, hs)):
            d = ctx.estimate_dtn(*h, 64, case.eps, case.h, seed=3, mesh_id=i)
            S, v = d.get(msk.FIELD_S), plan.dtn(i)
            assert np.array_equal(v.get(msk.FIELD_ROW_QUERIES), d.get(msk.FIELD_ROW_QUERIES))
            assert np.abs(v.get(msk.FIELD_S) - S).max() <= 1e-12 * np.abs(S).max()


@pytest.mark.parametrize("n_rows", [1, 2, 65, 300])
def test_tangent_balls_do_not_depend_on_the_leaf_width(ctx, n_rows):
    V, F = _mesh("sphere1280")
    V = (V * np.array([1.0, 0.6, 0.3])).astype(np.float32)
    rows = W.point_rows(V.astype(np.float64), F, n_rows, np.random.default_rng(4))
    tab = np.stack([np.ones(len(V)), V[:, 0], V[:, 1]], 1).astype(np.float32)
    res = []
    for leaf in (1, 4, 8):
        mesh = ctx.build_bvh(V, F.astype(np.int32), leaf_size=leaf)
        r = ctx.estimate_psd(mesh, ctx.rows(mesh, rows), ctx.basis(W.dense_basis(tab), len(V)), 3, 1e-4, seed=7, log=True)
        res.append(r)
    assert (res[0]["radius"] > 0).any()
    for r in res[1:]:
        for k in ("radius", "status", "tri", "bary"):
            assert np.array_equal(r[k], res[0][k]), k


@pytest.mark.parametrize("power", [-60, -31, 33, 60])
def test_kelvin_walks_in_any_unit(ctx, power):
    """A mesh in units of 2^power: every length of the inverted domain scales by 2^-power without rounding, so
    the walks hit the same triangles in the same number of queries. Squared lengths leave FP32's range there."""
    V, F = W.icosphere_recursive(3)
    tab = np.ones((len(V), 1), dtype=np.float32)
    rows = W.point_rows(V.astype(np.float32).astype(np.float64), F, 70, np.random.default_rng(8))
    out = []
    for u in (1.0, 2.0 ** power):
        Vu = (V.astype(np.float32) * np.float32(u)).astype(np.float32)
        ru = type(rows)(**{**vars(rows), "p": (rows.p * np.float32(u)).astype(np.float32), "w": rows.w * u * u})
        mesh = ctx.build_bvh(Vu, F.astype(np.int32))
        kv = ctx.kelvin(mesh, np.array([0.25, -0.125, 0.0625]) * u)
        out.append(ctx.estimate_kelvin(kv, ctx.rows(mesh, ru), ctx.basis(W.dense_basis(tab), len(V)), 8, 500,
                                       2.0 ** -14 * 2.0 / u, seed=5, log=True))
    a, b = out
    assert (a["nq"] > 0).any()
    for k in ("status", "tri", "nq"):
        assert np.array_equal(a[k], b[k]), k


# ------------------------------------------------------- small dense steps


@pytest.mark.parametrize("level,K", [(2, 8), (2, 60), (3, 64), (3, 100), (4, 120), (4, 130), (5, 40)])
def test_mesh_basis_of_every_block_width(ctx, level, K):
    """Blocks of 64 and 128 columns factor on the device, wider ones on the host; 162 to 10,242 vertices sum 4 to
    164 partial blocks. Eigenvalues of dense LAPACK within 1e-9 of the spectral bound (the residual target is
    1e-12 of it), Phi^T M Phi = I within 1e-10."""
    from oracle import laplace as LP

    V, F = W.icosphere_recursive(level)
    V = (V * np.array([1.0, 0.8, 0.6])).astype(np.float32)
    b, lam, Phi, info = ctx.basis_laplacian(V, F.astype(np.int32), K)
    b.close()
    L, m, _ = LP.cotan_laplacian(V.astype(np.float64), F)
    if len(V) <= 3000:
        s = 1.0 / np.sqrt(m)
        A = L.toarray() * s[:, None] * s[None, :]
        ref = np.linalg.eigvalsh(0.5 * (A + A.T))[:K]
    else:
        ref = LP.laplacian_basis(V.astype(np.float64), F, K)[0]
    print(f"[mesh basis] {len(V)} vertices, K = {K}: block {info['block']}, worst {np.abs(lam - ref).max():.2e} "
          f"of {info['bound']:.2e}", flush=True)
    assert info["converged"]
    assert np.abs(lam - ref).max() <= 1e-9 * info["bound"]
    assert np.abs(Phi.T @ (m[:, None] * Phi) - np.eye(K)).max() < 1e-10


@pytest.mark.parametrize("n_rows,k", [(513, 3), (577, 33), (1001, 64), (1030, 17)])
def test_eigen_step_of_odd_sizes(ctx, n_rows, k):
    """Row counts that no tile divides and whose rows are not 16-byte aligned, blocks of 32 to 64 columns, against
    LAPACK on the same estimate: products with C are FP32, Rayleigh quotients FP64, so 1e-6 |C|."""
    from paper_2606_05581_amd import msk

    V, F = _mesh("sphere5120")
    case = W._point_case(V * np.array([1.0, 0.7, 0.5]), F, n_rows, np.random.default_rng(1))
    mesh = ctx.build_bvh(case.V, case.F)
    rows = ctx.rows(mesh, case.rows)
    d = ctx.estimate_dtn(mesh, rows, ctx.basis(case.basis, case.V.shape[0]), 64, case.eps, case.h)
    S, disc = d.get(msk.FIELD_S), d.get(msk.FIELD_ROW_DISCARDED)
    keep = np.nonzero((case.rows.w > 0) & (disc == 0))[0]
    s = 1.0 / np.sqrt(case.rows.w[keep])
    C = 0.5 * (S + S.T)[np.ix_(keep, keep)] * s[:, None] * s[None, :]
    ref = np.linalg.eigvalsh(C)
    ev, psi, st = ctx.steklov_modes(d, k)
    print(f"[eigen step] {len(keep)} rows, k = {k}: {np.abs(ev - ref[:k]).max() / np.abs(ref).max():.2e} of |C|, "
          f"{st['iterations']} cycles, block {st['block']}", flush=True)
    assert st["converged"]
    assert np.abs(ev - ref[:k]).max() <= 1e-6 * np.abs(ref).max()
    P = psi[keep] * np.sqrt(case.rows.w[keep])[:, None]
    assert np.abs(P.T @ P - np.eye(k)).max() <= 1e-8
