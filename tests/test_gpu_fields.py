"""Right-hand sides and potentials of several columns and points against the oracle, at the
edges of the kernels' column groups and point tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("p,level,r", [(1, 1, 1), (2, 2, 3), (2, 1, 16), (1, 2, 17), (3, 1, 5), (4, 1, 33)])
def test_rhs_columns(kind, p, level, r):
    # sums of at most (p+1)^2 elements x 25 points of unit-modulus terms: a few tens of
    # roundings each, 1e-13 of the column's norm leaves a factor of more than ten
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B, workloads as W
    pats = W.cube_sphere()
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    sc = kind == "scalar"
    op = B.Operator(geom, p, level, 3.0, 4, 1.0, 5, 5, 1, kind=B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE)
    o = O.Oracle(pats, p, level, 3.0, g=5, gs=5, scalar=sc)
    dirs, pols = W.random_plane_waves(r, 11 + r)
    if sc:
        F = op.rhs_scalar(B.IGE_RHS_PLANE, dirs)
        ref = [o.rhs_scalar("plane", d) for d in dirs]
        pts = 0.3 * dirs
        F = np.concatenate([F, op.rhs_scalar(B.IGE_RHS_POINT, pts)])
        ref += [o.rhs_scalar("point", a) for a in pts]
    else:
        F = op.rhs_plane_wave(dirs, pols)
        ref = [o.rhs_plane_wave(d, q) for d, q in zip(dirs, pols)]
    for f, g in zip(F, ref):
        assert _rel(f, g) < 1e-13
    ctx.close()


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("p,level,g,r", [(1, 1, 1, 9), (1, 2, 2, 11), (2, 1, 3, 13), (2, 2, 4, 16), (2, 1, 8, 8), (3, 1, 5, 15),
                                         (2, 3, 6, 10), (4, 1, 5, 12)])
def test_rhs_ragged_columns(kind, p, level, g, r):
    # 8 to 16 columns, quadrature orders that fill a step of four points exactly, by one point and
    # less; at most 64 points per element: 1e-13 as above
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B, workloads as W
    pats = W.cube_sphere()
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    sc = kind == "scalar"
    op = B.Operator(geom, p, level, 3.0, 4, 1.0, g, 3, 1, kind=B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE)
    o = O.Oracle(pats, p, level, 3.0, g=g, gs=3, scalar=sc)
    dirs, pols = W.random_plane_waves(r, 7 + r)
    F = op.rhs_scalar(B.IGE_RHS_PLANE, dirs) if sc else op.rhs_plane_wave(dirs, pols)
    for c in range(r):
        ref = o.rhs_scalar("plane", dirs[c]) if sc else o.rhs_plane_wave(dirs[c], pols[c])
        assert _rel(F[c], ref) < 1e-13
    ctx.close()


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("p,level,npts", [(1, 1, 1), (2, 3, 3), (2, 2, 4), (3, 2, 5), (1, 4, 257)])
def test_potential_points(kind, p, level, npts):
    # 1e-13: as above, the sum of E x 25 terms; the kernel value itself is good to 1.2 ulp of
    # the phase kappa r (below 20 here)
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B, workloads as W
    pats = W.torus()
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    sc = kind == "scalar"
    op = B.Operator(geom, p, level, 5.0, 4, 1.0, 5, 5, 1, kind=B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE)
    o = O.Oracle(pats, p, level, 5.0, g=5, gs=5, scalar=sc)
    w = W.random_coeffs(op.N, 3, nrhs=2)
    rng = np.random.default_rng(npts)
    pts = rng.standard_normal((npts, 3))
    pts *= rng.uniform(1.8, 3.5, (npts, 1)) / np.linalg.norm(pts, axis=1, keepdims=True)
    E = op.potential(w, pts)
    for c in range(2):
        assert _rel(E[c], o.potential(w[c], pts)) < 1e-13
    ctx.close()
