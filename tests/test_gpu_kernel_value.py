"""The kernel value e^{i kappa r} / (4 pi r) at large phases, by itself and in the regular
quadrature of the near field (assembled without far field)."""
import numpy as np
import pytest

from paper_1807_03097_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("top", [1e6, 4.9e7, 6e7, 1e9])
def test_value_at_large_phases(top):
    # the phase is rounded to double on the way, here and in numpy (root, product): 4 ulp of it
    from paper_1807_03097_amd import binding as B
    ctx = B.Context(0)
    r = np.linspace(0.5, 1.0, 100001)
    got = B.ige_helmholtz_eval(ctx.h, top, r * r)
    ref = np.exp(1j * top * r) / (4 * np.pi * r)
    assert np.max(np.abs(got - ref) / np.abs(ref)) <= 4 * np.spacing(top)
    ctx.close()


@pytest.mark.parametrize("kappa", [3.0, 2e8])
def test_regular_pairs_at_large_wavenumbers(oracle_mod, kappa):
    # elements on opposite faces, distances of 1 to 2: every term is off by a few ulp of its phase
    # and by the wavenumber times a few ulp of its points' positions, relative to the sum of the
    # moduli (the entries' own sums cancel)
    from paper_1807_03097_amd import binding as B
    pats = W.cube_sphere()
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    op = B.Operator(geom, 1, 1, kappa, 4, 0.0, 4, 4, -1, kind=B.IGE_OP_SCALAR)
    o = oracle_mod.Oracle(pats, 1, 1, kappa, g=4, gs=4, scalar=True)
    A, Ag = o.dense_matrix(), op.apply(np.eye(op.N, dtype=np.complex128)).T
    big = np.max(np.abs(oracle_mod.Oracle(pats, 1, 1, 0.001, g=4, gs=4, scalar=True).dense_matrix()))
    # unknowns of faces without a common corner meet only regular element pairs
    n = op.N // 6
    opposite = [(a, b) for a in range(6) for b in range(6)
                if np.allclose(o.geom(a, [[0.5, 0.5]])[0, :3], -o.geom(b, [[0.5, 0.5]])[0, :3], atol=1e-9)]
    assert len(opposite) == 6
    for a, b in opposite:
        d = np.abs(Ag - A)[a * n:(a + 1) * n, b * n:(b + 1) * n]
        assert np.max(d) <= (8 * np.spacing(2.0 * kappa) + kappa * 8 * 2.0 ** -52 + 1e-13) * big
    ctx.close()
