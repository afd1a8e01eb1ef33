"""The one-column FP64 coupling at the edges of its row tiles and column groups: degrees whose
nodes fill tiles of 16 rows exactly, leave one row over (taken by single lanes), leave a few,
and take several row and column chunks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("q", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11])
def test_one_column_coupling_degrees(q, kind):
    # against the literal FMM of the oracle; sums of at most 2,000 terms per unknown in either
    # order, so a few hundred roundings of the largest terms: 1e-12 of the norm
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B, workloads as W
    pats = W.cube_sphere()
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    sc = kind == "scalar"
    op = B.Operator(geom, 1, 2, 3.0, q, 1.6, 4, 4, 1, kind=B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE)
    assert op.info.far_pairs > 0
    o = O.Oracle(pats, 1, 2, 3.0, g=4, gs=4, scalar=sc)
    x = W.random_coeffs(op.N, q)
    y = op.apply(x)
    yo = o.fmm_apply(x, q, 1.6, 1)
    assert np.linalg.norm(y - yo) < 1e-12 * np.linalg.norm(yo)
    ctx.close()
