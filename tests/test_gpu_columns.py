"""FP64 products of several columns at the edges of their tiles: column counts around the tiles
of 8 and chunks of 64, leaves whose slots fill no, one or several row tiles of 16 and more than
eight of them, degrees whose nodes leave ragged row tiles and groups of four."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,p,m,q,depth", [
    ("efie", 1, 2, 3, 1),      # 12 slots, 16 nodes
    ("efie", 2, 3, 4, 1),      # 24 slots, 25 nodes
    ("efie", 2, 3, 6, 2),      # 60 slots, 49 nodes
    ("efie", 2, 4, 9, 3),      # 180 slots, 100 nodes
    ("scalar", 1, 3, 10, 2),   # 25 slots, 121 nodes
    ("scalar", 3, 2, 5, 2),    # 49 slots, 36 nodes
])
def test_columns_equal_single_columns(kind, p, m, q, depth):
    # single columns take other kernels over the same values; sums of at most a few thousand
    # terms in another order: under 1e-13 of the norm
    from paper_1807_03097_amd import binding as B, workloads as W
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.cube_sphere())
    op = B.Operator(geom, p, m, 3.0, q, 1.6, 4, 4, depth, kind=B.IGE_OP_SCALAR if kind == "scalar" else B.IGE_OP_EFIE)
    X = np.stack([W.random_coeffs(op.N, 10 + c) for c in range(130)])
    Y1 = {c: op.apply(X[c].copy()) for c in (0, 1, 2, 4, 7, 8, 16, 63, 64, 129)}
    for r in (2, 3, 5, 8, 9, 17, 64, 65, 130):
        Y = op.apply(X[:r].copy())
        for c, y in Y1.items():
            if c < r:
                assert np.linalg.norm(Y[c] - y) < 1e-13 * np.linalg.norm(y), (r, c)
    ctx.close()
