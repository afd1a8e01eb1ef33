"""The coupling's work lists: several FP64 columns with a list whose items are longer than those of
the list that the kernel prefers, so that the two differ in length either way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", ["64", "33", "8", "1"])
def test_columns_with_any_item_size(monkeypatch, chunk):
    # 504 targets of up to 63 partners: with 64 partners per item 504 items, with 32 (those that 40
    # columns take) 984; single columns take other kernels over the same values, sums in another
    # order: under 1e-13 of the norm
    from paper_1807_03097_amd import binding as B, workloads as W
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.cube_sphere())
    monkeypatch.setenv("IGE_M2L_CHUNK", chunk)
    op = B.Operator(geom, 1, 3, 3.0, 2, 1.6, 4, 4, 0)
    far = op.partition()["far"]
    count = np.unique(far[:, 0].astype(np.int64) * 1000000 + far[:, 1], return_counts=True)[1]
    items = {n: int(np.sum(-(-count // n))) for n in (32, 64)}
    assert items[32] > items[64] and items[32] * ((4 * 40 + 63) // 64) >= 2048
    X = np.stack([W.random_coeffs(op.N, c) for c in range(40)])
    Y = op.apply(X)
    for c in (0, 15, 16, 39):
        y = op.apply(X[c].copy())
        assert np.linalg.norm(Y[c] - y) < 1e-13 * np.linalg.norm(y), c
    ctx.close()
