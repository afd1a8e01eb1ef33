"""The one-column FP64 coupling over unordered far pairs against forms that share no kernel with
it: stored blocks, several columns (ordered pairs), and the oracle.  Meshes with enough far pairs
for whole clusters per work item, so that degrees 8 to 15 take six and eight row tiles, the single
row over (81 nodes) and several row chunks, in the launch shared with the near field and by itself."""
import numpy as np
import pytest

from paper_1807_03097_amd import workloads as W

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


MESHES = {"sphere": (3, 5520),   # two or four partners per item
          "torus": (2, 1920)}    # one partner per item


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("surface", sorted(MESHES))
@pytest.mark.parametrize("q", [2, 4, 6, 7, 8, 9, 10, 11])
def test_one_column_equals_other_forms(q, surface, kind):
    # the same kernel values (within 1.2 ulp of the phase) and sums of a few thousand terms in
    # another order: under 1e-13 of the norm; 1e-12 against the oracle
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B
    level, npairs = MESHES[surface]
    pats = W.cube_sphere() if surface == "sphere" else W.torus()
    sc = kind == "scalar"
    kd = B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    op = B.Operator(geom, 1, level, 3.0, q, 1.6, 4, 4, 1, kind=kd)
    st = B.Operator(geom, 1, level, 3.0, q, 1.6, 4, 4, 1, kind=kd, store_coupling=1)
    assert op.info.far_pairs == npairs and npairs // 2 >= 256
    x = W.random_coeffs(op.N, q)
    y = op.apply(x)
    op.set_overlap(False)   # the coupling and the near field in launches of their own
    assert _rel(op.apply(x), y) < 1e-13
    assert _rel(st.apply(x), y) < 1e-13
    for c in op.apply(np.stack([x, x])):
        assert _rel(c, y) < 1e-13
    assert _rel(y, O.Oracle(pats, 1, level, 3.0, g=4, gs=4, scalar=sc).fmm_apply(x, q, 1.6, 1)) < 1e-12
    ctx.close()


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("degrees", [(4, 5, 15), (4, 15, 12), (3, 10, 8), (2, 3, 11), (12, 8, 1)])
def test_one_column_degree_per_level(degrees, kind):
    # far pairs on the levels 1 and 2, node counts from 4 to 256 in one launch
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B
    pats = W.cube_sphere()
    sc = kind == "scalar"
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    op = B.Operator(geom, 1, 3, 3.0, 4, 1.6, 4, 4, 1, kind=B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE, q_level=degrees)
    assert set(op.partition()["far"][:, 0]) == {1, 2}
    x = W.random_coeffs(op.N, 5)
    y = op.apply(x)
    op.set_overlap(False)
    assert _rel(op.apply(x), y) < 1e-13
    for c in op.apply(np.stack([x, x, x])):
        assert _rel(c, y) < 1e-13
    assert _rel(y, O.Oracle(pats, 1, 3, 3.0, g=4, gs=4, scalar=sc).fmm_apply(x, list(degrees), 1.6, 1)) < 1e-12
    ctx.close()


def test_info_names_asked_items_only(monkeypatch):
    # m2l_unordered says whether the items were asked for; the coupling is over unordered pairs
    # either way, and both operators match the stored blocks
    from paper_1807_03097_amd import binding as B
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.cube_sphere())
    op = B.Operator(geom, 1, 3, 3.0, 6, 1.6, 4, 4, 1)
    st = B.Operator(geom, 1, 3, 3.0, 6, 1.6, 4, 4, 1, store_coupling=1)
    monkeypatch.setenv("IGE_M2L_SYM", "1")
    asked = B.Operator(geom, 1, 3, 3.0, 6, 1.6, 4, 4, 1)
    assert (op.info.m2l_unordered, asked.info.m2l_unordered) == (0, 1)
    x = W.random_coeffs(op.N, 1)
    y = st.apply(x)
    assert _rel(op.apply(x), y) < 1e-13 and _rel(asked.apply(x), y) < 1e-13
    ctx.close()


@pytest.mark.parametrize("kind", ["efie", "scalar"])
@pytest.mark.parametrize("q", [4, 8, (4, 6, 10), (4, 10, 3)])
def test_stored_fp64_blocks_equal_evaluated(monkeypatch, q, kind):
    # 8, 9 and 70 columns: one chunk, a ragged one, several; the same values and sums of a few
    # thousand terms in another order: under 1e-13 of the norm
    from oracle import oracle as O
    from paper_1807_03097_amd import binding as B
    pats = W.cube_sphere()
    sc = kind == "scalar"
    kw = dict(kind=B.IGE_OP_SCALAR if sc else B.IGE_OP_EFIE, q_level=q if isinstance(q, tuple) else None)
    q0 = q[0] if isinstance(q, tuple) else q
    ctx = B.Context(0)
    geom = B.Geometry(ctx, pats)
    op = B.Operator(geom, 1, 3, 3.0, q0, 1.6, 4, 4, 1, **kw)
    monkeypatch.setenv("IGE_M2L_F64", "stored")
    st = B.Operator(geom, 1, 3, 3.0, q0, 1.6, 4, 4, 1, **kw)
    far = st.partition()["far"]
    deg = [d if isinstance(q, int) else q[l] for l, d in zip(far[:, 0], [q0] * len(far))]
    qp = [32 * (-(-(d + 1) ** 2 // 32)) for d in deg]
    blocks = sum(2 * n * n * 8 for n in qp)   # per ordered pair [Qp][2 Qp] doubles
    held = {o: int(B.ige_op_info(o.h).device_bytes) for o in (op, st)}
    X = np.stack([W.random_coeffs(op.N, 40 + c) for c in range(70)])
    for r in (8, 9, 70):
        Y, Z = op.apply(X[:r].copy()), st.apply(X[:r].copy())
        for c in range(r):
            assert _rel(Z[c], Y[c]) < 1e-13, (r, c)
    more = {o: int(B.ige_op_info(o.h).device_bytes) - held[o] for o in (op, st)}
    assert more[st] - more[op] >= blocks   # the second operator did store them
    yo = O.Oracle(pats, 1, 3, 3.0, g=4, gs=4, scalar=sc).fmm_apply(X[69], list(q) if isinstance(q, tuple) else q, 1.6, 1)
    assert _rel(Z[69], yo) < 1e-12
    ctx.close()


def test_autotuner_gives_back_rejected_blocks():
    # the memory of the stored blocks is held after the call only if they were chosen
    from paper_1807_03097_amd import binding as B
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.torus())
    op = B.Operator(geom, 1, 3, 3.0, 6, 1.6, 4, 4, 1)
    X = np.stack([W.random_coeffs(op.N, c) for c in range(9)])
    Y = op.apply(X)
    held = int(B.ige_op_info(op.h).device_bytes)
    chosen = op.autotune(9)["m2l_f64_matrix_cores"]
    more = int(B.ige_op_info(op.h).device_bytes) - held
    blocks = int(op.info.far_pairs) * 64 * 2 * 64 * 8   # 49 nodes: [64][128] doubles per ordered pair
    print(f"stored blocks chosen {chosen}: {more} bytes more, blocks {blocks}", flush=True)
    assert more >= blocks if chosen == 1 else more == 0
    Z = op.apply(X)
    for c in range(9):
        assert _rel(Z[c], Y[c]) < 1e-13
    # asked for again, they are made again
    assert op.autotune(9)["m2l_f64_matrix_cores"] in (0, 1)
    ctx.close()
