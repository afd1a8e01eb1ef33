"""Device memory of operators: what a request is admitted for covers what its operator holds, small
objects are admitted on small budgets, and workspaces of calls that are not made are not held."""
import numpy as np
import pytest

from paper_1807_03097_amd import workloads as W

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.mark.parametrize("surface,p,level,q,eta,depth,waves,budget", [
    ("sphere", 1, 1, 4, 1.0, -1, 1, 2),      # 0.6 MiB of data
    ("sphere", 1, 2, 4, 1.0, 1, 1, 5),
    ("sphere", 2, 2, 6, 1.0, 1, 7, 16),
    ("sphere", 2, 4, 7, 1.6, 2, 1, 177),     # the serving loop's object
    ("sphere", 4, 3, 8, 1.6, 1, 2, 182),
    ("torus", 1, 3, 7, 1.6, -1, 3, 100),
])
def test_small_objects_fit_small_budgets(surface, p, level, q, eta, depth, waves, budget):
    from paper_1807_03097_amd import binding as B
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.cube_sphere() if surface == "sphere" else W.torus())
    dirs, pols = W.random_plane_waves(waves, 3)
    srv = B.Server(ctx, 1, budget * MIB, max_merge=1)
    t = srv.submit(geom, p, level, 2.0, dirs, pols, q=q, eta=eta, leaf_depth=depth, tol=1e-6, restart=20, maxit=20)
    fp = srv.wait(t)["footprint"]
    srv.close()
    op = B.Operator(geom, p, level, 2.0, q, eta, 5, 5, depth)
    held = [int(B.ige_op_info(op.h).device_bytes)]
    F = op.rhs_plane_wave(dirs, pols)
    op.solve(F, tol=1e-6, restart=20, maxit=20)
    held.append(int(B.ige_op_info(op.h).device_bytes))
    print(f"footprint {fp / MIB:.2f} MiB, assembled {held[0] / MIB:.2f}, after a solve {held[1] / MIB:.2f}", flush=True)
    assert max(held) <= fp <= budget * MIB
    ctx.close()


@pytest.mark.parametrize("surface,p,level,q,depth,q_level", [
    ("sphere", 2, 5, 8, 3, None),            # 2,760 pairs of 96 padded nodes
    ("torus", 1, 3, 7, -1, None),            # leaves of one element
    ("sphere", 2, 5, 8, 3, [8, 8, 5]),       # level by level
])
def test_stored_fp64_coupling_is_admitted(monkeypatch, surface, p, level, q, depth, q_level):
    # stored blocks, their operands and partials are part of what a request of 8 waves is admitted for
    from paper_1807_03097_amd import binding as B
    monkeypatch.setenv("IGE_M2L_F64", "stored")
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.cube_sphere() if surface == "sphere" else W.torus())
    plan = B.Operator(geom, p, level, 2.0, q, 1.6, 5, 5, depth, plan_only=True)
    dirs, pols = W.random_plane_waves(8, 3)
    srv = B.Server(ctx, 1, 16 << 30, max_merge=1)
    t = srv.submit(geom, p, level, 2.0, dirs, pols, q=q, eta=1.6, leaf_depth=depth, tol=1e-6, restart=5, maxit=3,
                   q_level=q_level)
    fp = srv.wait(t)["footprint"]
    srv.close()
    op = B.Operator(geom, p, level, 2.0, q, 1.6, 5, 5, depth, q_level=q_level)
    before = int(B.ige_op_info(op.h).device_bytes)
    op.solve(op.rhs_plane_wave(dirs, pols), tol=1e-6, restart=5, maxit=3)
    held = int(B.ige_op_info(op.h).device_bytes)
    pairs = len(plan.partition()["far"]) // 2
    print(f"{pairs} pairs, footprint {fp / MIB:.1f} MiB, assembled {before / MIB:.1f}, after a solve {held / MIB:.1f}", flush=True)
    assert held <= fp
    ctx.close()


def test_potential_workspace_on_first_use():
    # sources of 24 x 25 points and a few points and results: well under 1 MiB
    from paper_1807_03097_amd import binding as B
    ctx = B.Context(0)
    geom = B.Geometry(ctx, W.cube_sphere())
    op = B.Operator(geom, 2, 1, 2.0, 4, 1.0, 5, 5, 1)
    before = int(B.ige_op_info(op.h).device_bytes)
    pts = 3.0 * np.eye(3)
    w = W.random_coeffs(op.N, 1)
    E = op.potential(w, pts)
    after = int(B.ige_op_info(op.h).device_bytes)
    assert 24 * 25 * 88 <= after - before < MIB
    assert np.array_equal(op.potential(w, pts), E) and int(B.ige_op_info(op.h).device_bytes) == after
    ctx.close()


@pytest.mark.parametrize("p,level", [(1, 1), (2, 3), (3, 2), (4, 1)])
def test_captured_right_hand_sides_keep_their_scratch(p, level):
    # a captured call of 20 columns finds the operator's own scratch, which later calls with more
    # room neither replace nor share: replays give the eager result
    import torch
    from paper_1807_03097_amd import binding as B
    stream = torch.cuda.Stream()
    ctx = B.Context(0, stream.cuda_stream)
    geom = B.Geometry(ctx, W.cube_sphere())
    op = B.Operator(geom, p, level, 3.0, 4, 1.0, 4, 4, 1)
    dirs, pols = W.random_plane_waves(20, 9)
    with torch.cuda.stream(stream):
        out = torch.zeros((20, op.N), dtype=torch.complex128, device="cuda:0")
        ref = torch.zeros_like(out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            op.rhs_plane_wave(dirs, pols, out=out)
        for k in range(3):
            op.rhs_plane_wave(dirs, pols, out=ref)   # its own scratch, made after the capture
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            err = float((out - ref).norm() / ref.norm())
            assert err < 1e-14, (k, err)
    ctx.close()
