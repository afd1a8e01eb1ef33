"""The performance cases of the framework: what its users have it do, over the range of
sizes, precisions and options that they use, each through the Python binding.

  listed()            the cases that are followed
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what a user's program holds before the call, on the device
  run(state)          one pass: the call, and all that it returns
  work(case)          bytes and floating-point operations that the pass cannot do without
  exact(case, seed)   what run returns, in plain numpy / torch in 64 bits, where the result is
                      a quadrature that takes seconds that way (right-hand sides and
                      potentials).  The operator's own products, assemblies and solves have
                      none: a value to compare with is a complete literal FMM with singular
                      quadrature of every touching element pair, minutes of plain numpy.

Every case is a scattering problem on one of the closed surfaces of `workloads`, its
control points moved a little by the seed (another seed is another scatterer), with the
splines, cluster tree and interpolation degree that the case names.  `call` says what the
pass is:

  apply      y = A x of `cols` columns in the coupling precision `prec`, on device vectors
  assemble   a new operator, applied to its first vector, and given back
  solve      GMRES on `cols` incident waves from x = 0
  rhs        the right-hand sides of `cols` incident waves
  potential  the scattered field of one current at `points` points around the object
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1807_03097_amd import binding as B
from paper_1807_03097_amd import workloads as W

GAUSS = 5          # points per direction of the regular and of the singular rules
JITTER = 2e-3      # standard deviation of the control points' displacement
SOLVE_ITERS = 800  # iterations that work() counts for a solve (the listed one takes 829)
RESTART = 300      # Krylov basis of a solve

_context = None


def _ctx():
    """the process's one device context, as a program keeps it"""
    global _context
    if _context is None:
        torch.cuda.set_device(0)
        _context = B.Context(0)
    return _context


def _case(name, call, **kw):
    c = {"name": name, "call": call, "surface": "sphere", "kind": "efie", "p": 2, "level": 5, "kappa": 8.0, "q": 8,
         "eta": 1.6, "leaf_depth": 3, "rule": False, "kappa_cap": 0.0, "cols": 1, "prec": B.IGE_F64, "points": 0}
    c.update(kw)
    return c


def listed():
    return [
        # a small object far below the device's size: launches and latency
        _case("matvec_l3", "apply", level=3, q=6, eta=1.0, leaf_depth=1),
        # the product inside every solve of the benchmark's mesh (N = 13,068)
        _case("matvec_l5", "apply"),
        # the same in the precision of the inner solves of one refined right-hand side, on
        # a torus with first-degree splines and the library's own leaf size
        _case("matvec_f32_torus", "apply", surface="torus", p=1, level=4, kappa=5.0, q=7, leaf_depth=-1,
              prec=B.IGE_F32),
        # high wavenumber, one degree per level from the kappa * diam rule (N = 50,700)
        _case("matvec_l6_rule", "apply", level=6, kappa=16.0, rule=True),
        # a handful of sources on the scalar single layer
        _case("scalar_block5", "apply", kind="scalar", level=4, kappa=3.0, q=7, eta=1.0, leaf_depth=2, cols=5),
        # a radar sweep of an odd number of incident directions
        _case("block23_torus", "apply", surface="torus", level=4, kappa=6.0, q=6, leaf_depth=2, cols=23),
        # the benchmark's 64 waves: outer residuals in FP64, inner products in split BF16
        _case("block64_l6", "apply", level=6, kappa=16.0, cols=64),
        _case("block64_l6_split", "apply", level=6, kappa=16.0, cols=64, prec=B.IGE_BF16X3_ALL),
        # every request of the serving loop on a new object begins with this
        _case("assemble_l5", "assemble"),
        # one request of the serving loop
        _case("solve_l4", "solve", level=4, kappa=6.0, q=7, leaf_depth=2),
        # the right-hand sides of 64 waves, and the field around the object afterwards
        _case("rhs64_l6", "rhs", level=6, kappa=16.0, cols=64),
        _case("potential_l5", "potential", points=3000),
    ]


def draw(rng):
    call = rng.choice(["apply"] * 7 + ["assemble", "solve", "rhs", "potential"])
    surface = rng.choice(["sphere", "torus"])
    kind = rng.choice(["efie", "efie", "scalar"])
    c = {"call": call, "surface": surface, "kind": kind, "p": rng.choice([1, 2, 2, 3])}
    top = 5 if surface == "torus" else 6      # 16 patches against 6
    if call in ("assemble", "solve"):
        top -= 1
    if call == "solve":
        top -= 1
    c["level"] = rng.randint(2 if surface == "torus" else 3, top)
    c["kappa"] = round(math.exp(rng.uniform(math.log(1.0), math.log(16.0))), 2)
    c["q"] = rng.randint(4, 9)
    c["eta"] = rng.choice([0.8, 1.0, 1.6])
    c["leaf_depth"] = rng.choice([-1, 2, 3]) if c["level"] > 3 else -1
    c["rule"] = call == "apply" and rng.random() < 0.2
    c["kappa_cap"] = 8.0 if rng.random() < 0.1 else 0.0
    c["cols"], c["prec"], c["points"] = 1, B.IGE_F64, 0
    if call == "apply":
        c["cols"] = rng.choice([1, 1, int(round(math.exp(rng.uniform(math.log(2.0), math.log(64.0)))))])
        c["prec"] = rng.choice([B.IGE_F64] * 4 + [B.IGE_F32, B.IGE_BF16X3, B.IGE_BF16X3_ALL])
        if c["prec"] >= B.IGE_BF16X3:
            c["cols"] = max(c["cols"], 8)
            c["rule"] = False
    elif call == "solve":
        c["kind"] = "efie"
        c["cols"] = rng.choice([1, 1, 4, 11])
    elif call == "rhs":
        c["cols"] = int(round(math.exp(rng.uniform(0.0, math.log(64.0)))))
    elif call == "potential":
        c["points"] = int(round(math.exp(rng.uniform(math.log(10.0), math.log(3000.0)))))
        c["level"] = min(c["level"], 5)
    return c


# ---- what a program holds before the call ------------------------------------------------
def _patches(case, seed):
    base = W.torus() if case["surface"] == "torus" else W.cube_sphere()
    return W.jitter(base, JITTER, seed)


def _operator(geom, case, plan_only=False):
    kind = B.IGE_OP_SCALAR if case["kind"] == "scalar" else B.IGE_OP_EFIE
    args = (case["p"], case["level"], case["kappa"], case["q"], case["eta"], GAUSS, GAUSS, case["leaf_depth"])
    levels = None
    if case["rule"]:
        plan = B.Operator(geom, *args, plan_only=True, kappa_cap=case["kappa_cap"], kind=kind)
        far = set(plan.partition()["far"][:, 0].tolist())
        levels = B.degree_rule(plan.info, case["kappa"], case["q"], far)
        plan.close()
    return B.Operator(geom, *args, plan_only=plan_only, kappa_cap=case["kappa_cap"], kind=kind, q_level=levels)


def _columns(n, r, seed, device):
    """r columns of N(0,1) + i N(0,1) entries, as [r][n] (one column: [n])"""
    g = torch.Generator(device="cpu").manual_seed(seed)
    x = torch.randn((r, n, 2), generator=g, dtype=torch.float64)
    x = torch.view_as_complex(x).to(device)
    return x[0].contiguous() if r == 1 else x


def _points(n, seed):
    """points of a shell around the object, 1.6 to 3 times its radius"""
    rng = np.random.default_rng(seed)
    d = rng.standard_normal((n, 3))
    return d / np.linalg.norm(d, axis=1, keepdims=True) * rng.uniform(1.6, 3.0, (n, 1))


def prepare(case, seed):
    st = {"case": case, "geom": B.Geometry(_ctx(), _patches(case, seed))}
    dev = torch.device("cuda:0")
    call, r = case["call"], case["cols"]
    if call == "assemble":
        plan = _operator(st["geom"], case, plan_only=True)
        st["x"] = _columns(plan.N, 1, seed, dev)
        plan.close()
        torch.cuda.synchronize()
        return st
    op = st["op"] = _operator(st["geom"], case)
    if call == "apply":
        st["x"] = _columns(op.N, r, seed, dev)
        st["y"] = torch.empty_like(st["x"])
    elif call in ("solve", "rhs"):
        st["dirs"], st["pols"] = W.random_plane_waves(r, seed)
        st["f"] = torch.empty((r, op.N), dtype=torch.complex128, device=dev)
        if call == "solve":
            _rhs(st)
    else:
        st["w"] = _columns(op.N, 1, seed, dev)
        st["points"] = _points(case["points"], seed)
    torch.cuda.synchronize()
    return st


def _rhs(st):
    if st["case"]["kind"] == "scalar":
        return st["op"].rhs_scalar(B.IGE_RHS_PLANE, st["dirs"], out=st["f"])
    return st["op"].rhs_plane_wave(st["dirs"], st["pols"], out=st["f"])


# ---- one pass ------------------------------------------------------------------------------
def run(st):
    case = st["case"]
    call = case["call"]
    if call == "apply":
        return st["op"].apply(st["x"], st["y"], prec=case["prec"])
    if call == "assemble":
        op = _operator(st["geom"], case)
        y = op.apply(st["x"])
        op.close()
        return y
    if call == "solve":
        return st["op"].solve(st["f"], tol=1e-6, restart=RESTART, maxit=3000)[0]
    if call == "rhs":
        return _rhs(st)
    return st["op"].potential(st["w"], st["points"])


# ---- what a pass cannot do without -----------------------------------------------------------
def _product(info, plan, r, scalar):
    """bytes and operations of one product of r columns: every distinct near-field entry read
    once and used for both of its unknowns, one kernel value per unordered node pair of the
    far blocks (46 operations with the first column's products), its products with the
    columns, the moments at a lower order"""
    n, near = int(info.n_dof), int(info.near_distinct)
    far = plan.partition()["far"] if info.far_pairs else np.zeros((0, 3), np.int32)
    per = np.array([(int(info.q_level[l]) + 1) ** 2 for l in range(int(info.leaf_level) + 1)], np.float64)
    nodes = float(np.sum(per[far[:, 0]] ** 2)) if len(far) else 0.0
    fields = 1 if scalar else 4
    return 16.0 * near + 32.0 * n * r, 16.0 * near * r + nodes * (0.5 * 30 + 8.0 * fields * r)


def work(case):
    geom = B.Geometry(B.Context(-1), _patches(case, 0))
    plan = _operator(geom, case, plan_only=True)
    info, call, r, scalar = plan.info, case["call"], case["cols"], case["kind"] == "scalar"
    n, el, g2, p = plan.N, int(info.n_elements), GAUSS ** 2, case["p"]
    nl = (p + 1) ** 2 if scalar else 2 * p * (p + 1)
    nb, nf = _product(info, plan, r, scalar)
    if call == "apply":
        w = {"bytes": nb, "flops": nf}
    elif call == "assemble":
        # the element pairs of the near leaf pairs, each unordered pair once, with the regular
        # rule: kernel values and the two products with the local functions (4 fields)
        leaf = el / (4.0 ** int(info.leaf_level) * geom_patches(case))
        pairs = 0.5 * float(info.near_leaf_pairs) * leaf * leaf
        per = g2 * g2 * 46.0 + 16.0 * (g2 * g2 * nl + g2 * nl * nl)
        sing = float(info.singular_pairs) * 3300.0 * (46.0 + 4.0 * nl * nl)
        w = {"bytes": nb, "flops": nf + pairs * per + sing}
    elif call == "solve":
        basis = SOLVE_ITERS * RESTART / 2
        w = {"bytes": SOLVE_ITERS * nb + 32.0 * basis * n * r, "flops": SOLVE_ITERS * nf + 16.0 * basis * n * r}
    elif call == "rhs":
        w = {"bytes": 72.0 * el * g2 + 16.0 * n * r, "flops": r * el * g2 * (40.0 + 8.0 * 2 + 4.0 * nl)}
    else:
        w = {"bytes": 72.0 * el * g2 + 72.0 * case["points"],
             "flops": el * g2 * (case["points"] * (46.0 + (8.0 if scalar else 44.0)) + 8.0 * nl)}
    plan.close()
    return w


def geom_patches(case):
    return 16 if case["surface"] == "torus" else 6


# ---- plain 64-bit values ------------------------------------------------------------------------
def _splines(p, n, t):
    """values and derivatives of the B-splines of degree p on n uniform spans, [len(t)][n+p]"""
    kn = np.r_[np.zeros(p + 1), np.arange(1, n) / n, np.ones(p + 1)]
    span = np.minimum((t * n).astype(int), n - 1) + p
    b = np.zeros((len(t), len(kn) - 1))
    b[np.arange(len(t)), span] = 1.0
    lower = b
    for k in range(1, p + 1):
        lower, c = b, np.zeros((len(t), len(kn) - 1 - k))
        for i in range(c.shape[1]):
            if kn[i + k] > kn[i]:
                c[:, i] += (t - kn[i]) / (kn[i + k] - kn[i]) * b[:, i]
            if kn[i + k + 1] > kn[i + 1]:
                c[:, i] += (kn[i + k + 1] - t) / (kn[i + k + 1] - kn[i + 1]) * b[:, i + 1]
        b = c
    d = np.zeros_like(b)
    for i in range(b.shape[1] if p else 0):
        if kn[i + p] > kn[i]:
            d[:, i] += p / (kn[i + p] - kn[i]) * lower[:, i]
        if kn[i + p + 1] > kn[i + 1]:
            d[:, i] -= p / (kn[i + p + 1] - kn[i + 1]) * lower[:, i + 1]
    return b, d


def _surface(patch, t, s):
    """points and both tangents of a one-span rational patch on the grid s x t, [s][t][3]"""
    def bern(p, z):
        c = np.array([math.comb(p, i) for i in range(p + 1)], float)
        v = np.stack([c[i] * z ** i * (1 - z) ** (p - i) for i in range(p + 1)], 1)
        e = np.stack([math.comb(p - 1, i) * z ** i * (1 - z) ** (p - 1 - i) for i in range(p)], 1)
        d = np.zeros_like(v)
        d[:, 1:] += p * e
        d[:, :-1] -= p * e
        return v, d
    hom = patch["ctrl"].copy()
    hom[..., :3] *= hom[..., 3:]
    (u, du), (v, dv) = bern(patch["deg"][0], t), bern(patch["deg"][1], s)
    h, hu, hv = (np.einsum("bj,ai,jik->bak", y, x, hom) for x, y in ((u, v), (du, v), (u, dv)))
    F = h[..., :3] / h[..., 3:]
    return F, (hu[..., :3] - F * hu[..., 3:]) / h[..., 3:], (hv[..., :3] - F * hv[..., 3:]) / h[..., 3:]


def _unknowns(patches, p, n):
    """index and sign of the divergence-conforming functions, [patch][component][i2][i1]: the
    normal-flux functions of shared edges are one unknown, numbered where it first occurs"""
    ends = {}
    for j, pt in enumerate(patches):
        for k, (t, s) in enumerate((((0, .3, 1), (0,)), ((1,), (0, .3, 1)), ((0, .3, 1), (1,)), ((0,), (0, .3, 1)))):
            ends[j, k] = _surface(pt, np.array(t, float), np.array(s, float))[0].reshape(3, 3)
    mate = {}   # edge -> (partner, reversed); a reversed partner has the point t = .3 at t = .7
    for a in ends:
        for b in ends:
            if a != b and np.abs(ends[a][[0, 2]] - ends[b][[0, 2]]).max() < 1e-9:
                if np.abs(ends[a][1] - ends[b][1]).max() < 1e-9:
                    mate[a] = (b, False)
            elif a != b and np.abs(ends[a][[0, 2]] - ends[b][[2, 0]]).max() < 1e-9:
                j, k = b
                t = np.array([0.7])
                z = np.array([(0.0, 1.0, 1.0, 0.0)[k]])
                mid = _surface(patches[j], *((t, z) if k in (0, 2) else (z, t)))[0].reshape(3)
                if np.abs(ends[a][1] - mid).max() < 1e-9:
                    mate[a] = (b, True)
    side, m = (-1, 1, 1, -1), n + p
    dof = np.full((len(patches), 2, m, m), -1)
    sgn = np.ones((len(patches), 2, m, m))
    N = 0
    for j in range(len(patches)):
        for a in range(2):
            for i2 in range(m - 1 + a):
                for i1 in range(m - a):
                    if dof[j, a, i2, i1] >= 0:
                        continue
                    dof[j, a, i2, i1] = N
                    i, t = (i1, i2) if a == 0 else (i2, i1)
                    if i in (0, m - 1):
                        k = (3, 1)[i > 0] if a == 0 else (0, 2)[i > 0]
                        (jb, kb), back = mate[j, k]
                        tb = m - 2 - t if back else t
                        at = ((1, 0, tb), (0, tb, m - 1), (1, m - 1, tb), (0, tb, 0))[kb]
                        dof[(jb,) + at] = N
                        sgn[(jb,) + at] = -side[k] * side[kb]
                    N += 1
    return dof, sgn, N


def exact(case, seed):
    if case["call"] not in ("rhs", "potential"):
        return None
    dev = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    patches, p, n, kappa = _patches(case, seed), case["p"], 1 << case["level"], case["kappa"]
    scalar = case["kind"] == "scalar"
    x, w = np.polynomial.legendre.leggauss(GAUSS)
    t = ((np.arange(n)[:, None] + 0.5 * (x + 1)) / n).ravel()
    wt = np.tile(0.5 * w / n, n)
    wt = torch.from_numpy(wt[:, None] * wt).to(dev)
    (bp, dp), (bq, _) = _splines(p, n, t), _splines(p - 1, n, t)
    bp, dp, bq = (torch.from_numpy(v).to(dev) for v in (bp, dp, bq))
    m = n + p
    if scalar:
        N = len(patches) * m * m
        dof, sgn = np.arange(N).reshape(len(patches), 1, m, m), np.ones((len(patches), 1, m, m))
    else:
        dof, sgn, N = _unknowns(patches, p, n)
    grids = [[torch.from_numpy(v).to(dev) for v in _surface(pt, t, t)] for pt in patches]
    area = [torch.linalg.norm(torch.cross(u, v, dim=-1), dim=-1) for _, u, v in grids]

    if case["call"] == "rhs":
        dirs, pols = (torch.from_numpy(v).to(dev) for v in W.random_plane_waves(case["cols"], seed))
        f = torch.zeros((case["cols"], N), dtype=torch.complex128, device=dev)
        for j, (F, u, v) in enumerate(grids):
            # (row factor, column factor, functions, tested field) of each component
            parts = [(bp, bp, (slice(0, m), slice(0, m)), area[j])] if scalar else \
                [(bq, bp, (slice(0, m - 1), slice(0, m)), u), (bp, bq, (slice(0, m), slice(0, m - 1)), v)]
            for a, (b2, b1, sl, tang) in enumerate(parts):
                i = torch.from_numpy(np.ascontiguousarray(dof[j, a][sl]).ravel()).to(dev)
                s = torch.from_numpy(np.ascontiguousarray(sgn[j, a][sl]).ravel()).to(dev)
                for c in range(case["cols"]):
                    e = torch.exp(1j * kappa * (F @ dirs[c])) * wt
                    e = e * tang if scalar else -e * (tang.to(torch.complex128) @ pols[c])
                    f[c].index_add_(0, i, s * (b2.T.to(e.dtype) @ e @ b1.to(e.dtype)).ravel())
        return f

    wx = _columns(N, 1, seed, dev)
    X, S, D = [], [], []   # points, weighted vector density, weighted divergence / scalar density
    for j, (F, u, v) in enumerate(grids):
        co = [wx[torch.from_numpy(np.maximum(dof[j, a], 0)).to(dev)] * torch.from_numpy(sgn[j, a]).to(dev)
              for a in range(dof.shape[1])]
        cx = [z.to(torch.complex128) for z in (bp, dp, bq)]
        if scalar:
            D.append((cx[0] @ co[0] @ cx[0].T * area[j] * wt).ravel())
        else:
            c0, c1 = co[0][:m - 1, :m], co[1][:m, :m - 1]
            S.append(((cx[2] @ c0 @ cx[0].T * wt)[..., None] * u + (cx[0] @ c1 @ cx[2].T * wt)[..., None] * v)
                     .reshape(-1, 3))
            D.append(((cx[2] @ c0 @ cx[1].T + cx[1] @ c1 @ cx[2].T) * wt).ravel())
        X.append(F.reshape(-1, 3))
    X, D, S = torch.cat(X), torch.cat(D), torch.cat(S) if S else None
    out = torch.zeros((case["points"], 3), dtype=torch.complex128, device=dev)
    for i, pt in enumerate(torch.from_numpy(_points(case["points"], seed)).to(dev)):
        d = pt - X
        r = torch.linalg.norm(d, dim=1)
        G = torch.exp(1j * kappa * r) / (4 * math.pi * r)
        if scalar:
            out[i, 0] = torch.sum(G * D)
        else:
            grad = G * (1j * kappa * r - 1) / r ** 2 * D / kappa ** 2
            out[i] = torch.sum(G[:, None] * S + grad[:, None] * d, 0)
    return out.cpu().numpy()
