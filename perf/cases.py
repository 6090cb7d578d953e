"""Workloads by which the solver's speed is followed.

Every case is one pass of a program that uses the library: a forward solve
from rest that returns seismograms (a shot), a batch of shots in one context,
a restart (state in, one LTS cycle, state out), the plane-wave check run, or
a gradient of a seismogram misfit.  Meshes follow the repository's own
recipes: the layered box (100 / 200 / 300 m layers under 298.5 m columns,
jitter 15%), the graded basin and the periodic Kuhn cube; vertex ids and the
local vertex order of each tet are shuffled, as an unstructured mesher leaves
them.  Materials, sources, initial states and observed data come from the
seed.

`exact` solves the same discrete problem with plain torch in 64 bits (dense
reference matrices, closed-form Godunov flux, the B1/B2/B3 rules of clustered
rate-2 local time stepping); gradients come from torch's autograd.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

COLUMN = 20000.0 / 67          # column width of the layered box [m]
CFL = 0.5
BAND = (0.1, 10.0)             # attenuation band [Hz]
SAMPLES = 4.37                 # receiver samples per LTS cycle (never on a step boundary for long)


# --------------------------------------------------------------------------- the cases

def _case(kind, mesh, nx, ny, nz, order, mech, clusters, cycles, *, fp64=False, runs=1, sources=4, receivers=16,
          graph=False, remap=False, every=0):
    return dict(kind=kind, mesh=mesh, nx=nx, ny=ny, nz=nz, order=order, mech=mech, clusters=clusters, cycles=cycles,
                fp64=fp64, runs=runs, sources=sources, receivers=receivers, graph=graph, remap=remap, every=every)


def listed():
    return [
        # the convergence check every change of the scheme starts with: 1,296 tets, 50 global steps in FP64 of a
        # periodic plane wave, state in and out
        dict(_case("plane", "cube", 6, 6, 6, 3, 0, 1, 50, fp64=True, sources=0, receivers=0), name="plane_o3_fp64"),
        # the 5,082-tet box of the gradient checks as a plain shot: launches count
        dict(_case("shot", "layers", 11, 11, 7, 4, 3, 2, 20, sources=1, receivers=6, graph=True), name="shot_o4_5k"),
        # the small basin: five clusters (16 launches a cycle), a finite fault of Hann subfaults
        dict(_case("shot", "basin", 14, 14, 7, 5, 3, 5, 2, sources=64, receivers=16, graph=True), name="basin_o5_8k"),
        # an ordinary anelastic shot
        dict(_case("shot", "layers", 24, 24, 18, 5, 3, 3, 6, graph=True), name="shot_o5_62k"),
        # the 996,558-tet box of the headline benchmark
        dict(_case("shot", "layers", 67, 67, 37, 5, 3, 3, 2, receivers=64, graph=True, remap=True), name="shot_o5_1m"),
        # low order on a mesh of the gradient workload's size, elastic
        dict(_case("shot", "layers", 41, 41, 20, 3, 0, 2, 6, receivers=32), name="shot_o3_elastic_202k"),
        # an anelastic shot in FP64, as the accuracy of FP32 runs is checked
        dict(_case("shot", "layers", 13, 13, 11, 5, 3, 3, 3, fp64=True), name="shot_o5_fp64_11k"),
        # sixteen shots that share a mesh in one context
        dict(_case("batch", "layers", 16, 16, 12, 4, 3, 3, 3, runs=16, sources=1, graph=True), name="batch16_o4_18k"),
        # restart: a saved state goes in, one cycle, the state comes out
        dict(_case("restart", "layers", 9, 9, 8, 5, 3, 3, 1, sources=0, receivers=0), name="restart_o5_4k"),
        # an FP64 misfit gradient through torch.autograd, as gradient checks run it
        dict(_case("autograd", "layers", 11, 11, 7, 4, 0, 2, 4, fp64=True, sources=2, receivers=32, every=4),
             name="autograd_o4_fp64_5k"),
        # the elastic gradient workload: 201,720 tets, replayed segments
        dict(_case("gradient", "layers", 41, 41, 20, 4, 0, 2, 4, receivers=32, graph=True, every=2),
             name="gradient_o4_elastic_202k"),
        # the anelastic order-5 gradient, one recorded segment
        dict(_case("gradient", "layers", 24, 24, 18, 5, 3, 3, 2, receivers=32, graph=True, every=2),
             name="gradient_o5_62k"),
    ]


def _columns(rng, lo, hi):
    """Odd box shapes with about exp(U[log lo, log hi]) tets."""
    k = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    nz = rng.randint(5, 12 if k < 20000 else 30)
    nx = max(3, round(math.sqrt(k / (6 * nz)) * rng.uniform(0.8, 1.25)))
    ny = max(3, round(k / (6 * nz * nx)))
    return nx, ny, nz


def draw(rng):
    kind = rng.choice(["shot", "shot", "shot", "batch", "plane", "restart", "autograd", "gradient", "gradient"])
    mech = rng.choice([0, 3])
    if kind == "plane":
        n = rng.randint(4, 14)
        return _case(kind, "cube", n, n, n, rng.choice([2, 3, 4, 5]), 0, 1, rng.randint(10, 60),
                     fp64=rng.random() < 0.7, sources=0, receivers=0)
    if kind == "shot":
        if rng.random() < 0.2:
            n = rng.randint(10, 20)
            return _case(kind, "basin", n, n, max(5, n // 2), rng.choice([4, 5]), 3, rng.choice([4, 5]),
                         rng.randint(1, 3), sources=rng.randint(16, 100), receivers=rng.randint(4, 64), graph=True)
        fp64 = rng.random() < 0.25
        nx, ny, nz = _columns(rng, 1500, 20000 if fp64 else 250000)
        order = rng.choice([2, 3, 4, 5, 5])
        return _case(kind, "layers", nx, ny, nz, order, mech, rng.randint(1, 3), rng.randint(2, 6), fp64=fp64,
                     sources=rng.randint(1, 8), receivers=rng.randint(4, 64), graph=rng.random() < 0.5,
                     remap=rng.random() < 0.5)
    if kind == "batch":
        nx, ny, nz = _columns(rng, 1500, 15000)
        return _case(kind, "layers", nx, ny, nz, rng.choice([3, 4, 5]), mech, rng.randint(1, 3), rng.randint(2, 4),
                     runs=rng.randint(2, 20), sources=1, receivers=rng.randint(4, 32), graph=rng.random() < 0.5)
    if kind == "restart":
        nx, ny, nz = _columns(rng, 1000, 6000)
        return _case(kind, "layers", nx, ny, nz, rng.choice([3, 4, 5]), mech, rng.randint(1, 3), rng.randint(1, 3),
                     fp64=rng.random() < 0.3, sources=0, receivers=0)
    if kind == "autograd":
        nx, ny, nz = _columns(rng, 1000, 8000)
        return _case(kind, "layers", nx, ny, nz, rng.choice([3, 4]), mech, rng.randint(1, 2), rng.randint(2, 4),
                     fp64=rng.random() < 0.5, sources=2, receivers=rng.randint(4, 32), every=rng.randint(1, 4))
    order = rng.choice([3, 4, 5])
    nx, ny, nz = _columns(rng, 3000, 120000 if order < 5 or mech == 0 else 60000)
    return _case(kind, "layers", nx, ny, nz, order, mech, rng.randint(1, 3), rng.randint(2, 3), sources=4,
                 receivers=rng.randint(4, 32), graph=rng.random() < 0.5, every=rng.randint(1, 3))


# --------------------------------------------------------------------------- meshes and inputs

_KUHN = np.array([[0, 1, 3, 7], [0, 1, 5, 7], [0, 2, 3, 7], [0, 2, 6, 7], [0, 4, 5, 7], [0, 4, 6, 7]])


def _axis(n, h, s0, gmax, centred):
    u = (np.arange(n + 1) - (n / 2 if centred else 0)) * h
    return u * np.minimum(1.0 + np.abs(u) / s0, gmax)


def _axes(kind, nx, ny, nz):
    """Node coordinates per axis; the depth axis ascends to 0 at the surface."""
    if kind == "cube":
        return [np.linspace(0.0, 1000.0, n + 1) for n in (nx, ny, nz)]
    if kind == "basin":
        return [_axis(nx, 50.0, 40.0, 10.0, True), _axis(ny, 50.0, 40.0, 10.0, True),
                -_axis(nz, 50.0, 40.0, 10.0, False)[::-1]]
    dz = np.array(([100.0] * 4 + [200.0] * 3 + [300.0] * nz)[:nz])
    return [np.arange(nx + 1) * COLUMN, np.arange(ny + 1) * COLUMN,
            np.concatenate([[0.0], -np.cumsum(dz)])[::-1]]


@functools.lru_cache(maxsize=16)
def _mesh(kind, nx, ny, nz):
    """Kuhn-split hex grid: tet_verts [K,4], tet_xyz [K,4,3], face_bc [K,4]."""
    rng = np.random.default_rng(1000 * nx + 100 * ny + nz)
    n = np.array([nx, ny, nz])
    axes = _axes(kind, nx, ny, nz)
    corner = np.array([[c & 1, c >> 1 & 1, c >> 2 & 1] for c in range(8)])
    cube = np.stack(np.meshgrid(*[np.arange(m) for m in n], indexing="ij"), -1).reshape(-1, 3)
    lat = (cube[:, None, None, :] + corner[_KUHN]).reshape(-1, 4, 3)
    # local vertices in an arbitrary order per tet
    order = np.argsort(rng.random((len(lat), 4)), axis=1)
    lat = np.take_along_axis(lat, order[:, :, None], axis=1)
    xyz = np.stack([axes[d][lat[..., d]] for d in range(3)], -1)
    bc = np.zeros((len(lat), 4), dtype=np.int8)
    if kind == "cube":
        wrap = lat % n
        ids = (wrap[..., 0] * ny + wrap[..., 1]) * nz + wrap[..., 2]
    else:
        ids = (lat[..., 0] * (ny + 1) + lat[..., 1]) * (nz + 1) + lat[..., 2]
        grid = np.stack(np.meshgrid(*[np.arange(m + 1) for m in n], indexing="ij"), -1).reshape(-1, 3)
        move = rng.uniform(-0.15, 0.15, grid.shape)
        for d in range(3):
            gap = np.diff(axes[d])
            near = np.minimum(np.concatenate([[np.inf], gap]), np.concatenate([gap, [np.inf]]))
            move[:, d] *= near[grid[:, d]]
            move[(grid[:, d] == 0) | (grid[:, d] == n[d]), d] = 0.0
        xyz = xyz + move[ids]
        for i in range(4):       # free surface on top, absorbing elsewhere
            f = lat[:, [m for m in range(4) if m != i]]
            for d in range(3):
                bc[np.all(f[..., d] == 0, axis=1), i] = 2
                bc[np.all(f[..., d] == n[d], axis=1), i] = 1 if d == 2 else 2
    ids = rng.permutation(int(ids.max()) + 1)[ids]       # vertex numbers of no particular order
    return ids.astype(np.int64), xyz, bc


def _mesh_of(case):
    return _mesh(case["mesh"], case["nx"], case["ny"], case["nz"])


def _materials(case, seed):
    """rho, vp, vs by depth with a 2.5% perturbation, and constant-Q weights."""
    xyz = _mesh_of(case)[1]
    rng = np.random.default_rng([seed, 1])
    c = xyz.mean(axis=1)
    depth = -c[:, 2]
    if case["mesh"] == "cube":
        vs, ratio = np.full(len(c), 3464.0), 6000.0 / 3464.0
    elif case["mesh"] == "basin":
        e = np.sqrt((c[:, 0] / 400.0) ** 2 + (c[:, 1] / 300.0) ** 2 + (depth / 120.0) ** 2)
        vs = np.where(e < 1.0, 500.0 + 1000.0 * e ** 2, 1500.0 + 3000.0 * np.minimum(depth / 12000.0, 1.0) ** 0.6)
        ratio = np.clip(2.0 - 0.3 * (vs - 500.0) / 4000.0, 1.7, 2.0)
    else:
        steps = np.searchsorted([300.0, 600.0, 1000.0, 2000.0, 4000.0, 6000.0], depth, side="right")
        vs, ratio = np.array([800.0, 1000.0, 1400.0, 2000.0, 2600.0, 3200.0, 3500.0])[steps], 1.8
    if case["mesh"] != "cube":
        vs = vs * (1.0 + np.clip(rng.normal(0.0, 0.025, len(vs)), -0.05, 0.05))
    vp = ratio * vs
    rho = np.full(len(vs), 2700.0) if case["mesh"] == "cube" else 310.0 * vp ** 0.25
    m = case["mech"]
    if not m:
        return rho, vp, vs, None, None, None
    omega = 2 * math.pi * np.exp(np.linspace(*np.log(BAND), m))
    w = 2 * math.pi * np.exp(np.linspace(*np.log(BAND), 2 * m - 1))
    weights = []
    for q in (0.1 * vs, 0.05 * vs):     # Qp = 2 Qs, Qs = 50 vs [km/s]
        a = (omega * w[:, None] + omega ** 2 / q[:, None, None]) / (omega ** 2 + w[:, None] ** 2)
        at = a.transpose(0, 2, 1)
        weights.append(np.linalg.solve(at @ a, at.sum(-1, keepdims=True) / q[:, None, None])[..., 0])
    return rho, vp, vs, omega, weights[0], weights[1]


def _sources(case, seed, run):
    """Shallow moment-tensor sources: Ricker wavelets that start at once, or
    the Hann subfaults of a finite source in the basin."""
    rng = np.random.default_rng([seed, 2, run])
    n = case["sources"]
    xyz = _mesh_of(case)[1].reshape(-1, 3)
    lo, hi = xyz.min(axis=0), xyz.max(axis=0)
    p = lo + (hi - lo) * rng.uniform(0.2, 0.8, (n, 3))
    p[:, 2] = -rng.uniform(20.0, 150.0, n)
    moment = rng.normal(size=(n, 6))
    moment *= 1e15 / np.sqrt((np.sum(moment[:, :3] ** 2, 1) + 2 * np.sum(moment[:, 3:] ** 2, 1)) / 2)[:, None]
    if case["mesh"] == "basin":
        return p, moment / n, 1, np.stack([np.zeros(n), rng.uniform(0.05, 0.15, n)], 1)
    return p, moment, 0, np.stack([rng.uniform(4.0, 12.0, n), np.zeros(n)], 1)


def _receivers(case, seed):
    """Stations at the surface, a third of them (at least one) in boreholes
    beside the sources, where a short window already records."""
    rng = np.random.default_rng([seed, 3])
    xyz = _mesh_of(case)[1].reshape(-1, 3)
    lo, hi = xyz.min(axis=0), xyz.max(axis=0)
    p = lo + (hi - lo) * rng.uniform(0.1, 0.9, (case["receivers"], 3))
    p[:, 2] = 0.0
    near = np.concatenate([_sources(case, seed, r)[0] for r in range(case["runs"])])
    k = max(1, len(p) // 3)
    p[:k] = near[np.arange(k) % len(near)] + rng.uniform(-15.0, 15.0, (k, 3))
    return p


def _sampling(case, sync_dt):
    """Sample interval and number of samples of the window."""
    return sync_dt / SAMPLES, int(case["cycles"] * SAMPLES) + 1


def _initial(case, seed):
    """Modal DOFs: the plane P wave for the check run, otherwise amplitudes
    that fall off with the polynomial degree."""
    xyz = _mesh_of(case)[1]
    o = case["order"]
    rng = np.random.default_rng([seed, 4])
    t = _tables(o)
    if case["kind"] == "plane":
        wave = np.round(2 * (lambda v: v / np.linalg.norm(v))(rng.normal(size=3)))
        wave = wave if np.any(wave) else np.array([2.0, 0.0, 0.0])
        n = wave / np.linalg.norm(wave)
        rho, vp, vs = 2700.0, 6000.0, 3464.0
        s = -(rho * (vp * vp - 2 * vs * vs) * np.eye(3) + 2 * rho * vs * vs * np.outer(n, n)) / vp
        r = np.array([s[0, 0], s[1, 1], s[2, 2], s[0, 1], s[1, 2], s[0, 2], *n])
        pts, w = _tet_rule(o + 4)
        x = xyz[:, :1] + np.einsum("kcd,pc->kpd", xyz[:, 1:] - xyz[:, :1], pts)
        ph = np.sin(x @ (2 * math.pi / 1000.0 * wave) + rng.uniform(0.0, 2 * math.pi))
        return r[None, :, None] * ((ph * w) @ _phi(o, pts))[:, None, :]
    nq = 9 + 6 * case["mech"]
    scale = np.array([1e6] * 6 + [1.0] * 3 + [1e-3] * (nq - 9))
    deg = np.array([sum(i) for i in t["index"]])
    return rng.normal(size=(len(xyz), nq, len(deg))) * scale[:, None] * 3.0 ** -deg


def _observed(case, seed, n_rec, n_samples):
    """Recorded data a gradient compares with: velocities and stresses of the size a shot gives near its source."""
    rng = np.random.default_rng([seed, 5])
    d = np.cumsum(rng.normal(size=(n_rec, n_samples, 9)), axis=1)
    return d * np.array([1e5] * 6 + [0.05] * 3)


# --------------------------------------------------------------------------- the passes

def prepare(case, seed):
    from paper_2202_10313_amd import FLAG_GRAPH, Context
    verts, xyz, bc = _mesh_of(case)
    rho, vp, vs, omega, yp, ys = _materials(case, seed)
    ctx = Context(case["order"], mechanisms=case["mech"], n_clusters=case["clusters"], fp64=case["fp64"], cfl=CFL,
                  lam=1.0, n_runs=case["runs"], flags=FLAG_GRAPH if case["graph"] else 0)
    ctx.upload_mesh(verts, xyz, bc)
    ctx.upload_materials(rho, vp, vs, omega, yp, ys)
    ctx.upload_clusters(None)
    if case["remap"]:
        ctx.set_plan(xcd_remap=1)
    sync = ctx.get_clusters()["sync_dt"]
    s = dict(case=case, ctx=ctx, t=case["cycles"] * sync)
    if case["sources"]:
        for run in range(case["runs"]):
            p, moment, stf, par = _sources(case, seed, run)
            ctx.set_sources(p, moment, stf, par, run=run)
    if case["receivers"]:
        s["sample"], n = _sampling(case, sync)
        ctx.set_receivers(_receivers(case, seed), s["sample"], n)
    if case["kind"] in ("plane", "restart"):
        s["q0"] = _initial(case, seed)
    if case["kind"] in ("autograd", "gradient"):
        s["observed"] = torch.from_numpy(_observed(case, seed, ctx.n_rec, ctx.n_samples)).cuda()
    if case["kind"] == "autograd":
        from paper_2202_10313_amd.autograd import Simulation
        s["sim"] = Simulation(ctx, s["t"], omega, yp, ys, checkpoint_every=case["every"])
        s["model"] = [torch.from_numpy(a).cuda() for a in (rho, vp, vs)]
    return s


def run(s):
    """One pass; results of FP32 contexts are kept in FP32."""
    case, ctx = s["case"], s["ctx"]
    real = torch.float64 if case["fp64"] else torch.float32
    if case["kind"] in ("plane", "restart"):
        ctx.rewind()
        ctx.set_initial(s["q0"])
        ctx.advance_to(s["t"])
        return torch.from_numpy(ctx.read_dofs()).to(real)
    if case["kind"] in ("shot", "batch"):
        ctx.rewind()
        ctx.advance_to(s["t"])
        return torch.stack([ctx.read_receivers_device("cuda", run=r) for r in range(case["runs"])]).to(real)
    if case["kind"] == "autograd":
        model = [a.clone().requires_grad_() for a in s["model"]]
        seis = s["sim"].seismograms(*model)
        misfit = 0.5 * s["sample"] * ((seis - s["observed"]) ** 2).sum()
        misfit.backward()
        return dict(seis=seis.detach().to(real), **{k: a.grad.to(real) for k, a in zip(("rho", "vp", "vs"), model)})
    ctx.rewind()
    ctx.set_checkpointing(case["every"])
    ctx.advance_to(s["t"])
    seis = ctx.read_receivers_device("cuda")
    g = ctx.adjoint_device((seis - s["observed"]) * s["sample"])
    return dict(seis=seis.to(real), **{k: g["g_" + k].to(real) for k in ("rho", "vp", "vs")})


def work(case):
    """Per element update: the state read and written, the time integral of the
    elastic rows written and the neighbours' read once, 48 parameter words;
    the sparse operator products (the paper's 212,688 operations at order 5
    with three mechanisms, scaled by the entries of the matrices).  A gradient
    needs the forward and, per update, about twice that again."""
    o, m = case["order"], case["mech"]
    b, f = o * (o + 1) * (o + 2) // 6, o * (o + 1) // 2
    word = 8 if case["fp64"] else 4
    cl = _clustering(case, _materials(case, 0)[1])[0]
    per = 2 ** (case["clusters"] - 1)
    updates = case["cycles"] * case["runs"] * float(np.sum(per // 2 ** cl))
    nbytes = word * (2 * (9 + 6 * m) * b + 18 * b + 48)
    flops = 2 * (9 * o * (b * b / 3.4) + (15 if m else 9) * 4 * f * b * 0.36 + 36 * f * b * 0.36 + b * o * (60 + 60 * m))
    if case["kind"] in ("autograd", "gradient"):
        nbytes, flops = 3 * nbytes, 3 * flops
    state = 0 if case["kind"] not in ("plane", "restart") else 2 * 8 * len(cl) * (9 + 6 * m) * b
    return {"bytes": updates * nbytes + state, "flops": updates * flops}


# --------------------------------------------------------------------------- 64 bits

def _jacobi(n, a, x):
    """P_0..P_n^(a,0) at x."""
    p = [np.ones_like(x), ((a + 2) * x + a) / 2]
    for k in range(2, n + 1):
        c = 2 * k + a
        p.append((((c - 1) * (c * (c - 2) * x + a * a)) * p[-1] - 2 * (k + a - 1) * (k - 1) * c * p[-2])
                 / (2 * k * (k + a) * (c - 2)))
    return p


def _tet_rule(n):
    """Gauss points of the unit tetrahedron by collapsing a cube."""
    x, w = np.polynomial.legendre.leggauss(n + 2)
    x, w = (x + 1) / 2, w / 2
    r, s, t = (v.ravel() for v in np.meshgrid(x, x, x, indexing="ij"))
    wt = np.einsum("i,j,k->ijk", w, w, w).ravel() * (1 - s) * (1 - t) ** 2
    return np.stack([r * (1 - s) * (1 - t), s * (1 - t), t], 1), wt


def _tri_rule(n):
    x, w = np.polynomial.legendre.leggauss(n + 1)
    x, w = (x + 1) / 2, w / 2
    r, s = (v.ravel() for v in np.meshgrid(x, x, indexing="ij"))
    return np.stack([r * (1 - s), s], 1), np.outer(w, w).ravel() * (1 - s)


def _index(o):
    return [(i, j, n - i - j) for n in range(o) for i in range(n, -1, -1) for j in range(n - i, -1, -1)]


def _dubiner(o, p):
    """Unnormalised Dubiner functions at interior points p [P,3] -> [P,B]."""
    x, y, z = p.T
    a = 2 * x / (1 - y - z) - 1
    b = 2 * y / (1 - z) - 1
    c = 2 * z - 1
    pa = _jacobi(o, 0, a)
    return np.stack([pa[i] * ((1 - b) / 2) ** i * _jacobi(o, 2 * i + 1, b)[j] * ((1 - c) / 2) ** (i + j)
                     * _jacobi(o, 2 * i + 2 * j + 2, c)[k] for i, j, k in _index(o)], 1)


def _powers(o, p):
    return np.stack([p[:, 0] ** i * p[:, 1] ** j * p[:, 2] ** k for i, j, k in _index(o)], 1)


@functools.lru_cache(maxsize=None)
def _monomials(o):
    """Coefficients of the orthonormal basis in monomials: [monomial, b]."""
    pts, w = _tet_rule(o)
    v = _dubiner(o, pts)
    v = v / np.sqrt(w @ (v * v))
    return np.linalg.lstsq(_powers(o, pts), v, rcond=None)[0]


def _phi(o, p):
    return _powers(o, p) @ _monomials(o)


def _dphi(o, p):
    out = []
    for d in range(3):
        g = np.zeros((len(p), len(_index(o))))
        for c, e in enumerate(_index(o)):
            if e[d]:
                f = list(e)
                f[d] -= 1
                g[:, c] = e[d] * p[:, 0] ** f[0] * p[:, 1] ** f[1] * p[:, 2] ** f[2]
        out.append(g @ _monomials(o))
    return out


_CORNERS = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])


@functools.lru_cache(maxsize=None)
def _tables(o):
    """Stiffness matrices K_c[b, bb] = int phi_b d_c phi_bb and face projections
    onto an orthonormal face basis, faces spanned by their vertices in order."""
    pts, w = _tet_rule(o)
    phi = _phi(o, pts)
    stiff = np.stack([(w[:, None] * phi).T @ d for d in _dphi(o, pts)])
    fp, fw = _tri_rule(o)
    mono = np.stack([fp[:, 0] ** i * fp[:, 1] ** (n - i) for n in range(o) for i in range(n + 1)], 1)
    psi = np.linalg.qr(mono * np.sqrt(fw)[:, None])[0] / np.sqrt(fw)[:, None]
    bary = np.stack([1 - fp.sum(1), fp[:, 0], fp[:, 1]], 1)
    face = []
    for i in range(4):
        x = bary @ _CORNERS[[m for m in range(4) if m != i]]
        face.append(_phi(o, x).T @ (fw[:, None] * psi))
    return dict(index=_index(o), stiff=stiff, face=np.stack(face))


@functools.lru_cache(maxsize=16)
def _geometry(kind, nx, ny, nz):
    """Geometry and neighbours with every tet's vertices sorted by number."""
    verts, xyz, bc = _mesh(kind, nx, ny, nz)
    k = len(verts)
    perm = np.argsort(verts, axis=1)
    v = np.take_along_axis(verts, perm, 1)
    x = np.take_along_axis(xyz, perm[:, :, None], 1)
    bc = np.take_along_axis(bc, perm, 1).astype(np.int64)
    jac = (x[:, 1:] - x[:, :1]).transpose(0, 2, 1)
    det = np.abs(np.linalg.det(jac))
    normal, area = np.empty((k, 4, 3)), np.empty((k, 4))
    key = np.empty((k, 4), dtype=np.int64)
    top = int(v.max()) + 1
    for i in range(4):
        a, b, c = [m for m in range(4) if m != i]
        n = np.cross(x[:, b] - x[:, a], x[:, c] - x[:, a])
        n *= -np.sign(np.einsum("kd,kd->k", n, x[:, i] - x[:, a]))[:, None]
        area[:, i] = np.linalg.norm(n, axis=1) / 2
        normal[:, i] = n / (2 * area[:, i, None])
        key[:, i] = (v[:, a] * top + v[:, b]) * top + v[:, c]
    order = np.argsort(key.ravel(), kind="stable")
    same = np.nonzero(np.diff(key.ravel()[order]) == 0)[0]
    f, g = order[same], order[same + 1]
    nbr = np.full(4 * k, -1)
    nbr[f], nbr[g] = g, f
    return dict(perm=perm, x=x, bc=bc, det=det, inv=np.linalg.inv(jac), normal=normal, area=area,
                nbr=np.where(nbr < 0, -1, nbr // 4).reshape(k, 4), nface=(nbr % 4).reshape(k, 4))


def _clustering(case, vp):
    """Rate-2 clusters (0 = finest) at lambda = 1, and the finest step."""
    g = _geometry(case["mesh"], case["nx"], case["ny"], case["nz"])
    r = g["det"] / 2 / g["area"].sum(1)
    dt = CFL * 2 * r / ((2 * case["order"] - 1) * vp)
    cl = np.zeros(len(dt), dtype=np.int64)
    for l in range(1, case["clusters"]):
        cl[dt >= 2 ** l * dt.min()] = l
    while True:
        low = np.where(g["nbr"] >= 0, cl[g["nbr"]], 99).min(1) + 1
        if not np.any(low < cl):
            return cl, dt.min()
        cl = np.minimum(cl, low)


_VOIGT = ((0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (0, 2))


def _moment_rate(kind, par, t):
    """Integral of the moment rate up to t."""
    if kind == 0:
        tau = t - par[1]
        return tau * math.exp(-(math.pi * par[0] * tau) ** 2)
    tau = min(max(t - par[0], 0.0), par[1])
    return (tau - par[1] / (2 * math.pi) * math.sin(2 * math.pi * tau / par[1])) / par[1]


class _Solver:
    """The discrete scheme on one device in 64 bits, cluster by cluster."""

    def __init__(self, case, model, omega, yp, ys):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        dev = self.dev
        tt = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=dev)  # noqa: E731
        self.case, self.o, self.m = case, case["order"], case["mech"]
        g = self.g = _geometry(case["mesh"], case["nx"], case["ny"], case["nz"])
        self.cl, dt0 = _clustering(case, model[1])
        self.nc = case["clusters"]
        self.dt = [dt0 * 2 ** l for l in range(self.nc)]
        t = _tables(self.o)
        self.stiff, self.face = tt(t["stiff"]), tt(t["face"])
        self.model = [tt(a) for a in model]
        self.omega = omega
        self.weights = [tt(yp), tt(ys)] if self.m else None
        self.ids = [np.nonzero(self.cl == l)[0] for l in range(self.nc)]
        self.pos = np.empty(len(self.cl), dtype=np.int64)      # place within the cluster
        for i in self.ids:
            self.pos[i] = np.arange(len(i))
        self.at, self.jf, self.nb = [], [], []
        for l, ids in enumerate(self.ids):
            nb = g["nbr"][ids]
            inner = nb >= 0
            nb = np.where(inner, nb, ids[:, None])             # a boundary face sees its own element
            off = np.where(self.cl[nb] == l, 0, np.where(self.cl[nb] < l, len(ids),
                                                         len(ids) + (len(self.ids[l - 1]) if l else 0)))
            self.at.append(tt(off + self.pos[nb]))
            self.jf.append(tt(np.where(inner, g["nface"][ids], np.arange(4))))
            self.nb.append(tt(nb))
        self.inv = [tt(g["inv"][i]) for i in self.ids]
        self.normal = [tt(g["normal"][i]) for i in self.ids]
        self.scale = [tt(2 * g["area"][i] / g["det"][i, None]) for i in self.ids]
        self.bc = [tt(np.where(g["nbr"][i] >= 0, 0, g["bc"][i])) for i in self.ids]

    def parameters(self):
        """Moduli and impedances of the current model, per cluster."""
        rho, vp, vs = self.model
        mu = rho * vs * vs
        lam = rho * vp * vp - 2 * mu
        self.par = []
        for l, ids in enumerate(self.ids):
            i = torch.as_tensor(ids, device=self.dev)
            p = dict(lam=lam[i], mu=mu[i], rho=rho[i], zp=(rho * vp)[i], zs=(rho * vs)[i],
                     zpn=(rho * vp)[self.nb[l]], zsn=(rho * vs)[self.nb[l]])
            if self.m:
                y, z = (w[i] for w in self.weights)
                p["a"] = (lam + 2 * mu)[i, None] * y - 2 * mu[i, None] * z
                p["b"] = 2 * mu[i, None] * z
            self.par.append(p)

    def stress_velocity(self, grad, p):
        """(stress rate, velocity rate, strain rate) of physical gradients grad[d] = d_d q, q [n, 9, B]."""
        lam, mu, ir = (v[:, None] for v in (p["lam"], p["mu"], 1 / p["rho"]))
        eps = [0.5 * (grad[j][:, 6 + i] + grad[i][:, 6 + j]) for i, j in _VOIGT]
        div = eps[0] + eps[1] + eps[2]
        sig = [2 * mu * e + (lam * div if c < 3 else 0) for c, e in enumerate(eps)]
        vel = [ir * (grad[0][:, s[0]] + grad[1][:, s[1]] + grad[2][:, s[2]]) for s in ((0, 3, 5), (3, 1, 4), (5, 4, 2))]
        return sig, vel, eps

    def predict_part(self, l, q, inv, p, dts):
        """Time integrals over each of dts, the time derivatives of the elastic rows and the volume term over dts[0]."""
        d, deriv, integral = q, [], [0] * len(dts)
        om = self.omega
        for k in range(self.o):
            deriv.append(d[:, :9])
            integral = [s + h ** (k + 1) / math.factorial(k + 1) * (d if a == 0 else d[:, :9])
                        for a, (s, h) in enumerate(zip(integral, dts))]
            if k + 1 == self.o:
                break
            ref = [d[:, :9] @ self.stiff[c].T for c in range(3)]
            grad = [sum(inv[:, c, x, None, None] * ref[c] for c in range(3)) for x in range(3)]
            sig, vel, eps = self.stress_velocity(grad, p)
            d = self.relaxed(d, sig, vel, eps, p, om)
        t = integral[0]
        ref = [t[:, :9] @ self.stiff[c] for c in range(3)]
        grad = [sum(inv[:, c, x, None, None] * ref[c] for c in range(3)) for x in range(3)]
        sig, vel, eps = self.stress_velocity(grad, p)
        vol = self.relaxed(t, [-s for s in sig], [-v for v in vel], [-e for e in eps], p, om)
        return integral, deriv, vol

    def relaxed(self, d, sig, vel, eps, p, om):
        """Rows of the rate with the memory variables' part added."""
        if not self.m:
            return torch.stack(sig + vel, 1)
        mem = []
        sig = list(sig)
        for l in range(self.m):
            th = d[:, 9 + 6 * l:15 + 6 * l]
            tr = th[:, 0] + th[:, 1] + th[:, 2]
            for c in range(6):
                sig[c] = sig[c] - p["b"][:, l, None] * th[:, c] - (p["a"][:, l, None] * tr if c < 3 else 0)
                mem.append(om[l] * (eps[c] - th[:, c]))
        return torch.stack(sig + vel + mem, 1)

    def predict(self, l, step):
        n, size = len(self.ids[l]), 1 << 17
        dts = [self.dt[l], self.dt[l] / 2]
        parts = []
        keep = {r: [] for r in self.rec_of[l]}
        for a in range(0, max(n, 1), size):
            b = min(n, a + size)
            p = {k: v[a:b] for k, v in self.par[l].items()}
            integral, deriv, vol = self.predict_part(l, self.q[l][a:b], self.inv[l][a:b], p, dts)
            parts.append([vol] + [torch.stack([t[:, :9] @ self.face[i] for i in range(4)], 1) for t in integral])
            for r in keep:
                k = self.rec_pos[r]
                if a <= k < b:
                    keep[r] = [d[k - a] for d in deriv]
        self.vol[l], self.b1[l], self.b2[l] = (torch.cat(x) for x in zip(*parts))
        self.b3[l] = self.b1[l] if step % 2 == 0 else self.b3[l] + self.b1[l]
        t0, h = step * self.dt[l], self.dt[l]
        for r, d in keep.items():
            for s in range(self.ns):
                x = s * self.sample - t0
                if -1e-9 * h <= x < h - 1e-9 * h:
                    self.seis[(r, s)] = sum(x ** k / math.factorial(k) * (d[k] @ self.rec_phi[r])
                                            for k in range(self.o))

    def update(self, l, step):
        ids = self.ids[l]
        src = [self.b1[l]] + ([self.b3[l - 1]] if l else [])
        if l + 1 < self.nc:
            src.append(self.b2[l + 1] if step % 2 == 0 else self.b1[l + 1] - self.b2[l + 1])
        src = torch.cat(src)
        dq = []
        size = 1 << 17
        for a in range(0, max(len(ids), 1), size):
            b = min(len(ids), a + size)
            other = src[self.at[l][a:b], self.jf[l][a:b]]          # [n, 4, 9, F]
            dq.append(self.flux(l, self.b1[l][a:b], other, slice(a, b)))
        self.q[l] = self.q[l] + self.vol[l] + torch.cat(dq)
        for e, kind, par, moment, phi, det in self.src_of[l]:
            w = _moment_rate(kind, par, (step + 1) * self.dt[l]) - _moment_rate(kind, par, step * self.dt[l])
            inc = torch.zeros_like(self.q[l][:1])
            inc[0, :6] = -(w / det) * moment[:, None] * phi[None, :]
            self.q[l] = self.q[l].index_add(0, torch.tensor([e], device=self.dev), inc)

    def flux(self, l, own, other, part):
        """The surface term: one Godunov state per face mode, lifted."""
        n = self.normal[l][part][..., None, :, None]               # [k, 4, 1, 3, 1]
        p = {k: v[part] for k, v in self.par[l].items()}
        bc = self.bc[l][part][..., None, None]

        def state(q):
            s = [[q[:, :, c] for c in row] for row in ((0, 3, 5), (3, 1, 4), (5, 4, 2))]
            trac = torch.stack([sum(s[i][j] * n[:, :, 0, j] for j in range(3)) for i in range(3)], 2)
            return trac, q[:, :, 6:9]

        tm, vm = state(own)
        tp, vp = state(other)
        tp = torch.where(bc == 1, -tm, torch.where(bc == 2, torch.zeros_like(tp), tp))
        vp = torch.where(bc == 1, vm, torch.where(bc == 2, torch.zeros_like(vp), vp))
        n = n[:, :, 0]                                              # [k, 4, 3, 1]
        proj = lambda v: (v * n).sum(2, keepdim=True)               # noqa: E731
        zpm, zsm = p["zp"][:, None, None, None], p["zs"][:, None, None, None]
        zpp, zsp = p["zpn"][..., None, None], p["zsn"][..., None, None]

        def mixed(a, b, t1, v1, t2, v2):
            return (a * v1 + b * v2 + t2 - t1) / (a + b), (b * t1 + a * t2 + a * b * (v2 - v1)) / (a + b)

        tnm, vnm, tnp, vnp = proj(tm), proj(vm), proj(tp), proj(vp)
        vn, tn = mixed(zpm, zpp, tnm, vnm, tnp, vnp)
        vt, tt = mixed(zsm, zsp, tm - tnm * n, vm - vnm * n, tp - tnp * n, vp - vnp * n)
        v, t = vn * n + vt, tn * n + tt
        s = self.scale[l][part][..., None]
        rate = [0.5 * (n[:, :, i] * v[:, :, j] + n[:, :, j] * v[:, :, i]) * s for i, j in _VOIGT]
        lam, mu, ir = (x[:, None, None] for x in (p["lam"], p["mu"], 1 / p["rho"]))
        div = rate[0] + rate[1] + rate[2]
        rows = [2 * mu * e + (lam * div if c < 3 else 0) for c, e in enumerate(rate)]
        rows += [ir * t[:, :, i] * s for i in range(3)]
        lift = lambda r: sum(x[:, i] @ self.face[i].T for i in range(4) for x in (torch.stack(r, 2),))  # noqa: E731
        el = lift(rows)
        if not self.m:
            return el
        mem = lift(rate)
        return torch.cat([el] + [w * mem for w in self.omega], 1)

    def locate(self, pts):
        """(element, reference point in the sorted frame): the lowest element that covers each point."""
        x0 = torch.as_tensor(self.g["x"][:, 0], device=self.dev)
        inv = torch.as_tensor(self.g["inv"], device=self.dev)
        out = []
        for p in pts:
            xi = (inv @ (torch.as_tensor(p, device=self.dev) - x0)[:, :, None])[:, :, 0]
            k = int(torch.nonzero((xi.min(1).values >= -1e-10) & (xi.sum(1) <= 1 + 1e-10))[0, 0])
            out.append((k, xi[k].cpu().numpy()))
        return out

    def solve(self, q0, sources, receivers):
        dev, o = self.dev, self.o
        self.parameters()
        b = len(_index(o))
        nq = 9 + 6 * self.m
        self.q = [torch.zeros(len(i), nq, b, dtype=torch.float64, device=dev) if q0 is None else
                  torch.as_tensor(q0[i], device=dev) for i in self.ids]
        self.vol, self.b1, self.b2, self.b3 = ([None] * self.nc for _ in range(4))
        self.src_of = [[] for _ in self.ids]
        if sources is not None:
            pts, moment, kind, par = sources
            for (k, xi), mm, pp in zip(self.locate(pts), moment, par):
                self.src_of[self.cl[k]].append((int(self.pos[k]), kind, pp, torch.as_tensor(mm, device=dev),
                                                torch.as_tensor(_phi(o, xi[None])[0], device=dev), self.g["det"][k]))
        self.rec_of = [[] for _ in self.ids]
        self.rec_pos, self.rec_phi, self.seis = {}, {}, {}
        self.sample, self.ns = _sampling(self.case, self.dt[-1])
        if receivers is not None:
            for r, (k, xi) in enumerate(self.locate(receivers)):
                self.rec_of[self.cl[k]].append(r)
                self.rec_pos[r] = int(self.pos[k])
                self.rec_phi[r] = torch.as_tensor(_phi(o, xi[None])[0], device=dev)
        last = self.case["cycles"] * 2 ** (self.nc - 1)
        for l in range(self.nc):
            self.predict(l, 0)
        for j in range(1, last + 1):
            active = [l for l in range(self.nc) if j % 2 ** l == 0]
            for l in active:
                self.update(l, j // 2 ** l - 1)
            for l in active if j < last else []:
                self.predict(l, j // 2 ** l)
        if receivers is None:
            return None
        zero = torch.zeros(9, dtype=torch.float64, device=dev)
        return torch.stack([torch.stack([self.seis.get((r, s), zero) for s in range(self.ns)])
                            for r in range(len(receivers))])

    def vertex_matrices(self):
        """Per vertex order: the matrix from the caller's modes to the sorted frame's."""
        pts, w = _tet_rule(self.o)
        bary = np.concatenate([1 - pts.sum(1, keepdims=True), pts], 1)
        phi = w[:, None] * _phi(self.o, pts)
        perm = self.g["perm"]
        code = perm @ np.array([64, 16, 4, 1])
        for c in np.unique(code):
            k = np.nonzero(code == c)[0]
            own = np.empty_like(bary)
            own[:, perm[k[0]]] = bary
            yield k, phi.T @ _phi(self.o, own[:, 1:])

    def to_sorted(self, q):
        out = np.empty_like(q)
        for k, c in self.vertex_matrices():
            out[k] = q[k] @ c.T
        return out

    def to_caller(self):
        q = np.empty((len(self.cl),) + tuple(self.q[0].shape[1:]))
        for i, x in zip(self.ids, self.q):
            q[i] = x.cpu().numpy()
        out = np.empty_like(q)
        for k, c in self.vertex_matrices():
            out[k] = q[k] @ c
        return out


def exact(case, seed):
    rho, vp, vs, omega, yp, ys = _materials(case, seed)
    grad = case["kind"] in ("autograd", "gradient")
    s = _Solver(case, (rho, vp, vs), omega, yp, ys)
    if grad:        # the graph of every step stays in memory
        nq, b = 9 + 6 * case["mech"], len(_index(case["order"]))
        steps = case["cycles"] * float(np.sum(2 ** (case["clusters"] - 1) // 2 ** s.cl)) + len(s.cl)
        if steps * nq * b * 8 * case["order"] * 9 > (1.5e11 if s.dev == "cuda" else 1.5e10):
            return None
        s.model = [a.requires_grad_() for a in s.model]
    with torch.enable_grad() if grad else torch.no_grad():
        if case["kind"] in ("plane", "restart"):
            s.solve(s.to_sorted(_initial(case, seed)), None, None)
            return s.to_caller()
        rec = _receivers(case, seed)
        if not grad:
            return torch.stack([s.solve(None, _sources(case, seed, r), rec) for r in range(case["runs"])])
        seis = s.solve(None, _sources(case, seed, 0), rec)
        observed = torch.as_tensor(_observed(case, seed, len(rec), s.ns), device=s.dev)
        (0.5 * s.sample * ((seis - observed) ** 2).sum()).backward()
        return dict(seis=seis.detach(), **{k: a.grad for k, a in zip(("rho", "vp", "vs"), s.model)})
