"""Receivers and sources beside the element groups of a level launch, at counts
around a wave, a workgroup and a row of eight workgroups: every receiver of a
crowded context samples what it samples alone, bit for bit (several in one
element, in every cluster); sources sharing an element add up to one source of
their summed moment, and each run has its own."""
import numpy as np
import pytest

import synth
from tests.helpers import anelastic_setup

pytestmark = pytest.mark.gpu


def _context(w, order, fp64, runs=1, graph=False):
    from paper_2202_10313_amd import FLAG_GRAPH, Context
    m, a = w["mesh"], w["attn"]
    ctx = Context(order, mechanisms=3, n_clusters=3, lam=1.0, fp64=fp64, n_runs=runs, flags=FLAG_GRAPH if graph else 0)
    ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
    ctx.upload_materials(w["mat"]["rho"], w["mat"]["vp"], w["mat"]["vs"], a["omega"], a["yp"], a["ys"])
    ctx.upload_clusters(None)
    return ctx


def _points(w, n, seed):
    lo, hi = w["mesh"]["box"][:, 0], w["mesh"]["box"][:, 1]
    x = lo + (hi - lo) * np.random.default_rng(seed).uniform(0.05, 0.95, (n, 3))
    x[1::3] = x[0::3][: len(x[1::3])]          # every third pair shares its element
    return x


@pytest.mark.parametrize("order,fp64,n", [(2, 0, 1), (3, 0, 17), (4, 0, 32), (5, 0, 33), (3, 1, 16), (5, 1, 130)])
def test_crowded_receivers_equal_single(order, fp64, n):
    w = anelastic_setup("tiny", order, 3)
    K, B = w["mesh"]["tet_verts"].shape[0], order * (order + 1) * (order + 2) // 6
    q0 = synth.random_state(3, K, 27, B)
    pts = _points(w, n, 4)
    pick = sorted({0, 1, n // 2, n - 1} & set(range(n)))

    def shot(xyz):
        ctx = _context(w, order, fp64)
        sync = ctx.get_clusters()["sync_dt"]
        ctx.set_initial(q0)
        ctx.set_sources(pts[:1], [[1e12] * 6], 0, [[20.0, 0.01]])
        ctx.set_receivers(xyz, sync / 7.3, 25)
        ctx.advance_to(2 * sync)
        ctx.advance_to(3 * sync)
        out = ctx.read_receivers()
        ctx.close()
        return out
    crowd = shot(pts)
    assert np.all(np.any(crowd[:, :21] != 0, axis=-1)) and not np.any(crowd[:, 22:])
    for i in pick:
        assert np.array_equal(crowd[i], shot(pts[i:i + 1])[0])


@pytest.mark.parametrize("order,fp64,n,graph", [(2, 0, 3, True), (4, 0, 33, False), (5, 0, 9, True), (4, 1, 70, True)])
def test_sources_of_an_element_add_up(order, fp64, n, graph):
    w = anelastic_setup("tiny", order, 3)
    rng = np.random.default_rng(2)
    x = _points(w, 2, 9)[0]
    other = _points(w, n, 11)
    mom = rng.uniform(0.5, 1.0, (n, 6)) * 1e12
    stf = [[20.0, 0.01]]

    def run(per_run):
        ctx = _context(w, order, fp64, runs=len(per_run), graph=graph)
        sync = ctx.get_clusters()["sync_dt"]
        for r, (xyz, mm) in enumerate(per_run):
            if len(xyz):
                ctx.set_sources(xyz, mm, 0, np.tile(stf, (len(xyz), 1)), run=r)
        ctx.advance_to(6 * sync)
        out = [ctx.read_dofs(run=r) for r in range(len(per_run))]
        ctx.close()
        return out
    many, none, far = run([(np.tile(x, (n, 1)), mom), (np.zeros((0, 3)), np.zeros((0, 6))), (other, mom)])
    one, = run([(x[None], mom.sum(0)[None])])
    far_alone, = run([(other, mom)])
    assert not np.any(none) and np.array_equal(far, far_alone)
    # n roundings per element and step against one
    tol = 4 * n * (2.0 ** -53 if fp64 else 2.0 ** -24)
    assert np.linalg.norm(many - one) <= tol * np.linalg.norm(one) and np.any(one)


@pytest.mark.parametrize("order", [3, 5])
def test_source_in_every_element_of_a_group(order):
    """A source in any element of a workgroup's seven: a step that finishes and
    predicts in one launch equals stopping in between, bit for bit."""
    w = anelastic_setup("tiny", order, 3)
    ctx = _context(w, order, 0)
    sync = ctx.get_clusters()["sync_dt"]
    mesh = w["mesh"]
    mid = mesh["tet_xyz"].mean(axis=1) if mesh["tet_xyz"].ndim == 3 else mesh["tet_xyz"][mesh["tet_verts"]].mean(axis=1)
    n = len(mid)
    ctx.set_sources(mid, np.ones((n, 6)) * 1e12, 0, np.tile([[20.0, 0.01]], (n, 1)))
    ctx.advance_to(3 * sync)
    whole = ctx.read_dofs()
    ctx.rewind()
    for k in (1, 2, 3):
        ctx.advance_to(k * sync)
    assert np.array_equal(whole, ctx.read_dofs()) and np.all(np.any(whole != 0, axis=(1, 2)))
    ctx.close()


@pytest.mark.parametrize("graph", [False, True])
def test_points_of_a_level_without_elements(graph):
    """No element in the finest cluster: the levels that only it would step in
    still sample and evaluate.  A sample at a synchronisation point is phi . Q
    there; a run that stops at each of them equals one that does not."""
    from paper_2202_10313_amd import FLAG_GRAPH, Context
    w = anelastic_setup("tiny", 3, 3)
    m = w["mesh"]
    K = m["tet_verts"].shape[0]
    ctx = Context(3, mechanisms=0, n_clusters=2, lam=0.6, fp64=True, flags=FLAG_GRAPH if graph else 0)
    ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
    ctx.upload_materials(w["mat"]["rho"], w["mat"]["vp"], w["mat"]["vs"])
    ctx.upload_clusters(np.full(K, 2))
    sync = ctx.get_clusters()["sync_dt"]
    pts = _points(w, 5, 3)
    src = (pts[:4], np.ones((4, 6)) * 1e12, 0, np.tile([[20.0, 0.01]], (4, 1)))

    def start(with_sources):
        ctx.rewind()
        ctx.set_sources(*src) if with_sources else ctx.set_sources(np.zeros((0, 3)), np.zeros((0, 6)), 0, np.zeros((0, 2)))
        ctx.set_receivers(pts, sync, 7)
    start(True)
    ctx.advance_to(6 * sync)
    whole, seis = ctx.read_dofs(), ctx.read_receivers()
    start(True)
    states = []
    for k in range(6):
        states.append(ctx.read_dofs())
        ctx.advance_to((k + 1) * sync)
    assert np.array_equal(whole, ctx.read_dofs()) and np.array_equal(seis, ctx.read_receivers())
    for k in (1, 2, 5):
        start(False)
        ctx.set_initial(states[k])
        ctx.advance_to(sync)
        assert np.linalg.norm(ctx.read_receivers()[:, 0] - seis[:, k]) <= 1e-12 * np.linalg.norm(seis[:, k]) != 0
    ctx.close()
