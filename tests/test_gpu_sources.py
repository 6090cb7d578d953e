"""Many sources in few elements: their sum, in one and in several runs, when the
list of a run changes or empties, and the time that they take."""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _context(columns, order, mech, fp64, runs, n_clusters=2):
    from paper_2202_10313_amd import Context
    mesh = synth.layered_box(columns, columns, [100.0, 100.0, 200.0], 150.0 * columns, 150.0 * columns, jitter=0.1,
                             seed=3)
    K = mesh["tet_verts"].shape[0]
    mat = synth.random_materials(K, 4)
    a = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else {}
    ctx = Context(order, mechanisms=mech, n_clusters=n_clusters, fp64=fp64, n_runs=runs, lam=1.0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *[a.get(k) for k in ("omega", "yp", "ys")])
    ctx.upload_clusters(None)
    return ctx, mesh


# 63, 64, 65 and 130 sources: a wave evaluates up to 64 at a time
@pytest.mark.parametrize("order,mech,fp64", [(2, 0, True), (3, 3, False), (5, 0, True)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 130])
def test_sources_of_an_element_add_up(order, mech, fp64, n):
    """n sources at one point of each of three elements (two of them in one group)
    equal one source with the summed moment there."""
    ctx, mesh = _context(3, order, mech, fp64, 3)
    sync = ctx.get_clusters()["sync_dt"]
    rng = np.random.default_rng(n)
    at = [mesh["tet_xyz"][k].mean(0) for k in (11, 12, 90)]
    out = []
    for many in (True, False):
        for run in range(3):
            rng = np.random.default_rng([n, run])
            m = rng.uniform(0.5, 1.5, size=(3, n, 6)) * 1e9
            order_of = rng.permutation(3 * n)
            if many:
                xyz, mom = np.repeat(at, n, axis=0)[order_of], m.reshape(-1, 6)[order_of]
            else:
                xyz, mom = at, m.sum(1)
            ctx.set_sources(xyz, mom, 1, np.tile([[0.0, 3 * sync]], (len(xyz), 1)), run=run)
        ctx.rewind()
        ctx.advance_to(2 * sync)
        out.append([ctx.read_dofs(run=r) for r in range(3)])
    eps = np.finfo(np.float64 if fp64 else np.float32).eps
    for x, y in zip(*out):
        for rows in (slice(0, 6), slice(6, 9)):
            assert 0 < np.linalg.norm(y[:, rows])
            assert np.linalg.norm(x[:, rows] - y[:, rows]) <= 200 * eps * np.linalg.norm(y[:, rows])
    ctx.close()


def test_lists_of_runs_change():
    """A run's sources replaced, moved and emptied leave what a context gives that
    only ever had the last lists."""
    def lists(mesh, k):
        rng = np.random.default_rng(k)
        n = int(rng.integers(1, 9))
        ids = rng.integers(0, len(mesh["tet_xyz"]), n)
        return np.array([mesh["tet_xyz"][i].mean(0) for i in ids]), rng.normal(size=(n, 6)) * 1e9

    final = {0: 3, 1: None, 2: 7}
    out = []
    for history in (((0, 1), (1, 2), (2, 4), (0, 5), (2, None), (1, None), (0, None), (0, 3), (2, 7)), ((2, 7), (0, 3))):
        ctx, mesh = _context(3, 2, 0, True, 3)
        sync = ctx.get_clusters()["sync_dt"]
        for run, k in history:
            xyz, mom = (np.zeros((0, 3)), np.zeros((0, 6))) if k is None else lists(mesh, k)
            ctx.set_sources(xyz, mom, 1, np.tile([[0.0, 3 * sync]], (len(xyz), 1)), run=run)
        ctx.advance_to(2 * sync)
        out.append([ctx.read_dofs(run=r) for r in range(3)])
        ctx.close()
    for r in range(3):
        assert np.array_equal(out[0][r], out[1][r]) and np.any(out[0][r]) == (final[r] is not None)


def _best(f, n=7):
    t = []
    for _ in range(n):
        a = time.perf_counter()
        f()
        t.append(time.perf_counter() - a)
    return min(t)


def test_a_crowded_element_does_not_hold_up_the_level():
    """1,024 sources in one element against one in each of 1,024: the launch that
    adds them takes a sum that is formed beside the launch before (a loop over them
    in the element's own workgroup takes about a microsecond each)."""
    ctx, mesh = _context(8, 4, 0, False, 1, n_clusters=1)
    sync = ctx.get_clusters()["sync_dt"]
    K = len(mesh["tet_xyz"])
    assert K >= 1024
    took = []
    for ids in (np.arange(1024), np.full(1024, 500)):
        w = np.random.default_rng(1).dirichlet(np.full(4, 3.0), 1024)
        ctx.set_sources(np.einsum("sv,svd->sd", w, mesh["tet_xyz"][ids]), np.full((1024, 6), 1e6), 0,
                        np.tile([[8.0, 0.0]], (1024, 1)))

        def run():
            ctx.rewind()
            ctx.advance_to(20 * sync)
        run()
        took.append(_best(run))
    ctx.close()
    print(f"[sources] 20 steps: spread {took[0] * 1e6:.0f} us, one element {took[1] * 1e6:.0f} us", flush=True)
    assert took[1] <= 8 * took[0]


def test_setting_the_sources_of_a_run_costs_its_sources():
    """One source set in a context of 32 runs on 96k tets against one in a context
    of one run: the cost is that of the sources, not of the groups of all runs."""
    took = []
    for runs in (1, 32):
        ctx, mesh = _context(73, 2, 0, False, runs, n_clusters=1)
        xyz = [mesh["tet_xyz"][700].mean(0)]

        def set_one():
            ctx.set_sources(xyz, np.ones((1, 6)), 0, [[8.0, 0.0]], run=runs - 1)
        set_one()
        took.append(_best(set_one))
        ctx.close()
    print(f"[sources] set one: 1 run {took[0] * 1e6:.0f} us, 32 runs {took[1] * 1e6:.0f} us", flush=True)
    assert took[1] <= 3 * took[0]
