"""Sources and receivers of the levels and the level count of captured cycles: every combination of sources, receivers and runs, replayed
cycles with host reads in between against eager launches, bit for bit."""
import numpy as np
import pytest

import synth
from tests.helpers import anelastic_setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src,n_rec,runs", [(0, 0, 1), (0, 3, 2), (2, 0, 1), (3, 5, 3), (1, 4, 1)])
def test_replayed_cycles_equal_eager(n_src, n_rec, runs):
    from paper_2202_10313_amd import FLAG_GRAPH, Context
    w = anelastic_setup("tiny", 3, 2)
    m, a = w["mesh"], w["attn"]
    K = m["tet_verts"].shape[0]
    q0 = synth.random_state(3, K, 27, 10)
    box = m["box"]
    lo, hi = box[:, 0], box[:, 1]
    out = []
    for flags in (0, FLAG_GRAPH):
        ctx = Context(3, mechanisms=3, n_clusters=2, lam=1.0, n_runs=runs, flags=flags)
        ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
        ctx.upload_materials(w["mat"]["rho"], w["mat"]["vp"], w["mat"]["vs"], a["omega"], a["yp"], a["ys"])
        ctx.upload_clusters(None)
        sync = ctx.get_clusters()["sync_dt"]
        for r in range(runs):
            rng = np.random.default_rng(10 + r)
            ctx.set_initial(q0 * (1 + r), run=r)
            if n_src:
                ctx.set_sources(lo + (hi - lo) * rng.uniform(0.2, 0.8, (n_src, 3)), rng.normal(size=(n_src, 6)) * 1e12, 0,
                                np.tile([[20.0, 0.01]], (n_src, 1)), run=r)
        if n_rec:
            rng = np.random.default_rng(5)
            ctx.set_receivers(lo + (hi - lo) * rng.uniform(0.1, 0.9, (n_rec, 3)), sync / 3.3, 40)
        for cycles in (1, 4, 9):
            ctx.advance_to(cycles * sync)
            ctx.read_dofs(run=0)
        out.append([(ctx.read_dofs(run=r), ctx.read_receivers(run=r) if n_rec else 0) for r in range(runs)])
        assert ctx.time() == pytest.approx(9 * sync, rel=1e-14)
        ctx.close()
    for (qa, sa), (qb, sb) in zip(*out):
        assert np.array_equal(qa, qb) and np.array_equal(sa, sb)
    if n_rec:      # every sample of the window is written, and only those
        s = out[0][0][1]
        assert np.all(np.any(s[:, :29] != 0, axis=-1)) and not np.any(s[:, 30:])
