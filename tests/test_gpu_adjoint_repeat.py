"""A reverse sweep repeats bit for bit: the gradient words of an element come
from several waves and from the faces one by one, and several receivers of one
element add to the same derivatives."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [2, 3, 4, 5])
@pytest.mark.parametrize("mech,fp64", [(0, True), (3, True), (0, False), (3, False)])
def test_sweeps_repeat(order, mech, fp64):
    from paper_2202_10313_amd import Context
    mesh = synth.layered_box(5, 5, [100.0, 100.0, 200.0], 800.0, 800.0, jitter=0.15, seed=3)
    K = mesh["tet_verts"].shape[0]
    mat = synth.random_materials(K, 4)
    attn = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else None
    ctx = Context(order, mechanisms=mech, n_clusters=2, fp64=fp64, cfl=0.5, lam=1.0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *([attn[k] for k in ("omega", "yp", "ys")] if mech else []))
    ctx.upload_clusters(None)
    sync = ctx.get_clusters()["sync_dt"]
    rng = np.random.default_rng(order)
    w = rng.dirichlet(np.ones(4), 12)
    ctx.set_receivers(np.einsum("rv,rvd->rd", w, mesh["tet_xyz"][[7, 7, 90, 7, 90, 7, 200, 201, 7, 90, 7, 300]]),
                      sync / 4.3, 9)
    ctx.set_checkpointing(2)
    ctx.set_initial(synth.random_state(5, K, ctx.nq, ctx.B))
    ctx.advance_to(2 * sync)
    sb = rng.standard_normal((12, 9, 9))
    first = ctx.adjoint(dj_dseis=sb)
    assert np.any(first["g_rho"])
    for _ in range(8):
        again = ctx.adjoint(dj_dseis=sb)
        for k in first:
            assert np.array_equal(first[k], again[k]), k
    ctx.close()
