"""The one-launch reverse levels (transposed predictions and, of the same
elements, transposed updates) where their face slots are reused soonest: many
groups per launch, four explicit clusters, so that fine elements write a new
step's slot while a coarser neighbour reads two earlier ones.  Against the
oracle's discrete adjoint, with the bars of the other adjoint tests."""
import numpy as np
import pytest

import synth
from oracle.adjoint import adjoint as oracle_adjoint
from oracle.solver import Oracle
from tests.helpers import parity
from tests.test_gpu_adjoint import TOL64_G, TOL64_Q, _distance_clusters, _grad_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,mech,fp64,graph", [(2, 0, True, False), (3, 3, True, True), (3, 0, False, False)])
def test_four_clusters_match_oracle(order, mech, fp64, graph):
    from paper_2202_10313_amd import FLAG_GRAPH, Context
    mesh = synth.layered_box(5, 4, [100.0, 100.0, 200.0], 800.0, 700.0, jitter=0.1, seed=3)
    K = mesh["tet_verts"].shape[0]
    mat = synth.random_materials(K, 4)
    attn = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else None
    cl = _distance_clusters(Oracle(mesh, mat, 2).nbr, 4)
    ctx = Context(order, mechanisms=mech, n_clusters=4, fp64=fp64, cfl=0.5 / 8, lam=1.0,
                  flags=FLAG_GRAPH if graph else 0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *([attn[k] for k in ("omega", "yp", "ys")] if mech else []))
    ctx.upload_clusters(cl)
    info = ctx.get_clusters()
    assert len(np.unique(info["clusters"])) == 4
    rec = dict(xyz=np.array([[150.0, 170.0, -20.0], [560.0, 300.0, -150.0]]), dt_sample=info["sync_dt"] / 3.7,
               n_samples=8)
    rng = np.random.default_rng(order)
    x = synth.random_state(5, K, ctx.nq, ctx.B)
    y = rng.standard_normal((K, ctx.nq, ctx.B)) * np.where(np.arange(ctx.nq) < 6, 1e-6, 1.0)[None, :, None]
    sb = rng.standard_normal((2, 8, 9))
    t = 2 * info["sync_dt"]
    ctx.set_receivers(rec["xyz"], rec["dt_sample"], rec["n_samples"])
    ctx.set_checkpointing(1)
    ctx.set_initial(x)
    ctx.advance_to(t)
    res = ctx.adjoint(dj_dseis=sb, dj_dq=y)
    orc = Oracle(mesh, mat, order, attn=attn, receivers=rec, n_clusters=4, lam=info["lam"], clusters=info["clusters"],
                 dt_min=info["dt_min"])
    orc.set_initial(x)
    ores = oracle_adjoint(orc, t, seis_b=sb, q_b=y, attn=attn)
    assert parity(res["q0_b"], ores["q0_b"]) <= (TOL64_Q if fp64 else 2e-5)
    assert _grad_err(res, ores) <= (TOL64_G if fp64 else 1e-4)
