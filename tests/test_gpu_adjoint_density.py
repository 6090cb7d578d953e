"""dJ/drho where its terms cancel.  An advance of two steps from rest moves only
in its second step, and only in the elements with a source: there the recorded
stresses do not depend on rho at fixed vp and vs (lam/rho, mu/rho and the
anelastic moduli over rho are fixed) and the recorded velocities are
proportional to 1/rho.  So the exact gradient is known,

  dJ/drho_k = -1/rho_k sum of (recorded velocity) * (its adjoint), receivers in k,

while its parts through 1/rho and through the moduli are each about 1e12 times
larger (stress samples of the sources' size, weighted alike).  Each value is a
sum of a few hundred products, each rounded: 300 half units in the last place.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [2, 3, 4, 5])
@pytest.mark.parametrize("mech", [0, 3])
@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("n_clusters", [1, 2])
def test_two_steps_from_rest(order, mech, fp64, n_clusters):
    from paper_2202_10313_amd import Context
    mesh = synth.layered_box(3, 3, [100.0, 100.0, 200.0], 600.0, 600.0, jitter=0.15, seed=3)
    K = mesh["tet_verts"].shape[0]
    mat = synth.random_materials(K, 4)
    attn = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else None
    ctx = Context(order, mechanisms=mech, n_clusters=n_clusters, fp64=fp64, cfl=0.5 / n_clusters, lam=1.0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *([attn[k] for k in ("omega", "yp", "ys")] if mech else []))
    # with two clusters one element is fine, far from the sources (which take two coarse steps)
    ctx.upload_clusters(None if n_clusters == 1 else np.where(np.arange(K) == 0, 1, 2).astype(np.int32))
    sync = ctx.get_clusters()["sync_dt"]
    at = [40, K // 2, K - 9]
    rng = np.random.default_rng(1)
    ctx.set_sources([mesh["tet_xyz"][k].mean(0) for k in at], rng.normal(size=(3, 6)) * 1e12, 0,
                    np.tile([[8.0, 0.0]], (3, 1)))
    ctx.set_receivers([np.array([0.4, 0.3, 0.2, 0.1]) @ mesh["tet_xyz"][k] for k in at], sync / 4.3, 8)
    ctx.set_checkpointing(2)
    ctx.advance_to(2 * sync)
    seis = ctx.read_receivers()
    sb = rng.normal(size=seis.shape) * np.array([1e5] * 6 + [0.05] * 3)
    got = ctx.adjoint(dj_dseis=sb)["g_rho"]
    ctx.close()
    want = np.zeros(K)
    for r, k in enumerate(at):
        want[k] = -np.sum(sb[r, :, 6:] * seis[r, :, 6:]) / mat["rho"][k]
    assert np.min(np.abs(want[at])) > 0
    assert np.linalg.norm(got - want) <= 300 * np.finfo(np.float64 if fp64 else np.float32).eps / 2 * np.linalg.norm(want)
