"""The reverse sweep of orders 4 and 5 on three explicit clusters: against the oracle's
discrete adjoint on a small mesh, and on one of many rounds of workgroups by the
dot-product identity (FP64) and against FP64 (FP32), with the bars of the other adjoint
tests."""
import numpy as np
import pytest

import synth
from oracle.adjoint import adjoint as oracle_adjoint
from tests.helpers import parity
from tests.test_gpu_adjoint import TOL64_G, TOL64_Q, _grad_err, _inputs, _oracle, _run_gpu, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [4, 5])
@pytest.mark.parametrize("mech", [0, 3])
@pytest.mark.parametrize("fp64", [True, False])
def test_three_clusters_match_oracle(order, mech, fp64):
    ctx, w = _setup(order, mech, 3, fp64, explicit=True)
    x, y, sb = _inputs(ctx, 70 + order + mech)
    t = 2 * w["sync"]
    qT, seis, res = _run_gpu(ctx, x, y, sb, t, 1)
    orc = _oracle(w)
    orc.set_initial(x)
    ores = oracle_adjoint(orc, t, seis_b=sb, q_b=y, attn=w["attn"])
    assert parity(res["q0_b"], ores["q0_b"]) <= (TOL64_Q if fp64 else 2e-5)
    assert _grad_err(res, ores) <= (TOL64_G if fp64 else 1e-4)
    ctx.close()


@pytest.mark.parametrize("order,mech", [(4, 0), (4, 3), (5, 0), (5, 3)])
def test_many_rounds_of_workgroups(order, mech):
    """12,096 elements: 1,728 groups in all and about 570 in each of the clusters, by depth."""
    from paper_2202_10313_amd import Context
    mesh = synth.layered_box(12, 12, [100.0] * 14, 1200.0, 1200.0, jitter=0.1, seed=3)
    K = mesh["tet_verts"].shape[0]
    mat = synth.random_materials(K, 4)
    attn = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else {}
    depth = -mesh["tet_xyz"].mean(1)[:, 2]
    cl = 1 + np.minimum((depth / 1400.0 * 3).astype(np.int32), 2)
    rng = np.random.default_rng(order + mech)
    out = {}
    for fp64 in (True, False):
        ctx = Context(order, mechanisms=mech, n_clusters=3, fp64=fp64, cfl=0.5 / 4, lam=1.0)
        ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
        ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *[attn.get(k) for k in ("omega", "yp", "ys")])
        ctx.upload_clusters(cl)
        sync = ctx.get_clusters()["sync_dt"]
        if fp64:
            x = synth.random_state(5, K, ctx.nq, ctx.B)
            y = rng.standard_normal((K, ctx.nq, ctx.B)) * np.where(np.arange(ctx.nq) < 6, 1e-6, 1.0)[None, :, None]
            sb = rng.standard_normal((20, 6, 9))
            rec = mesh["tet_xyz"][rng.integers(0, K, 20)].mean(1)
        ctx.set_receivers(rec, sync / 2.7, 6)
        ctx.set_checkpointing(1)
        ctx.set_initial(x)
        ctx.advance_to(2 * sync)
        qT, seis = ctx.read_dofs(), ctx.read_receivers()
        res = out[fp64] = ctx.adjoint(dj_dseis=sb, dj_dq=y)
        if fp64:
            lhs, rhs = np.sum(qT * y) + np.sum(seis * sb), np.sum(x * res["q0_b"])
            assert abs(lhs - rhs) <= 1e-12 * (np.sum(np.abs(qT * y)) + np.sum(np.abs(seis * sb)))
        ctx.close()
    assert parity(out[False]["q0_b"], out[True]["q0_b"]) <= 2e-5
    assert _grad_err(out[False], out[True]) <= 1e-4
