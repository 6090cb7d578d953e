"""DOF conversion on the device (edg_set_initial, edg_read_dofs, the device
forms of edg_adjoint) against the host conversion of edg_set_dofs_subset /
edg_read_dofs_subset: same bits, for partly filled groups, every vertex order
and host arrays of more than one staging step."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _context(mesh, order, mech, fp64, n_clusters):
    from paper_2202_10313_amd import Context
    K = len(mesh["tet_verts"])
    mat = synth.random_materials(K, 4)
    ctx = Context(order, mechanisms=mech, n_clusters=n_clusters, fp64=fp64, lam=1.0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    a = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else {}
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *[a.get(k) for k in ("omega", "yp", "ys")])
    ctx.upload_clusters(None)
    return ctx


def _shuffled(mesh, seed):
    """The mesh with an arbitrary local vertex order per tet."""
    rng = np.random.default_rng(seed)
    o = np.argsort(rng.random(mesh["tet_verts"].shape), axis=1)
    return dict(tet_verts=np.take_along_axis(mesh["tet_verts"], o, 1),
                tet_xyz=np.take_along_axis(mesh["tet_xyz"], o[:, :, None], 1),
                face_bc=np.take_along_axis(mesh["face_bc"], o, 1))


@pytest.mark.parametrize("columns,order,mech,fp64", [(1, 2, 0, False), (2, 3, 3, True), (3, 4, 0, True),
                                                     (3, 5, 3, False), (11, 5, 3, False)])
def test_matches_host_conversion(columns, order, mech, fp64):
    dz = [100.0] * 4 + [200.0] * (9 if columns == 11 else 1)
    mesh = _shuffled(synth.layered_box(columns, columns, dz, 150.0 * columns, 150.0 * columns, jitter=0.1, seed=7), 8)
    ctx = _context(mesh, order, mech, fp64, 2)
    if columns == 11:      # two steps of the 64 MiB staging buffer
        assert ctx.K * ctx.nq * ctx.B * 8 > 64 << 20
    q = synth.random_state(9, ctx.K, ctx.nq, ctx.B)
    q[ctx.K // 2] = 0.0
    ids = np.arange(ctx.K)
    sync = ctx.get_clusters()["sync_dt"]
    out = []
    for whole in (True, False):
        ctx.rewind()
        if whole:
            ctx.set_initial(q)
        else:
            ctx.set_dofs_subset(ids, q)
        start = ctx.read_dofs_subset(ids)
        assert np.array_equal(start, ctx.read_dofs())
        ctx.advance_to(sync)        # the padding words, too, are as they were
        out.append((start, ctx.read_dofs()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    eps = 1e-13 if fp64 else 6e-7 * np.sqrt(ctx.B)     # two orthogonal products of B words each
    assert np.linalg.norm(out[0][0] - q) <= eps * np.linalg.norm(q)


def test_adjoint_device_dofs_equal_host_dofs():
    import torch
    mesh = _shuffled(synth.layered_box(2, 2, [100.0, 200.0], 400.0, 400.0, jitter=0.15, seed=3), 5)
    ctx = _context(mesh, 3, 3, True, 2)
    ctx.set_receivers(np.array([[150.0, 170.0, -20.0]]), 2e-3, 4)
    ctx.set_checkpointing(1)
    ctx.set_initial(synth.random_state(1, ctx.K, ctx.nq, ctx.B))
    ctx.advance_to(ctx.get_clusters()["sync_dt"])
    qb = np.random.default_rng(2).standard_normal((ctx.K, ctx.nq, ctx.B))
    sb = torch.zeros((1, 4, 9), dtype=torch.float64, device="cuda")
    h = ctx.adjoint(dj_dseis=sb.cpu().numpy(), dj_dq=qb)
    d = ctx.adjoint_device(sb, torch.from_numpy(qb).cuda(), want_q0=True)
    assert np.array_equal(h["q0_b"], d["q0_b"].cpu().numpy())
