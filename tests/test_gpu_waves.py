"""The element update's wave splits at the smallest meshes of every order and
at launches of many rounds, against the FP64 update of the same mesh (which
the oracle pins): the FP32 parity bar, 2e-5 relative per quantity group.
Launches of different size round alike: runs of a batch equal the single run."""
import numpy as np
import pytest

import synth
from tests.helpers import parity

pytestmark = pytest.mark.gpu


def _advance(mesh, mat, attn, order, fp64, q, cycles):
    from paper_2202_10313_amd import Context
    mech = 0 if attn is None else 3
    ctx = Context(order, mechanisms=mech, n_clusters=2, fp64=fp64, lam=1.0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *([] if attn is None else [attn[k] for k in ("omega", "yp", "ys")]))
    ctx.upload_clusters(None)
    ctx.set_initial(q)
    ctx.advance_to(cycles * ctx.get_clusters()["sync_dt"])
    out = ctx.read_dofs()
    ctx.close()
    return out


@pytest.mark.parametrize("columns,layers,order,mech", [((27, 28), 25, 4, 3), ((28, 28), 25, 4, 0), ((19, 13), 11, 5, 3),
                                                       ((1, 1), 2, 2, 3), ((1, 1), 2, 3, 3), ((1, 1), 2, 5, 0)])
def test_fp32_split_matches_fp64(columns, layers, order, mech):
    mesh = synth.layered_box(columns[0], columns[1], [100.0] * (layers // 2) + [200.0] * (layers - layers // 2),
                             150.0 * columns[0], 150.0 * columns[1], jitter=0.1, seed=11)
    K = len(mesh["tet_verts"])
    mat = synth.random_materials(K, 12)
    attn = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else None
    q = synth.random_state(13, K, 9 + 6 * mech, order * (order + 1) * (order + 2) // 6)
    a = _advance(mesh, mat, attn, order, False, q, 1)
    b = _advance(mesh, mat, attn, order, True, q, 1)
    assert parity(a, b) <= 2e-5


def test_batch_equals_single_run():
    """9 runs of 2,016 groups in one launch."""
    from paper_2202_10313_amd import Context
    mesh = synth.layered_box(14, 14, [100.0] * 4 + [200.0] * 8, 2100.0, 2100.0, jitter=0.1, seed=11)
    K = len(mesh["tet_verts"])
    mat = synth.random_materials(K, 12)
    attn = synth.attenuation_inputs(mat, 3, 0.1, 10.0)
    q = synth.random_state(13, K, 27, 20)
    out = []
    for runs in (1, 9):
        ctx = Context(4, mechanisms=3, n_clusters=1, lam=1.0, n_runs=runs)
        ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
        ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], attn["omega"], attn["yp"], attn["ys"])
        ctx.upload_clusters(None)
        ctx.set_initial(q, run=runs - 1)
        ctx.advance_to(3 * ctx.get_clusters()["sync_dt"])
        out.append(ctx.read_dofs(run=runs - 1))
        ctx.close()
    assert np.array_equal(out[0], out[1])
