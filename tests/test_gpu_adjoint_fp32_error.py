"""Rounding of FP32 material gradients: the geometric mean, over eight sets of
inputs and the three gradients, of the relative L2 distance from an FP64 context.
FP32 products are summed in FP64, mode by mode and row by row; the bars are 1.15
times what the first kernels with such sums gave on these inputs."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

BARS = {(2, 0): 1.15 * 6.64e-8, (2, 3): 1.15 * 5.99e-8, (3, 0): 1.15 * 7.22e-8, (3, 3): 1.15 * 7.02e-8}


def _gradients(order, mech, fp64, seed):
    from paper_2202_10313_amd import Context
    mesh = synth.layered_box(4, 4, [100.0, 100.0, 200.0], 700.0, 700.0, jitter=0.15, seed=3)
    K = mesh["tet_verts"].shape[0]
    mat = synth.random_materials(K, seed)
    attn = synth.attenuation_inputs(mat, mech, 0.1, 10.0) if mech else None
    ctx = Context(order, mechanisms=mech, n_clusters=1, fp64=fp64, cfl=0.5, lam=1.0)
    ctx.upload_mesh(mesh["tet_verts"], mesh["tet_xyz"], mesh["face_bc"])
    ctx.upload_materials(mat["rho"], mat["vp"], mat["vs"], *([attn[k] for k in ("omega", "yp", "ys")] if mech else []))
    ctx.upload_clusters(None)
    sync = ctx.get_clusters()["sync_dt"]
    rng = np.random.default_rng(seed)
    at = rng.integers(0, K, 4)
    xyz = np.array([mesh["tet_xyz"][k].mean(0) for k in at])
    ctx.set_sources(xyz, rng.normal(size=(4, 6)) * 1e12, 0, np.tile([[8.0, 0.0]], (4, 1)))
    ctx.set_receivers(np.array([np.array([0.4, 0.3, 0.2, 0.1]) @ mesh["tet_xyz"][k] for k in at]), sync / 4.3, 14)
    ctx.set_checkpointing(3)
    ctx.advance_to(3 * sync)
    sb = np.cumsum(rng.normal(size=(4, 14, 9)), axis=1) * np.array([1e5] * 6 + [0.05] * 3)
    g = ctx.adjoint(dj_dseis=sb)
    ctx.close()
    return [g[k] for k in ("g_rho", "g_vp", "g_vs")]


@pytest.mark.parametrize("order,mech", list(BARS))
def test_rounding_of_fp32_gradients(order, mech):
    err = []
    for seed in range(1, 9):
        a, b = (_gradients(order, mech, fp64, seed) for fp64 in (False, True))
        err += [np.linalg.norm(x - y) / np.linalg.norm(y) for x, y in zip(a, b)]
    mean = float(np.exp(np.mean(np.log(err))))
    print(f"[fp32 gradients] O={order} m={mech}: {mean:.2e}", flush=True)
    assert mean <= BARS[order, mech]
