"""Device DOF arrays of more elements than one conversion launch takes (a launch
has fewer than 2^32 threads): the arrays of edg_adjoint on the device and on the
host give the same bits, first and last elements included."""
import numpy as np
import pytest

import synth
from tests.test_gpu_layout import _context, _shuffled

pytestmark = pytest.mark.gpu


def test_more_elements_than_one_launch():
    import torch
    mesh = _shuffled(synth.layered_box(68, 68, [100.0] * 10, 10000.0, 10000.0, jitter=0.1, seed=7), 8)
    ctx = _context(mesh, 2, 0, False, 1)
    assert ctx.K > 1 << 18
    ctx.set_receivers(np.array([[150.0, 170.0, -20.0]]), 2e-3, 4)
    ctx.set_checkpointing(1)
    ctx.set_initial(synth.random_state(1, ctx.K, ctx.nq, ctx.B))
    ctx.advance_to(ctx.get_clusters()["sync_dt"])
    qb = np.random.default_rng(2).standard_normal((ctx.K, ctx.nq, ctx.B))
    sb = torch.zeros((1, 4, 9), dtype=torch.float64, device="cuda")
    h = ctx.adjoint(dj_dseis=sb.cpu().numpy(), dj_dq=qb)
    d = ctx.adjoint_device(sb, torch.from_numpy(qb).cuda(), want_q0=True)
    assert np.array_equal(h["q0_b"], d["q0_b"].cpu().numpy())
    assert np.all(np.any(h["q0_b"], axis=(1, 2)))
    for k in ("g_rho", "g_vp", "g_vs"):
        assert np.array_equal(h[k], d[k].cpu().numpy())
    ctx.close()
