"""Receivers whose samples do not fit: refused, and the context goes on without any."""
import numpy as np
import pytest

import synth
from tests.helpers import anelastic_setup

pytestmark = pytest.mark.gpu


# 1e13 samples of two receivers are more than any memory; 2^61 and more overflow their size in bytes
@pytest.mark.parametrize("samples", [10**13, 2**61, 2**63 - 1])
@pytest.mark.parametrize("flags", [0, 1])
def test_receivers_that_do_not_fit(samples, flags):
    from paper_2202_10313_amd import Context
    w = anelastic_setup("tiny", 3, 2)
    m, a = w["mesh"], w["attn"]
    K = m["tet_verts"].shape[0]
    q0 = synth.random_state(3, K, 27, 10)
    at = m["tet_xyz"].mean(1)
    ctx = Context(3, mechanisms=3, n_clusters=2, lam=1.0, flags=flags)
    ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
    ctx.upload_materials(*[w["mat"][k] for k in ("rho", "vp", "vs")], a["omega"], a["yp"], a["ys"])
    ctx.upload_clusters(None)
    sync = ctx.get_clusters()["sync_dt"]

    def run():
        ctx.rewind()
        ctx.set_initial(q0)
        ctx.advance_to(4 * sync)
        return ctx.read_dofs()
    want = run()
    ctx.set_receivers(at[:3], sync, 4)
    assert np.array_equal(run(), want)
    seen = ctx.read_receivers()
    with pytest.raises(RuntimeError):
        ctx.set_receivers(at[[5, K - 1]], sync, samples)
    assert np.array_equal(run(), want)
    ctx.set_receivers(at[:3], sync, 4)
    assert np.array_equal(run(), want) and np.array_equal(ctx.read_receivers(), seen) and np.any(seen)
    ctx.close()
