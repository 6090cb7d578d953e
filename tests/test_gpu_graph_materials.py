"""A captured cycle after new materials: other relaxation frequencies reach it."""
import numpy as np
import pytest

import synth
from tests.helpers import anelastic_setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("device", [False, True])
def test_frequencies_uploaded_after_a_capture(device):
    """Advances of five cycles, each on materials of its own frequencies: replayed cycles
    leave the DOFs that launches one by one leave."""
    import torch

    from paper_2202_10313_amd import FLAG_GRAPH, Context
    w = anelastic_setup("tiny", 3, 2)
    m, a = w["mesh"], w["attn"]
    q0 = synth.random_state(3, m["tet_verts"].shape[0], 27, 10)
    out = []
    for flags in (0, FLAG_GRAPH):
        ctx = Context(3, mechanisms=3, n_clusters=2, lam=1.0, flags=flags)
        ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
        states = []
        for scale in (1.0, 2.0, 2.0, 1.0):
            args = [w["mat"][k] for k in ("rho", "vp", "vs")] + [scale * np.asarray(a["omega"]), a["yp"], a["ys"]]
            if device and states:      # (clusters need materials first, from either side)
                args = [torch.tensor(np.asarray(x), dtype=torch.float64, device="cuda") for x in args]
            ctx.upload_materials(*args)
            if not states:
                ctx.upload_clusters(None)
                sync = ctx.get_clusters()["sync_dt"]
            ctx.rewind()
            ctx.set_initial(q0)
            ctx.advance_to(5 * sync)
            states.append(ctx.read_dofs())
        out.append(states)
        ctx.close()
    assert not np.array_equal(out[0][0], out[0][1])
    for x, y in zip(*out):
        assert np.array_equal(x, y)
