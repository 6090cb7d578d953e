"""A rewound context repeats its first run bit for bit, whatever the run before
left in its face buffers (here infinities and NaN); a Simulation at rest equals
one given zeros."""
import numpy as np
import pytest

import synth
from tests.helpers import anelastic_setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64,order,flags", [(0, 2, 0), (0, 5, 1), (1, 3, 0), (1, 4, 1)])
def test_rewound_run_equals_the_first(fp64, order, flags):
    from paper_2202_10313_amd import FLAG_GRAPH, Context
    w = anelastic_setup("tiny", order, 2)
    m, a = w["mesh"], w["attn"]
    B = order * (order + 1) * (order + 2) // 6
    q0 = synth.random_state(3, m["tet_verts"].shape[0], 27, B)
    lo, hi = m["box"][:, 0], m["box"][:, 1]
    ctx = Context(order, mechanisms=3, n_clusters=2, lam=1.0, fp64=fp64, flags=FLAG_GRAPH if flags else 0)
    ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
    ctx.upload_materials(w["mat"]["rho"], w["mat"]["vp"], w["mat"]["vs"], a["omega"], a["yp"], a["ys"])
    ctx.upload_clusters(None)
    sync = ctx.get_clusters()["sync_dt"]
    rng = np.random.default_rng(1)
    ctx.set_sources(lo + (hi - lo) * rng.uniform(0.2, 0.8, (2, 3)), rng.normal(size=(2, 6)) * 1e12, 0,
                    np.tile([[20.0, 0.01]], (2, 1)))
    ctx.set_receivers(lo + (hi - lo) * rng.uniform(0.1, 0.9, (3, 3)), sync / 3.3, 20)
    out = []
    for bad in (None, np.inf, np.nan):
        if bad is not None:
            ctx.set_initial(np.full_like(q0, bad))
            ctx.advance_to(ctx.time() + 2 * sync)
            ctx.rewind()
            assert ctx.time() == 0 and not np.any(ctx.read_dofs()) and not np.any(ctx.read_receivers())
        runs = []
        for x in (None, q0):             # at rest (sources only), then from a state
            if x is not None:
                ctx.rewind()
                ctx.set_initial(x)
            ctx.advance_to(3 * sync)
            runs += [ctx.read_dofs(), ctx.read_receivers()]
        ctx.rewind()
        out.append(runs)
    ctx.close()
    for runs in out[1:]:
        assert all(np.array_equal(x, y) and np.all(np.isfinite(x)) for x, y in zip(out[0], runs))


def test_simulation_at_rest_equals_zeros():
    import torch
    from paper_2202_10313_amd import Context
    from paper_2202_10313_amd.autograd import Simulation
    w = anelastic_setup("tiny", 2, 2)
    m, a = w["mesh"], w["attn"]
    lo, hi = m["box"][:, 0], m["box"][:, 1]
    ctx = Context(2, mechanisms=3, n_clusters=2, lam=1.0, fp64=True)
    ctx.upload_mesh(m["tet_verts"], m["tet_xyz"], m["face_bc"])
    ctx.upload_materials(w["mat"]["rho"], w["mat"]["vp"], w["mat"]["vs"], a["omega"], a["yp"], a["ys"])
    ctx.upload_clusters(None)
    sync = ctx.get_clusters()["sync_dt"]
    ctx.set_sources([(lo + hi) / 2], [[1e12, 1e12, 1e12, 0, 0, 0]], 0, [[20.0, 0.01]])
    ctx.set_receivers([lo + (hi - lo) * 0.4], sync / 4, 12)
    zeros = np.zeros((ctx.K, ctx.nq, ctx.B))
    rest, given = (Simulation(ctx, 2 * sync, a["omega"], a["yp"], a["ys"], q0=x) for x in (None, zeros))
    args = [torch.tensor(w["mat"][k], dtype=torch.float64, device="cuda") for k in ("rho", "vp", "vs")]

    def run(sim):
        x = [t.clone().requires_grad_() for t in args]
        s = sim.seismograms(*x)
        (s * s).sum().backward()
        return [s.detach()] + [t.grad for t in x]
    first, second = run(rest), run(given)
    assert all(torch.equal(x, y) for x, y in zip(first, second)) and float(first[0].abs().max()) > 0
    assert rest.q0.shape == zeros.shape and not np.any(rest.q0)
    rest.q0[...] = synth.random_state(3, ctx.K, ctx.nq, ctx.B)    # an array once asked for: changes count
    assert not torch.equal(run(rest)[0], first[0])
    ctx.close()
