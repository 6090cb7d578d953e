"""A Simulation at rest belongs to the mesh that its context held when it was made."""
import numpy as np
import pytest
import torch


class _Context:
    """What a Simulation asks of a context, with its check of a state's size."""
    def __init__(self, K):
        self.K, self.nq, self.B, self.calls = K, 9, 4, []

    def upload_materials(self, *a):
        pass

    rewind = set_checkpointing = advance_to = upload_materials

    def set_initial(self, q):
        self.calls.append(np.ascontiguousarray(q).reshape(self.K, self.nq, self.B))


def test_rest_state_of_another_mesh_is_refused(monkeypatch):
    from paper_2202_10313_amd import autograd
    monkeypatch.setattr(autograd.torch.cuda, "current_stream", lambda d: type("S", (), {"synchronize": lambda s: None})())
    x = [torch.ones(6)] * 3
    ctx = _Context(6)
    sim = autograd.Simulation(ctx, 1.0)
    sim._forward(*x)
    assert sim.generation == 1 and not ctx.calls          # at rest: nothing is sent
    ctx.K = 7                                             # another mesh since
    with pytest.raises(ValueError):
        sim._forward(*x)
    with pytest.raises(AttributeError):
        autograd.Simulation(None, 1.0)
